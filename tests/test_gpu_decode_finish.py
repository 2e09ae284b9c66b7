"""The decode path's second launch for batches with much adapter work (one work unit of the plan and 512 output columns per
workgroup), at the edges of its tiles, against the oracle: the bf16 tolerance of the layer, as everywhere (outputs rounded
to bf16: 2^-9 of a value of up to ~5 times the output's RMS, plus V rounded to bf16)."""
import numpy as np
import pytest

from workloads import make_custom, to_f64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,K,N,ranks", [
    (1, 64, 512, (8,)),                    # one row, one column group, one chunk of rank
    (16, 520, 513, (64, 8)),               # a full unit, one column past a group, a second slice of one chunk
    (17, 512, 511, (72,)),                 # a unit of one row behind a full one, rank just past one pass of 64
    (40, 4104, 1024, (128, 136, 512)),     # nine slices; ranks of one pass, just past it, and the largest
    (128, 264, 1537, (16, 32, 256, 8)),    # the largest batch, ragged last group
])
def test_finishing_launch_at_tile_edges(T, K, N, ranks):
    from gpu_common import check_against_oracle, ctx, gpu_linear, reset_options
    reset_options()
    rng = np.random.default_rng(T + N)
    ids = rng.integers(-1 if T > 16 else 0, len(ranks), size=T)
    if T > 64:
        ids[:40] = -1  # more rows without an adapter than one unit holds
    wl = make_custom(seed=3000 + T, dtype="bf16", K=K, N=N, ranks=ranks, scales=[16.0 / r for r in ranks], req_adapter=ids,
                     req_ntok=np.ones(T, np.int64), name=f"finish_T{T}_N{N}")
    ctx().set_option("expand_split", 1)
    for device_plan in (False, True):
        check_against_oracle(wl, gpu_linear(wl, device_plan=device_plan))
    reset_options()


def test_one_call_with_projections_of_both_kinds():
    """Three projections of one call: two with much adapter work (their own second launch), a narrow one without; each
    bit-equal to its single call."""
    import torch
    from workloads.configs import Projection
    from gpu_common import check_against_oracle, ctx, reset_options, rt
    reset_options()
    c = ctx()
    rng = np.random.default_rng(9)
    wl = make_custom(seed=3100, dtype="bf16", K=520, N=1100, ranks=(256, 8, 64, 512), scales=(0.1, 2.0, 0.5, 0.05),
                     req_adapter=rng.integers(-1, 4, size=100), req_ntok=np.ones(100, np.int64), name="finish_multi")
    wl.projections = [Projection("a", 520, 1100), Projection("b", 520, 48), Projection("c", 520, 640)]  # 113, 5, 66 MB of gathers
    wl.shared_x = True
    up = [rt.upload_workload(wl, q, c.device) for q in range(3)]
    pl = rt.plan(c, wl.req_adapter, wl.req_ntok, wl.ranks)
    outs = rt.linear_multi(c, pl, up[0][0], [(u[1], u[2]) for u in up])
    torch.cuda.synchronize()
    for q, u in enumerate(up):
        got = rt.bits_from_tensor(outs[q])
        assert np.array_equal(got, rt.bits_from_tensor(rt.linear(c, pl, up[0][0], u[1], u[2])))
        check_against_oracle(wl, to_f64(got), p=q)


def test_v_is_not_rounded_with_a_workspace_below_the_preferred_size():
    """Much adapter work and a minimal workspace: with small integers every sum is exact in fp32 while V needs more bits than bf16
    has (|V| up to several hundred), so Y is the exact result rounded once, bit for bit."""
    import torch
    from gpu_common import ctx, reset_options, rt
    from oracle import oracle_workload
    from workloads import bf16_bits_from_f32
    reset_options()
    c = ctx()
    T, K, N = 64, 520, 1544
    wl = make_custom(seed=3200, dtype="bf16", K=K, N=N, ranks=(128,) * 64, scales=(1.0,) * 64, req_adapter=np.arange(T),
                     req_ntok=np.ones(T, np.int64), name="finish_minimal", integer_valued=True)
    want = bf16_bits_from_f32(oracle_workload(wl).astype(np.float32))
    X, W0, table = rt.upload_workload(wl, 0, c.device)
    pl = rt.plan(c, wl.req_adapter, wl.req_ntok, wl.ranks)
    ws = [rt.workspace(T, K, N, pl.r_max, X.dtype, c.device, minimal=True) for _ in range(2)]
    Ys = [torch.empty((T, N), dtype=X.dtype, device=c.device) for _ in range(2)]
    rt.linear(c, pl, X, W0, table, Y=Ys[0], ws=ws[0])
    assert np.array_equal(rt.bits_from_tensor(Ys[0]), want)
    d = [rt.linear_desc(pl, X, W0, y, table, w) for y, w in zip(Ys, ws)]
    for y in Ys:
        y.fill_(float("nan"))
    rt.B.lora_linear_multi(c.handle, pl.struct, d, torch.cuda.current_stream().cuda_stream)
    for y in Ys:
        assert np.array_equal(rt.bits_from_tensor(y), want)
    reset_options()
