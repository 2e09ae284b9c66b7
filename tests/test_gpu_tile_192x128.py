"""The 192x128 tile of the tiled GEMM: alone, and split along K for mid-sized batches."""
import numpy as np
import pytest

from workloads import make_custom

pytestmark = pytest.mark.gpu

RANKS = (8, 16, 64, 128, 24)


def _batch(seed, T):
    rng = np.random.default_rng(seed)
    lens, ids = [], []
    while sum(lens) < T:
        lens.append(int(min(T - sum(lens), rng.choice([1, 2, 5, 40, 70, 150]))))
        ids.append(int(rng.integers(-1, len(RANKS))))
    return np.asarray(ids), np.asarray(lens)


# (rows: one tile, its edges, several with a ragged last one; columns: less than a tile, a multiple, ragged)
# (the split along K of this tile is bf16's alone)
@pytest.mark.parametrize("T,K,N,split,dtype", [(191, 520, 100, False, "bf16"), (193, 1000, 256, False, "bf16"), (700, 1000, 300, False, "bf16"),
                                               (191, 520, 100, False, "f32"), (193, 1000, 256, False, "f32"), (700, 1000, 300, False, "f32"),
                                               (150, 8264, 4097, True, "bf16"), (385, 8200, 2816, True, "bf16"), (577, 8264, 4000, True, "bf16")])
def test_integer_inputs_are_exact(T, K, N, split, dtype):
    """Integers small enough that every partial sum is exact in fp32, in any order: fp32 results are the oracle's bit for
    bit; bf16 ones, on requests without adapters (no rounded V), are the exact sums rounded once."""
    from gpu_common import B, ctx, gpu_linear, reset_options
    from oracle import oracle_workload
    from workloads import bf16_bits_from_f32, f32_from_bf16_bits
    reset_options()
    ids, lens = _batch(T + K, T)
    if dtype == "bf16":
        ids = np.full_like(ids, -1)
    wl = make_custom(seed=700 + T, dtype=dtype, K=K, N=N, ranks=RANKS, scales=(0.5, 0.25, 1.0, 0.125, 2.0), req_adapter=ids,
                     req_ntok=lens, name=f"tile192_{dtype}_{T}_{K}_{N}", integer_valued=True)
    Yo = oracle_workload(wl)
    if dtype == "bf16":
        Yo = f32_from_bf16_bits(bf16_bits_from_f32(Yo.astype(np.float32))).astype(np.float64)
    if split:
        assert B.lora_gemm_kernel_name(ctx().handle, T, K, N, 1).startswith("tile_192x128_splitk")
    else:
        ctx().set_option("gemm_variant", 12)
        ctx().set_option("gemm_split_k", 0)
        assert B.lora_gemm_kernel_name(ctx().handle, T, K, N, 1 if dtype == "bf16" else 0) == "tile_192x128"
    assert np.array_equal(gpu_linear(wl), Yo)
    reset_options()


@pytest.mark.parametrize("T,expand_split", [(385, -1), (385, 1), (700, 0), (700, 1)])
def test_adapters(T, expand_split):
    """The fused extension, the expand kernel's term in the epilogue and the split's sum, bf16, against the oracle."""
    from gpu_common import check_against_oracle, ctx, gpu_linear, reset_options
    reset_options()
    K, N = (8200, 2816) if T == 385 else (1000, 300)
    ids, lens = _batch(T, T)
    wl = make_custom(seed=800 + T, dtype="bf16", K=K, N=N, ranks=RANKS, scales=(0.5, 0.25, 1.0, 0.125, 2.0), req_adapter=ids,
                     req_ntok=lens, name=f"tile192_adapters_{T}")
    if T == 700:
        ctx().set_option("gemm_variant", 12)
    ctx().set_option("expand_split", expand_split)
    check_against_oracle(wl, gpu_linear(wl))
    reset_options()


@pytest.mark.parametrize("T,K,N", [(150, 8264, 4097), (250, 8200, 2816), (129, 4104, 1000)])
def test_fewer_stretches_in_a_smaller_workspace(T, K, N):
    """A workspace with room for some of the partial outputs only, down to none: exact sums rounded once, whatever the split."""
    from gpu_common import B, ctx, reset_options, rt
    import torch
    from oracle import oracle_workload
    from workloads import bf16_bits_from_f32
    reset_options()
    c = ctx()
    ids, lens = _batch(T + K, T)
    wl = make_custom(seed=900 + T, dtype="bf16", K=K, N=N, ranks=RANKS, scales=(0.5, 0.25, 1.0, 0.125, 2.0), req_adapter=np.full_like(ids, -1),
                     req_ntok=lens, name=f"fewer_{T}_{K}_{N}", integer_valued=True)
    want = bf16_bits_from_f32(oracle_workload(wl).astype(np.float32))
    name = B.lora_gemm_kernel_name(c.handle, T, K, N, 1)
    assert "splitk" in name
    X, W0, table = rt.upload_workload(wl, 0, c.device)
    pl = rt.plan(c, wl.req_adapter, wl.req_ntok, wl.ranks)
    size = B.lora_linear_workspace_bytes_preferred(T, K, N, pl.r_max, 1)
    one = T * ((N + 7) // 8 * 8) * 4
    for less in range(int(name.rpartition("splitk")[2]) + 1):
        ws = torch.empty(size - less * one, dtype=torch.uint8, device=c.device)
        Y = rt.linear(c, pl, X, W0, table, ws=ws)
        assert np.array_equal(rt.bits_from_tensor(Y), want), less


def test_fewer_stretches_with_adapters():
    """The same with the adapter term, whose room lies in front of the partial outputs, against the oracle."""
    from gpu_common import B, check_against_oracle, ctx, reset_options, rt
    import torch
    from workloads import to_f64
    reset_options()
    c = ctx()
    T, K, N = 150, 8264, 1200
    ids, lens = _batch(T, T)
    wl = make_custom(seed=950, dtype="bf16", K=K, N=N, ranks=RANKS, scales=(0.5, 0.25, 1.0, 0.125, 2.0), req_adapter=ids, req_ntok=lens,
                     name="fewer_adapters")
    most = int(B.lora_gemm_kernel_name(c.handle, T, K, N, 1).rpartition("splitk")[2])
    X, W0, table = rt.upload_workload(wl, 0, c.device)
    pl = rt.plan(c, wl.req_adapter, wl.req_ntok, wl.ranks)
    size = B.lora_linear_workspace_bytes_preferred(T, K, N, pl.r_max, 1)
    for less in range(most + 2):
        ws = torch.full((size - less * T * N * 4,), 255, dtype=torch.uint8, device=c.device)
        check_against_oracle(wl, to_f64(rt.bits_from_tensor(rt.linear(c, pl, X, W0, table, ws=ws))))
