"""The hot path under HIP graph capture: `lora_plan_device` + `lora_linear` (and `lora_linear_multi`) only launch
kernels -- no allocation, no synchronisation, no memset node -- so a captured step replays with new activations and
a new batch composition in the same buffers and gives, bit for bit, what the eager calls give."""
import numpy as np
import pytest
import torch

from workloads import make_custom
from workloads.configs import Projection

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("case", ["prefill_mixed", "decode", "split_k", "decode_much_adapter_work"])
def test_captured_step_replays_bit_exact(case):
    from gpu_common import B, rt, ctx, reset_options
    c = ctx()
    dev = c.device
    K, Ns, ranks = 264, (520, 264), (8, 16, 64, 40, 8, 24, 32, 48)
    if case == "prefill_mixed":  # long and short segments: shrink, separate expand kernel, tiled GEMM
        ids = [3, 0, -1, 5, 3, 1, 6, 2, 5, 3, 0, 4, -1, 6]
        L = [150, 1, 9, 64, 150, 63, 1, 17, 0, 141, 2, 5, 30, 1]
    elif case == "decode":  # decode-sized: the two launches of the decode path
        ids = [1, 1, 4, -1, 0, 7, 2, 2, 6, 5, 3, 0]
        L = [1] * 12
    elif case == "split_k":  # a few hundred rows, a long contraction axis: the GEMM split along K + the launch that sums
        ids = [3, 0, -1, 5, 3, 1, 6, 2]
        L = [70, 1, 9, 64, 90, 33, 1, 17]
        K = 2312
        assert "splitk" in B.lora_gemm_kernel_name(c.handle, sum(L), K, Ns[0], 1)
    else:  # 64 one-token requests on adapters of rank 128: the finishing kernel behind the stream
        ids = [i % 8 for i in range(64)]
        L = [1] * 64
        K, Ns, ranks = 520, (1544, 1536), (128,) * 8
    wl = make_custom(seed=970, dtype="bf16", K=K, N=Ns[0], ranks=ranks,
                     scales=(2.0, 0.5, 1.0, 0.25, 1.5, 1.0, 0.75, 1.0), req_adapter=np.asarray(ids), req_ntok=np.asarray(L),
                     name=f"graph_{case}")
    wl.projections = [Projection("a", K, Ns[0]), Projection("b", K, Ns[1])]
    wl.shared_x = True
    T, r_max = wl.T, wl.r_max
    up = [rt.upload_workload(wl, q, dev) for q in range(2)]
    X = up[0][0].clone()
    ra = torch.from_numpy(np.ascontiguousarray(wl.req_adapter)).to(dev)
    rn = torch.from_numpy(np.ascontiguousarray(wl.req_ntok)).to(dev)
    rk = torch.from_numpy(np.ascontiguousarray(wl.ranks)).to(dev)
    nbytes = B.lora_plan_bytes(wl.n_req, T, wl.n_adapters, r_max)

    def buffers():
        plan_buf = torch.empty(nbytes, dtype=torch.uint8, device=dev)
        Ys = [torch.zeros((T, u[1].shape[0]), dtype=X.dtype, device=dev) for u in up]
        wss = [rt.workspace(T, K, u[1].shape[0], r_max, X.dtype, dev) for u in up]
        return plan_buf, Ys, wss

    def step(plan_buf, Ys, wss):  # plan + one projection alone + both through the multi call, on the current stream
        st = int(torch.cuda.current_stream().cuda_stream)
        plan = B.lora_plan_device(c.handle, ra.data_ptr(), rn.data_ptr(), wl.n_req, rk.data_ptr(), wl.n_adapters, r_max, T,
                                  plan_buf.data_ptr(), nbytes, st)
        pl = rt.Plan(plan, plan_buf)
        d = [rt.linear_desc(pl, X, up[q][1], Ys[q], up[q][2], wss[q]) for q in range(2)]
        B.lora_linear(c.handle, plan, d[0], st)
        B.lora_linear_multi(c.handle, plan, d, st)
        return d

    g_bufs, e_bufs = buffers(), buffers()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):  # first calls outside the capture (they set kernel attributes)
        keep = step(*g_bufs)
    side.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        keep = step(*g_bufs)
    rng = np.random.default_rng(5)
    for trial in range(3):
        # new activations, and from the second replay on another batch composition of the same size
        X.copy_(torch.from_numpy(rng.standard_normal((T, K)).astype(np.float32)).to(dev).to(X.dtype))
        if trial > 0:
            perm = torch.from_numpy(rng.permutation(wl.n_req)).to(dev)
            ra.copy_(ra[perm].clone())
            rn.copy_(rn[perm].clone())
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        step(*e_bufs)  # the same step eagerly, into buffers of its own
        torch.cuda.synchronize()
        for q in range(2):
            assert torch.equal(g_bufs[1][q].view(torch.int16), e_bufs[1][q].view(torch.int16)), (case, trial, q)
        assert float(g_bufs[1][0].float().abs().max()) > 0
    reset_options()


@pytest.mark.parametrize("case", ["decode", "decode_much_adapter_work", "prefill"])
def test_captured_layers_follow_a_plan_rebuilt_by_lora_plan(case):
    """Only the layers are captured, on a plan of one small adapter; lora_plan() then fills the same buffer, outside the graph,
    for batches of the same sizes that use every adapter.  Each replay gives what eager calls on that plan give."""
    from gpu_common import B, ctx, reset_options, rt
    reset_options()
    c = ctx()
    dev = c.device
    K, N, T = 520, 1544, 64 if case != "prefill" else 300
    n_ad, r = 24, 128 if case == "decode_much_adapter_work" else 16
    ranks = np.full(n_ad, r, np.int32)
    ranks[0] = 8
    wl = make_custom(seed=971, dtype="bf16", K=K, N=N, ranks=ranks, scales=np.linspace(0.5, 2.0, n_ad), req_adapter=np.zeros(T, int),
                     req_ntok=np.ones(T, int), name=f"replan_{case}")
    X, W0, table = rt.upload_workload(wl, 0, dev)
    rng = np.random.default_rng(8)
    batches = [np.zeros(T, int), rng.integers(-1, n_ad, T), np.arange(T) % n_ad, np.full(T, -1)]
    buf = torch.empty(B.lora_plan_bytes(T, T, n_ad, r), dtype=torch.uint8, device=dev)
    pl = rt.plan(c, batches[0], np.ones(T, int), ranks, r, buf=buf)
    Y, Ym, Ys = (torch.zeros((T, N), dtype=X.dtype, device=dev) for _ in range(3))
    ws = [rt.workspace(T, K, N, r, X.dtype, dev) for _ in range(3)]
    d = [rt.linear_desc(pl, X, W0, y, table, w) for y, w in zip((Y, Ym, Ys), ws)]
    side = torch.cuda.Stream()

    def layers():
        st = torch.cuda.current_stream().cuda_stream
        B.lora_linear(c.handle, pl.struct, d[0], st)
        B.lora_linear_multi(c.handle, pl.struct, [d[1], d[2]], st)

    def staged(first):  # the first stage eagerly, the second from its own graph
        st = torch.cuda.current_stream().cuda_stream
        (B.lora_shrink if first else B.lora_gemm_expand)(c.handle, pl.struct, d[0], st)

    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        layers()
    side.synchronize()
    graph, second = torch.cuda.CUDAGraph(), torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        layers()
    with torch.cuda.graph(second, stream=side):
        staged(False)
    for ids in batches[1:] + batches[:1]:
        now = rt.plan(c, ids, np.ones(T, int), ranks, r, buf=buf)
        for y in (Y, Ym, Ys):
            y.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        want = rt.linear(c, now, X, W0, table)
        for y in (Y, Ym, Ys):
            assert torch.equal(y.view(torch.int16), want.view(torch.int16)), (case, ids[:8])
        Y.fill_(float("nan"))
        B.lora_shrink(c.handle, now.struct, d[0], torch.cuda.current_stream().cuda_stream)
        second.replay()
        torch.cuda.synchronize()
        assert torch.equal(Y.view(torch.int16), want.view(torch.int16)), (case, ids[:8])
    reset_options()


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("used", [60, 1000])
def test_results_do_not_depend_on_the_grids_bound(dtype, used):
    """1000 slots, some or all of them in use: the shrink has a few workgroups or more than 512 by what lora_plan() knows, and more
    than 512 by the sizes.  Eagerly, alone and beside two other projections, on a plan built on the device, and replayed: the
    same bits."""
    from gpu_common import B, ctx, reset_options, rt
    reset_options()
    c = ctx()
    dev = c.device
    K, N, T, n_ad, r = 1032, 264, 1500, 1000, 64
    rng = np.random.default_rng(used)
    ranks = rng.choice([8, 16, 40, 64], n_ad).astype(np.int32)
    wl = make_custom(seed=972, dtype=dtype, K=K, N=N, ranks=ranks, scales=np.linspace(0.5, 2.0, n_ad), req_adapter=np.arange(T) % used,
                     req_ntok=np.ones(T, int), name=f"bound_{dtype}_{used}")
    X, W0, table = rt.upload_workload(wl, 0, dev)
    ids, ones = np.ascontiguousarray(wl.req_adapter).astype(np.int32), np.ones(T, np.int32)
    bits = lambda y: y.view(torch.int16 if dtype == "bf16" else torch.int32)
    pl = rt.plan(c, ids, ones, ranks, r)
    want = rt.linear(c, pl, X, W0, table)
    for y in rt.linear_multi(c, pl, X, [(W0, table)] * 3):
        assert torch.equal(bits(y), bits(want))
    dpl = rt.plan_device(c, *(torch.from_numpy(v).to(dev) for v in (ids, ones, ranks)), r, T)
    assert torch.equal(bits(rt.linear(c, dpl, X, W0, table)), bits(want))
    Y = torch.zeros((T, N), dtype=X.dtype, device=dev)
    ws = rt.workspace(T, K, N, r, X.dtype, dev)
    d = rt.linear_desc(pl, X, W0, Y, table, ws)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        B.lora_linear(c.handle, pl.struct, d, torch.cuda.current_stream().cuda_stream)
    for _ in range(3):
        Y.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(bits(Y), bits(want))
    reset_options()
