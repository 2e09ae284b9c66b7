"""lora_plan() at the edges of the route that hands the device a table made by the host: the largest batch it takes and the
first one beyond it, empty requests, and more plans in flight than there are tables (bit-exact, as all plan tests)."""
import numpy as np
import pytest

from test_gpu_plan import _check_plan

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("R,T,n_ad", [(1, 1, 1), (2048, 2048, 2048), (2049, 4000, 300), (300, 16384, 40), (300, 16385, 40), (2048, 9000, 5000)])
def test_plan_from_host_arrays_at_the_edges(R, T, n_ad):
    rng = np.random.default_rng(R + T)
    cuts = np.sort(rng.integers(0, T + 1, R - 1))
    L = np.diff(np.concatenate([[0], cuts, [T]]))  # empty requests among them
    ids = rng.integers(-1, n_ad, R) if R > 1 else [0]
    _check_plan(ids, L, rng.choice([8, 16, 64], n_ad), False)


@pytest.mark.parametrize("variant", [0, 1])
@pytest.mark.parametrize("R", [1, 64, 65, 128, 300])
def test_host_arrays_through_the_device_s_builders(R, variant):
    """The upload and the builders behind it, which larger batches and stream capture take: mixed keys, and the same key in every
    lane of a wave."""
    rng = np.random.default_rng(R)
    ranks = rng.choice([8, 16, 64], 50)
    _check_plan(rng.integers(-1, 50, R), rng.integers(0, 4, R), ranks, False, plan_variant=variant)
    _check_plan(np.full(R, 7), np.ones(R, int), ranks, False, plan_variant=variant)
    _check_plan(np.full(R, -1), np.ones(R, int), ranks, False, plan_variant=variant)


def test_rank_axis_longer_than_one_workgroup_serves():
    _check_plan(np.arange(300), np.ones(300, int), np.full(300, 512), False)      # 19200 records: beyond the table's limit
    _check_plan(np.arange(256), np.ones(256, int), np.full(256, 512), False)      # 16384: at it


def test_more_plans_in_flight_than_tables():
    import torch
    from gpu_common import ctx, plan_reference, rt
    c = ctx()
    rng = np.random.default_rng(3)
    batches = [(rng.integers(-1, 9, 50 + i), rng.integers(0, 4, 50 + i)) for i in range(40)]
    ranks = rng.choice([8, 16, 32], 9)
    torch.cuda.synchronize()
    x = torch.randn(8192, 8192, device=c.device)
    x @ x  # (keeps the stream busy while the plans queue up)
    plans = [rt.plan(c, ids, L, ranks) for ids, L in batches]
    for (ids, L), pl in zip(batches, plans):
        got, ref = pl.to_host(c), plan_reference(ids.astype(np.int32), L.astype(np.int32), ranks.astype(np.int32))
        for k in ("perm", "row_seg", "seg_adapter", "seg_indptr", "seg_rank", "seg_ext"):
            assert np.array_equal(got[k], ref[k]), k


def test_plans_behind_a_stream_that_stays_busy():
    """The stream is busy for longer than lora_plan() waits for a table: the plans beyond the sixteenth are uploaded instead."""
    import torch
    from gpu_common import ctx, plan_reference, rt
    c = ctx()
    rng = np.random.default_rng(6)
    ranks = rng.choice([8, 16, 32], 9)
    batches = [(rng.integers(-1, 9, 30 + i), rng.integers(0, 4, 30 + i)) for i in range(19)]
    x = torch.randn(8192, 8192, device=c.device)
    torch.cuda.synchronize()
    for _ in range(100):  # (fp32, ~9 ms each)
        y = x @ x
    plans = [rt.plan(c, ids, L, ranks) for ids, L in batches]
    busy = not torch.cuda.current_stream().query()
    for (ids, L), pl in zip(batches, plans):
        got, ref = pl.to_host(c), plan_reference(ids.astype(np.int32), L.astype(np.int32), ranks.astype(np.int32))
        for k in ("perm", "row_seg", "seg_adapter", "seg_indptr", "seg_rank", "seg_ext"):
            assert np.array_equal(got[k], ref[k]), k
    assert busy and bool(torch.isfinite(y).all())


def test_pending_error_of_another_call():
    """A HIP call refused before lora_plan() (an argument error, nothing on the GPU) says nothing about the plan's launch: plans
    of different sizes queued behind other work all come out right."""
    import torch
    from gpu_common import B, ctx, plan_reference, rt
    c = ctx()
    hip = B.lib()  # (its own HIP runtime: dependencies of the library are searched too)
    rng = np.random.default_rng(4)
    ranks = rng.choice([8, 16, 32], 9).astype(np.int32)
    batches = [(rng.integers(-1, 9, n).astype(np.int32), rng.integers(0, 5, n).astype(np.int32)) for n in (400, 3, 64, 1, 200, 7)]
    bufs = [torch.empty(B.lora_plan_bytes(len(i), int(L.sum()), 9, 32), dtype=torch.uint8, device=c.device) for i, L in batches]
    torch.cuda.synchronize()
    st = torch.cuda.current_stream().cuda_stream
    x = torch.randn(8192, 8192, device=c.device)
    x @ x
    structs = []
    for (ids, L), buf in zip(batches, bufs):
        assert hip.hipSetDevice(1 << 20) != 0
        structs.append(B.lora_plan(c.handle, ids, L, ranks, 32, int(L.sum()), buf.data_ptr(), buf.numel(), st))
    hip.hipGetLastError()  # (torch would blame its next call)
    for (ids, L), buf, struct in zip(batches, bufs, structs):
        got, ref = rt.Plan(struct, buf).to_host(c), plan_reference(ids, L, ranks)
        for k in ("perm", "row_seg", "seg_adapter", "seg_indptr", "seg_rank", "seg_ext"):
            assert np.array_equal(got[k], ref[k]), k
