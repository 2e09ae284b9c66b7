"""Batches of more work units than two workgroups per CU: the shrink's four-wave workgroups, and the eight-wave ones that a short
contraction axis keeps (units of one row to several blocks of 64, ranks past one block of 64, K with and without a partial
stage), and the expand kernel's column groups (whole, ragged, a single column past one)."""
import numpy as np
import pytest

from workloads import make_custom

pytestmark = pytest.mark.gpu


def _workload(dtype, K, N, integer_valued):
    rng = np.random.default_rng(K + N)
    n = 300
    ranks = rng.choice([8, 24, 72, 128], n).astype(np.int32)
    lens = rng.choice([1, 1, 2, 5, 17, 40], n)
    lens[0] = 150
    ids = np.concatenate([np.arange(n - 20), np.full(20, -1)])
    return make_custom(seed=K * N, dtype=dtype, K=K, N=N, ranks=ranks, scales=np.full(n, 0.5, np.float32), req_adapter=ids, req_ntok=lens,
                       name=f"many_units_{dtype}_{K}_{N}", integer_valued=integer_valued)


@pytest.mark.parametrize("K", [72, 128, 520])
@pytest.mark.parametrize("N", [255, 256, 513])
def test_fp32_integers_are_exact(K, N):
    """Integers small enough that every sum is exact, in any order: the oracle's results bit for bit."""
    from gpu_common import ctx, gpu_linear, reset_options
    from oracle import oracle_workload
    reset_options()
    wl = _workload("f32", K, N, True)
    ctx().set_option("expand_split", 1)
    assert np.array_equal(gpu_linear(wl), oracle_workload(wl))
    reset_options()


@pytest.mark.parametrize("K,N", [(520, 257), (1024, 512), (4160, 300)])
def test_bf16_against_the_oracle(K, N):
    from gpu_common import check_against_oracle, ctx, gpu_linear, reset_options
    reset_options()
    wl = _workload("bf16", K, N, False)
    ctx().set_option("expand_split", 1)
    check_against_oracle(wl, gpu_linear(wl))
    reset_options()


@pytest.mark.parametrize("dtype,rank", [("bf16", 64), ("bf16", 128), ("bf16", 320), ("bf16", 512), ("f32", 32), ("f32", 128), ("f32", 256), ("f32", 320), ("f32", 512)])
@pytest.mark.parametrize("rows", [16, 64])
def test_expand_workgroups_are_exact(dtype, rank, rows):
    """Ranks up to those whose V leaves room for few workgroups on a CU, units of both sizes, small ranks beside the large: whole
    column groups of the two-, four- and eight-wave forms and what is left of them, integers that every sum and V in bf16 keep exactly."""
    from gpu_common import ctx, gpu_linear, reset_options
    from oracle import oracle_workload
    from workloads import bf16_bits_from_f32, f32_from_bf16_bits
    reset_options()
    n_ad = 30 if rows == 16 else 240
    rng = np.random.default_rng(rank)
    lens = rng.choice([1, 2, 5, 17], n_ad)
    for N in (1024, 1300):
        ranks = np.where(np.arange(n_ad) % 3 == 0, 8, rank).astype(np.int32)
        wl = make_custom(seed=rank + rows, dtype=dtype, K=16, N=N, ranks=ranks, scales=np.full(n_ad, 0.5, np.float32), req_adapter=np.arange(n_ad),
                         req_ntok=np.r_[70, lens[1:]], name=f"wide_expand_{dtype}_{rank}_{rows}_{N}", integer_valued=True)
        ctx().set_option("gemm_variant", 0)
        ctx().set_option("gemm_split_k", 0)
        ctx().set_option("expand_split", 1)
        want = oracle_workload(wl)
        if dtype == "bf16":
            want = f32_from_bf16_bits(bf16_bits_from_f32(want.astype(np.float32))).astype(np.float64)
        got, (_, _, _, pl, _) = gpu_linear(wl, return_all=True)
        assert pl.struct.unit_rows == rows
        assert np.array_equal(got, want)
    reset_options()
