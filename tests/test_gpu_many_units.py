"""Batches of more work units than two workgroups per CU: the shrink's four-wave workgroups (units of one row to several blocks of
64, ranks past one block of 64, a contraction axis with and without a partial stage, fewer stages than waves) and the expand
kernel's column groups (whole, ragged, a single column past one)."""
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
