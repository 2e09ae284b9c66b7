"""The tiled GEMM's pipeline at its edges: contraction axes of no whole stage to a few, with and without a partial one behind
them, on every tile shape -- exact sums (small integers), and the adapter extension behind them against the oracle."""
import numpy as np
import pytest

from workloads import make_custom

pytestmark = pytest.mark.gpu

TILES = {0: (128, 128), 1: (256, 128), 3: (64, 64), 5: (256, 256), 9: (128, 192), 10: (256, 192), 11: (256, 224), 12: (192, 128)}
RANKS = (8, 16, 64, 128, 24)


def _workload(dtype, K, rows, N, bare, integer_valued, name):
    rng = np.random.default_rng(K + rows)
    lens, ids = [], []
    while sum(lens) < rows:
        lens.append(int(min(rows - sum(lens), rng.choice([1, 3, 17, 70, 130]))))
        ids.append(-1 if bare else int(rng.integers(-1, len(RANKS))))
    return make_custom(seed=K, dtype=dtype, K=K, N=N, ranks=RANKS, scales=(0.5, 0.25, 1.0, 0.125, 2.0), req_adapter=np.asarray(ids),
                       req_ntok=np.asarray(lens), name=name, integer_valued=integer_valued)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("variant", sorted(TILES))
def test_stages_are_exact(variant, dtype):
    """No whole stage, one to five, each with and without a partial stage; one row and one column past a tile.  Integers small
    enough that every sum is exact: the oracle's results, rounded once, bit for bit."""
    from gpu_common import ctx, gpu_linear, reset_options
    from oracle import oracle_workload
    from workloads import bf16_bits_from_f32, f32_from_bf16_bits
    reset_options()
    ctx().set_option("gemm_variant", variant)
    ctx().set_option("gemm_split_k", 0)
    bm, bn = TILES[variant]
    stage = 64 if dtype == "bf16" else 32
    for stages in range(6):
        for rest in (0, 8, stage - 8):
            K = stages * stage + rest
            if K == 0:
                continue
            rows = max(bm + 1, 129)
            wl = _workload(dtype, K, rows, bn + 1 if rest else bn - 3, True, True, f"stages_{variant}_{dtype}_{K}")
            want = oracle_workload(wl)
            if dtype == "bf16":
                want = f32_from_bf16_bits(bf16_bits_from_f32(want.astype(np.float32))).astype(np.float64)
            assert np.array_equal(gpu_linear(wl), want), (stages, rest)
    reset_options()


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("variant", sorted(TILES))
def test_extension_behind_the_stages(variant, dtype):
    """The adapter term as stages behind K -- requested in front of the last stage, behind a partial one, or with no stage at
    all in front -- against the oracle, element by element within what the roundings allow: Y once, V once, and sums of K + r
    terms in fp32, each within 2^-24 of the running sum.  (A fraction of the output's RMS does not bound these: over a
    K of 8 the rows' sizes differ too much.)"""
    from gpu_common import ctx, gpu_linear, reset_options
    from oracle import oracle_workload
    from workloads import to_f64
    reset_options()
    ctx().set_option("gemm_variant", variant)
    ctx().set_option("gemm_split_k", 0)
    ctx().set_option("expand_split", 0)
    bm, bn = TILES[variant]
    stage = 64 if dtype == "bf16" else 32
    unit = 2.0 ** -8 if dtype == "bf16" else 2.0 ** -24  # half a step of the last of 8 (24) significant bits
    for K in (8, stage, stage + 8, 2 * stage, 3 * stage + 8, 4 * stage):
        wl = _workload(dtype, K, max(2 * bm + 5, 131), bn + 7, False, False, f"extension_{variant}_{dtype}_{K}")
        want = oracle_workload(wl)
        X, W = to_f64(wl.X(0)), to_f64(wl.W0(0))
        terms, term_v = np.abs(X) @ np.abs(W).T, np.zeros_like(want)
        row = 0
        for a, n in zip(wl.req_adapter, wl.req_ntok):
            if a >= 0:
                A, Bw, s, x = to_f64(wl.A(a, 0)), to_f64(wl.B(a, 0)), float(wl.scales[a]), X[row:row + n]
                term_v[row:row + n] = s * np.abs(x @ A.T) @ np.abs(Bw).T
                terms[row:row + n] += s * (np.abs(x) @ np.abs(A).T) @ np.abs(Bw).T
            row += n
        bound = unit * (np.abs(want) + term_v) * 1.01 + (K + max(RANKS)) * 2.0 ** -24 * terms
        assert (np.abs(gpu_linear(wl) - want) <= bound).all(), K
    reset_options()


@pytest.mark.parametrize("dtype,short", [("bf16", 64), ("bf16", 130), ("f32", 32), ("f32", 65)])
@pytest.mark.parametrize("variant", sorted(TILES))
def test_long_segment_behind_table_batches_without_a_column(variant, dtype, short):
    """One-row requests on adapters of rank 64, whose term comes from the expand kernel, in front of a long segment, whose term the
    GEMM computes: the first batches of the tile's column table (512 columns each) have none in use.  K of whole stages, so
    that the loads past its end are still on their way when the extension begins."""
    from gpu_common import check_against_oracle, ctx, gpu_linear, reset_options
    reset_options()
    ctx().set_option("gemm_variant", variant)
    ctx().set_option("gemm_split_k", 0)
    ctx().set_option("expand_split", 1)
    bm, bn = TILES[variant]
    for K in (64, 128, 320):
        lens = np.r_[np.ones(short, int), max(2 * bm, 130)]
        wl = make_custom(seed=K + short, dtype=dtype, K=K, N=bn + 9, ranks=np.full(short + 1, 64), scales=np.full(short + 1, 0.5),
                         req_adapter=np.arange(short + 1), req_ntok=lens, name=f"late_columns_{variant}_{dtype}_{short}_{K}")
        check_against_oracle(wl, gpu_linear(wl))
    reset_options()
