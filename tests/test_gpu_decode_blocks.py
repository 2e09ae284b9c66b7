"""Decode-sized batches at the edges of their 16-row blocks (every block count has kernels of its own)."""
import numpy as np
import pytest

from workloads import make_custom

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [1, 15, 17, 32, 33, 47, 48, 49, 65, 79, 80, 81, 97, 111, 112, 113, 128])
@pytest.mark.parametrize("expand_split", [0, 1])
def test_block_edges(T, expand_split):
    """Both second launches (reduction; one work unit per workgroup), rows with and without an adapter, a partial last
    slice of K and ragged columns; the workspace starts as NaN, so a row that was not stored cannot pass as zero."""
    import torch
    from gpu_common import check_against_oracle, ctx, reset_options, rt
    reset_options()
    ranks = (8, 16, 64, 40)
    rng = np.random.default_rng(T)
    wl = make_custom(seed=60 + T, dtype="bf16", K=1096, N=300, ranks=ranks, scales=(2.0, 0.5, 1.0, 0.25),
                     req_adapter=rng.integers(-1, len(ranks), size=T), req_ntok=np.ones(T, int), name=f"decode_block_{T}")
    ctx().set_option("gemm_variant", 4)
    ctx().set_option("expand_split", expand_split)
    X, W0, table = rt.upload_workload(wl, 0, ctx().device)
    plan = rt.plan(ctx(), wl.req_adapter, wl.req_ntok, wl.ranks)
    ws = rt.workspace(wl.T, 1096, 300, plan.r_max, X.dtype, ctx().device)
    ws.fill_(255)
    Y = rt.linear(ctx(), plan, X, W0, table, ws=ws)
    torch.cuda.synchronize()
    check_against_oracle(wl, rt_to_f64(Y))
    reset_options()


def rt_to_f64(Y):
    return Y.double().cpu().numpy()
