"""Infinities and NaN in one adapter's B_a, the adapter term inside the tiled GEMM: the MFMA multiplies 16 rows at a time, so rows
that share a 16-row block of the plan's order with the adapter's may turn NaN (0 x inf); no other row changes by a bit."""
import numpy as np
import pytest
import torch

from test_gpu_tile_stages import TILES

pytestmark = pytest.mark.gpu

RANKS = (16, 16, 8, 8, 8, 24, 40, 16)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("variant", sorted(TILES))
def test_other_adapters_rows_stay_as_they_are(variant, dtype):
    from gpu_common import ctx, plan_reference, reset_options, rt
    reset_options()
    c = ctx()
    c.set_option("gemm_variant", variant)
    c.set_option("gemm_split_k", 0)
    c.set_option("expand_split", 0)
    bm, bn = TILES[variant]
    K, N = 136, bn + 5
    rng = np.random.default_rng(variant)
    ids = np.r_[np.arange(len(RANKS)), -1, np.arange(len(RANKS))].astype(np.int32)
    ntok = np.maximum(rng.multinomial(2 * bm + 100, np.full(len(ids), 1 / len(ids))), 1).astype(np.int32)
    ranks, T = np.asarray(RANKS, np.int32), int(ntok.sum())
    gen = torch.Generator(device=c.device).manual_seed(variant)
    normal = lambda *shape: torch.randn(shape, generator=gen, device=c.device, dtype=dtype)
    X, W0, A = normal(T, K), normal(N, K), [normal(r, K) for r in RANKS]
    Bw = [normal(N, r) for r in RANKS]
    pl = rt.plan(c, ids, ntok, ranks)
    bits = torch.int16 if dtype == torch.bfloat16 else torch.int32
    clean = rt.linear(c, pl, X, W0, rt.AdapterTable(A, Bw, np.ones(len(RANKS)), c.device)).view(bits)
    perm = np.asarray(plan_reference(ids, ntok, ranks)["perm"])
    owner = np.repeat(ids, ntok)[perm]  # adapter of every slot
    for bad in range(len(RANKS)):
        Bbad = list(Bw)
        Bbad[bad] = Bw[bad].clone()
        Bbad[bad][::3] = float("inf")
        Bbad[bad][1::3] = float("nan")
        Y = rt.linear(c, pl, X, W0, rt.AdapterTable(A, Bbad, np.ones(len(RANKS)), c.device))
        reached = np.isin(np.arange(T) // 16, np.unique(np.flatnonzero(owner == bad) // 16))
        same = (Y.view(bits) == clean).all(dim=1).cpu().numpy()[perm]
        assert same[~reached].all(), (bad, owner[~reached & ~same][:8])
        assert not same[owner == bad].any(), bad
    reset_options()
