"""What the layer's entry points launch, on a stand-in HIP runtime: grids, kernels and the workspace they ask for."""
import pytest

import fake_hip


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    return fake_hip.build(tmp_path_factory.mktemp("fake_hip"))


@pytest.mark.parametrize("T,K,N", [(64, 520, 1544), (64, 4096, 4096), (128, 264, 320), (300, 520, 700), (700, 4096, 512)])
def test_captured_launches_have_room_for_every_batch_of_the_same_sizes(fake, T, K, N):
    """A captured layer may be replayed after lora_plan() has filled the buffer for another batch of the same sizes: its grids
    must not depend on what the batch at capture used.  Eager launches are for the plan at hand and may be smaller."""
    fake_hip.run(fake, f"""
        T, K, N = {T}, {K}, {N}
        ranks = np.full(64, 128)
        one = make_plan(np.zeros(64, int), np.diff(np.linspace(0, T, 65).astype(int)), np.where(np.arange(64) == 0, 8, 128), r_max=128)
        many = make_plan(np.arange(64), np.diff(np.linspace(0, T, 65).astype(int)), ranks, r_max=128)

        def grids(plan):
            d = [make_desc(plan, K, n) for n in (N, N + 16)]
            d[1].X = d[0].X
            out = []
            for call in (lambda: B.lora_linear(ctx, plan, d[0], 0), lambda: B.lora_linear_multi(ctx, plan, d, 0),
                         lambda: B.lora_shrink(ctx, plan, d[0], 0), lambda: B.lora_gemm_expand(ctx, plan, d[0], 0)):
                F.fake_reset()
                say("capturing", capturing)
                call()
                assert F.fake_launches() > 0
                out.append(launched())
            return out

        capturing = 1
        assert grids(one) == grids(many)
        captured = grids(one)
        capturing = 0
        assert grids(many) == captured  # (this batch uses all that its sizes allow)
        area = lambda launches: sum(g[0] * g[1] * g[2] for _, g, _ in launches)
        assert all(area(e) <= area(c) for e, c in zip(grids(one), captured))
    """)
