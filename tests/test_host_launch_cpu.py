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


@pytest.mark.parametrize("T,rank,sets,block", [(700, 16, 1, 8), (700, 16, 3, 16), (400, 64, 1, 16), (400, 64, 3, 32), (1216, 16, 2, 16)])
def test_shrink_rank_blocks_count_every_projection(fake, T, rank, sets, block):
    """Above 256 rows a unit's ranks are dealt out while the launch, all its projections together, has at most a workgroup per CU."""
    fake_hip.run(fake, f"""
        T, rank, sets, block = {T}, {rank}, {sets}, {block}
        plan = make_plan(np.arange(16), np.diff(np.linspace(0, T, 17).astype(int)), np.full(16, rank))
        assert plan.unit_rows == 16
        d = [make_desc(plan, 4096, 4096) for _ in range(sets)]
        for v in d:
            v.X = d[0].X

        def shrink():
            F.fake_reset()
            B.lora_linear_multi(ctx, plan, d, 0)
            return [l for l in launched() if "shrink_kernel" in l[0]]

        chosen = shrink()
        assert len(chosen) == 1
        B.lora_ctx_set_option(ctx, "shrink_rank_block", block)
        assert chosen == shrink()
        B.lora_ctx_set_option(ctx, "shrink_rank_block", 8)
        assert (chosen == shrink()) == (block == 8)
    """)


@pytest.mark.parametrize("T,n_ad,K,dtype,waves", [
    (200, 100, 4096, 1, 8), (200, 100, 4096, 0, 8), (200, 100, 5120, 1, 8), (256, 250, 1024, 0, 8), (257, 250, 1024, 0, 4),
    (257, 250, 4096, 1, 4), (600, 20, 4096, 1, 8), (1500, 600, 136, 1, 8), (1500, 600, 512, 1, 4), (1500, 600, 256, 0, 4),
    (1500, 600, 8184, 1, 4), (1500, 600, 8192, 1, 8), (1500, 600, 11008, 1, 8), (1500, 600, 4088, 0, 4), (1500, 600, 4096, 0, 8)])
def test_shrink_waves_of_a_workgroup(fake, T, n_ad, K, dtype, waves):
    """Four waves only where two such workgroups fit a CU (no staging of X, which batches of at most 256 rows have), the grid
    has more than two per CU, and a row of X is from 1 KB -- a stage for each of the eight slices -- to 16 KB long.  A plan built on the
    device, whose grid is for every slot, gets eight."""
    fake_hip.run(fake, f"""
        T, n_ad, K, waves, dtype = {T}, {n_ad}, {K}, {waves}, {dtype}
        plan = make_plan(np.arange(T) % n_ad, np.ones(T, int), np.full(n_ad, 64))
        B.lora_ctx_set_option(ctx, "gemm_variant", 0)  # (tiles at decode sizes too)
        d = [make_desc(plan, K, 264, dtype) for _ in range(3)]
        for v in d:
            v.X = d[0].X

        def shrink(plan):
            F.fake_reset()
            B.lora_linear_multi(ctx, plan, d, 0)
            return [b for name, _, b in launched() if "shrink_kernel" in name]

        assert shrink(plan) == [(64 * waves, 1, 1)], shrink(plan)
        n = B.lora_plan_bytes(T, T, n_ad, 64)
        device = B.lora_plan_device(ctx, mem(4 * T), mem(4 * T), T, mem(4 * n_ad), n_ad, 64, T, mem(n), n, 0)
        assert shrink(device) == [(512, 1, 1)], shrink(device)
    """)


@pytest.mark.parametrize("T,n_ad,rank,dtype,waves,kb", [
    (600, 64, 64, 1, 2, 2.25), (600, 64, 120, 1, 2, 4), (600, 64, 56, 0, 2, 3.75), (600, 64, 128, 1, 2, 4.25), (600, 64, 512, 1, 2, 16.25), (600, 64, 128, 0, 2, 8.25), (600, 64, 256, 0, 2, 16.25),
    (600, 64, 320, 0, 4, 20.25), (600, 64, 512, 0, 4, 32.25), (2000, 150, 256, 1, 2, 33), (2000, 150, 320, 1, 4, 41),
    (2000, 150, 512, 1, 4, 65), (2000, 150, 128, 0, 2, 33), (2000, 150, 256, 0, 4, 65), (2000, 150, 320, 0, 8, 81), (2000, 150, 512, 0, 8, 129)])
def test_expand_waves_of_a_workgroup(fake, T, n_ad, rank, dtype, waves, kb):
    """LDS for the rows of V that a unit of the plan can have, and as few waves as keep 8 (16 with units of 16 rows) on a CU of 160 KB;
    eight 16-column blocks per wave, four with two waves and rows of B_a of 256 bytes and more."""
    fake_hip.run(fake, f"""
        T, n_ad, rank, dtype, waves, kb = {T}, {n_ad}, {rank}, {dtype}, {waves}, {kb}
        plan = make_plan(np.arange(T) % n_ad, np.ones(T, int), np.full(n_ad, rank))
        rows = plan.unit_rows
        assert rows == (16 if T == 600 else 64)
        assert kb * 1024 == rows * (rank * (2 if dtype else 4) + 16)
        B.lora_ctx_set_option(ctx, "expand_split", 1)
        F.fake_reset()
        d = make_desc(plan, 2048, 2600, dtype)
        B.lora_linear(ctx, plan, d, 0)
        units = T // rows + n_ad
        shape = [(g, b) for name, g, b in launched() if "expand_kernel" in name]
        blocks = 4 if waves == 2 and rank * (2 if dtype else 4) >= 256 else 8
        assert shape == [((units * -(-2600 // (16 * blocks * waves)), 1, 1), (64 * waves, 1, 1))], shape
        held = 16 if rows == 16 else 8
        assert waves * (160 // kb) >= held
        assert waves == 2 or waves // 2 * (160 // kb) < held
    """)


def test_expand_grid_stays_launchable(fake):
    """65536 one-row requests on as many adapters of rank 128, 65536 columns: four blocks per wave would be more than 2^32 threads."""
    fake_hip.run(fake, """
        n, N = 65536, 65536
        ids, ones, ranks = np.arange(n), np.ones(n, int), np.full(n, 128)
        plan = make_plan(ids, ones, ranks)
        d = make_desc(plan, 16, N)
        F.fake_reset()
        B.lora_linear(ctx, plan, d, 0)
        shape = [(g, b) for name, g, b in launched() if "expand_kernel" in name]
        assert shape == [(((n // 64 + n) * (N // 256), 1, 1), (128, 1, 1))], shape
    """)


def test_finishing_kernel_only_with_a_workspace_of_the_preferred_size(fake):
    """The decode path's finishing kernel rounds V to bf16; calls with less workspace keep the reduction, whose V is fp32."""
    fake_hip.run(fake, """
        plan = make_plan(np.arange(64), np.ones(64, int), np.full(64, 128))
        K, N = 520, 1544
        pref = B.lora_linear_workspace_bytes_preferred(64, K, N, 128, 1)
        least = B.lora_linear_workspace_bytes(64, K, N, 128, 1)
        assert least < pref

        def second(calls):
            F.fake_reset()
            calls()
            return ["finish" if "decode_finish" in l[0] else "reduce" for l in launched() if "decode_stream" not in l[0]]

        for size, want in ((pref, "finish"), (pref - 1, "reduce"), (least, "reduce")):
            d = make_desc(plan, K, N, ws_bytes=size)
            assert second(lambda: B.lora_linear(ctx, plan, d, 0)) == [want]
            assert second(lambda: B.lora_gemm_expand(ctx, plan, d, 0)) == [want]
        both = [make_desc(plan, K, N, ws_bytes=least), make_desc(plan, K, N, ws_bytes=pref)]
        both[1].X = both[0].X
        assert second(lambda: B.lora_linear_multi(ctx, plan, both, 0)) == ["reduce", "finish"]
    """)


@pytest.mark.parametrize("K,N", [(11008, 4096), (4096, 4096), (13824, 5120)])
@pytest.mark.parametrize("kept", [768, 1024, 2048, "static"])
def test_kept_workspace_is_used_for_what_it_has_room_for(fake, K, N, kept):
    """A workspace kept for a larger batch (or the static one): the split along K takes as many stretches as there is room for
    behind the adapter term, at most as many as with a workspace of the preferred size, and below K = 8192 those or none."""
    fake_hip.run(fake, f"""
        K, N, kept = {K}, {N}, {kept!r}
        size = (32 << 20) if kept == "static" else B.lora_linear_workspace_bytes_preferred(kept, K, N, 16, 1)
        seen = set()
        for T in (160, 256, 300, 385, 450, 512, 576, 640, 700, 768, 1000):
            plan = make_plan(np.arange(16), np.diff(np.linspace(0, T, 17).astype(int)), np.full(16, 16))
            term = T * N * 4
            before = (B.lora_linear_workspace_bytes(T, K, N, 16, 1) + 255) // 256 * 256
            F.fake_reset()
            if kept == "static":
                d = make_desc(plan, K, N, ws_bytes=0)
                B.lora_linear_static(ctx, plan, d, 0)
            elif before > size:
                continue
            else:
                B.lora_linear(ctx, plan, make_desc(plan, K, N, ws_bytes=size), 0)
            names = [l[0] for l in launched()]
            tile = [l for l in launched() if "gemm_tile_kernel" in l[0]]
            assert len(tile) == 1
            got = tile[0][1][1]
            best = B.lora_gemm_kernel_name(ctx, T, K, N, 1).rpartition("splitk")
            most = int(best[2]) if best[1] else 1
            room = max(size - before - term, 0) // term
            if K < 8192 and room < most:
                room = 0
            assert got <= max(min(most, room), 1) and (got > 1) == (most > 1 and room > 1), (T, got, most, room)
            assert any("splitk_reduce" in n for n in names) == (got > 1)
            assert any("expand_kernel" in n for n in names) == (got > 1 or size >= B.lora_linear_workspace_bytes_preferred(T, K, N, 16, 1))
            seen.add((got > 1, got < most))
        assert seen
    """)
