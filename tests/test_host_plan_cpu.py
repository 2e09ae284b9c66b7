"""lora_plan()'s pinned tables on a stand-in HIP runtime: no table is handed out twice while a kernel may still read it."""
import pytest

import fake_hip


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    return fake_hip.build(tmp_path_factory.mktemp("fake_hip"))


def test_pending_error_of_another_call_is_not_the_launch_s(fake):
    """An error that an earlier HIP call left in the thread says nothing about the plan's launch: the plan is made, and the
    next one gets a table and a ticket of its own."""
    fake_hip.run(fake, """
        for i in range(6):
            say("pending", 101)  # an invalid device ordinal, for instance
            assert make_plan([0, 1, -1][: 1 + i % 3], [3, 0, 5][: 1 + i % 3], [8, 16], raw=True) == B.LORA_OK, i
        seen = tables()
        assert len(seen) == 6
        assert len({a for a, _ in seen}) == 6, seen
    """)


def test_failed_launch_is_reported_and_later_plans_work(fake):
    fake_hip.run(fake, """
        for i in range(40):
            say("launch_error", 2)
            assert make_plan([0], [1], [8], raw=True) == B.LORA_ERR_HIP
            say("launch_error", 0)
            if i % 8 == 0:
                assert make_plan([0, 1], [1, 4], [8, 16], raw=True) == B.LORA_OK
        seen = tables()
        assert len(seen) == 5 and len({a for a, _ in seen}) == 5, seen
    """)


def test_plan_kernels_that_never_run(fake):
    """More plans than there are tables, none of them read: every call returns within a bounded time -- through the upload,
    whose errors are reported -- and so does the end of the context."""
    fake_hip.run(fake, """
        import time
        for i in range(40):
            t = time.perf_counter()
            assert make_plan([0, 1, -1], [3, 0, 5], [8, 16], raw=True) == B.LORA_OK, i
            assert time.perf_counter() - t < 2.0
        seen = tables()
        assert len({a for a, _ in seen}) == len(seen) < 40
        assert F.fake_launches() == 40  # the others: one launch each of the device's own builder
        say("sync_error", 719)  # a device that is gone
        assert make_plan([0], [1], [8], raw=True) == B.LORA_ERR_HIP
        t = time.perf_counter()
        B.lora_ctx_destroy(ctx)
        assert time.perf_counter() - t < 2.0
    """, timeout=30)


def test_tables_are_taken_again_when_they_have_been_read(fake):
    """Every table but one is read: the plans go on through the tables and leave that one alone."""
    fake_hip.run(fake, """
        for i in range(100):
            make_plan([0, 1], [1, 2], [8, 16])
            if i != 3:
                read_table(i)
        seen = [a for a, _ in tables()]
        assert len(seen) == 100 and seen.count(seen[3]) == 1
        assert len({t for _, t in tables()}) == 100
    """)


def test_no_exception_leaves_lora_plan(fake):
    """Memory for a thousand counters is refused: a status comes back, or the plan is made without; nothing is thrown."""
    fake_hip.run(fake, """
        say("largest_new", 2048)
        status = make_plan([0, 1], [1, 2], [8] * 1000, raw=True)
        say("largest_new", 1 << 30)
        assert status in (B.LORA_OK, B.LORA_ERR_INVALID_ARG), status
        assert make_plan([0, 1], [1, 2], [8] * 1000, raw=True) == B.LORA_OK
    """)


def test_host_table_against_the_reference(fake):
    """Every request- and segment-level entry of the pinned table, for slots at the edges of the host's bit words, unused slots
    between, requests without rows and without adapter, batches one after another in the same scratch."""
    fake_hip.run(fake, """
        from oracle import plan_reference
        rng = np.random.default_rng(11)
        for n_ad in (1, 63, 64, 65, 200, 65536):
            for R in (0, 1, 5, 300):
                edge = [v for v in (0, 62, 63, 64, 127, 128, 65535) if v < n_ad]
                ids = np.where(rng.random(R) < 0.5, rng.choice(edge, R), rng.integers(-1, n_ad, R)).astype(np.int32)
                L = rng.integers(0, 4, R).astype(np.int32)
                ranks = rng.choice([8, 16, 64], n_ad).astype(np.int32)
                F.fake_reset()
                plan = make_plan(ids, L, ranks, r_max=64)
                ref = plan_reference(ids, L, ranks)
                S = len(ref["seg_adapter"])
                read_table(0)
                tab = np.ctypeslib.as_array((C.c_int32 * (3 * R + 5 * S + 4)).from_address(tables()[0][0]))
                at = 3 * R + 1
                tok = np.concatenate([[0], np.cumsum(L)])
                assert np.array_equal(tab[: R + 1], tok)
                slot_of = np.empty(int(L.sum()), int)
                slot_of[ref["perm"]] = np.arange(len(slot_of))
                full = np.flatnonzero(L)
                assert np.array_equal(tab[R + 1 : 2 * R + 1][full], slot_of[tok[full]])
                assert np.array_equal(tab[2 * R + 1 : at][full], ref["row_seg"][slot_of[tok[full]]])
                for name, n in (("seg_adapter", S), ("seg_indptr", S + 1), ("seg_rank", S), ("seg_ext", S + 1)):
                    assert np.array_equal(tab[at : at + n], ref[name]), (n_ad, R, name)
                    at += n
                rows = np.diff(ref["seg_indptr"])
                units = np.where(ref["seg_adapter"] >= 0, -(-rows // plan.unit_rows), 0)
                assert np.array_equal(tab[at : at + S + 1], np.concatenate([[0], np.cumsum(units)]))
    """)


def test_stream_whose_capture_status_is_not_told(fake):
    """The runtime refuses to say (the legacy stream while another thread captures): the calls go on as under capture and leave no
    error behind."""
    fake_hip.run(fake, """
        say("status_error", 906)
        plan = make_plan([0, 1, 1], [1, 2, 3], np.full(9, 8))
        B.lora_linear(ctx, plan, make_desc(plan, 512, 512), 0)
        assert "plan_tiny" in launched()[0][0] and F.fake_launches() == 3
        assert F.hipGetLastError() == 0
    """)


def test_options_and_capture_reach_the_device_s_builders(fake):
    """lora_plan() with "plan_variant" or "plan_fused_rows" set, or under stream capture, uploads the arrays and launches the builders
    that lora_plan_device() launches; otherwise the table's kernel."""
    fake_hip.run(fake, """
        def kernels(R, option=None, value=-1, capturing=0):
            F.fake_reset()
            if option:
                B.lora_ctx_set_option(ctx, option, value)
            say("capturing", capturing)
            make_plan(np.arange(R) % 7, np.ones(R, int), np.full(7, 8))
            if option:
                B.lora_ctx_set_option(ctx, option, -1)
            return [next(k for k in ("apply", "tiny", "mid", "small", "segments", "fill") if f"plan_{k}_kernel" in l[0]) for l in launched()]

        for R, by_size in ((5, "tiny"), (64, "tiny"), (100, "mid"), (300, "small")):
            assert kernels(R) == ["apply"]
            assert kernels(R, "plan_variant", 0) == [by_size] == kernels(R, capturing=1)
            assert kernels(R, "plan_variant", 1) == ["small"]
            assert "apply" not in kernels(R, "plan_fused_rows", 0) and kernels(R, "plan_fused_rows", 0)[-1] == "fill"
            assert kernels(R) == ["apply"]
    """)
