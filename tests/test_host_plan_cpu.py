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
        def read(i):  # what the kernel does: the launch's word receives its ticket
            a = F.fake_arg1(i)
            C.c_uint32.from_address(C.c_uint64.from_address(a + 8).value).value = C.c_uint32.from_address(a + 16).value
        for i in range(100):
            make_plan([0, 1], [1, 2], [8, 16])
            if i != 3:
                read(i)
        seen = [a for a, _ in tables()]
        assert len(seen) == 100 and seen.count(seen[3]) == 1
        assert len({t for _, t in tables()}) == 100
    """)
