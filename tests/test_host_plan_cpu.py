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
