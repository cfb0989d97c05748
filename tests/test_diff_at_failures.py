"""psfs_diff_forward_at when the runtime fails half-way (host code against
tests/hip_double.c): no copy into the plan's host buffer is under way after
its return, and the plan is as before."""
import pytest

from tests.host_driver import check


@pytest.mark.parametrize("fail,ok", [("record", False), (1, False), (0, True)])
def test_no_copy_outlives_the_call(tmp_path_factory, fail, ok):
    got = check(tmp_path_factory, "diff_forward_at", dict(fail=fail))
    assert (got["rc"] == 0) == ok and got["ready"] == ok and got["matrices"] == ok
    assert got["pending"] == 0


@pytest.mark.parametrize("launch", [2, 3])               # the fusion and the loss, after the maps
def test_the_plan_is_unchanged_by_a_late_failure(tmp_path_factory, launch):
    got = check(tmp_path_factory, "diff_forward_at", dict(fail=launch))
    assert got["rc"] == -5 and not got["ready"] and not got["matrices"] and got["pending"] == 0
