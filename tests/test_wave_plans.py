"""The schedules of the planner's own plans, run lane by lane on the CPU from the kernel's own source: bad orderings, bounds that are none
(which read nothing that is not there), candidates that have been scheduled already, and the winners."""
import pytest

from test_wave_makespan import build, pytestmark  # noqa: F401
from test_wave_path import ask

FAULT_ORDERING, FAULT_BOUNDS = 4, 8


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    return build(tmp_path_factory.mktemp("plans"), "plans_driver")


# one workgroup that picks and several, times of 32-bit and of 64-bit sums
@pytest.mark.parametrize("counts", ["7", "2 31", "1 9 40 70"])
@pytest.mark.parametrize("search,free", [(0, 0), (1, 0), (0, 1)])
def test_planners_plans(exe, counts, search, free):
    lines = ["%d %d %d %d %d %d %d %s" % (S, N, S + N, hi, search, free, len(counts.split()), counts)
             for S, N in ((1, 40), (2, 64), (3, 130), (5, 700), (8, 65), (11, 260), (33, 40)) for hi in (2, 10**4, 2**45)
             if S * N < 3000 or not search]
    torn = 0
    for line, got in zip(lines, ask(exe, lines)):
        assert got[0] == 0 and got[2:4] == [0, 0], line
        assert bool(got[1] & FAULT_BOUNDS) == (got[4] > 0) and not got[1] & ~(FAULT_BOUNDS | FAULT_ORDERING), line
        torn += got[4]
    assert torn > 0
