"""Plans of one stage: a device that does not exist is reported wherever in a wave's share of the list
it stands."""
import numpy as np
import pytest

from paper_2204_10562_amd import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L", [1, 20, 88, 89, 128, 129])
@pytest.mark.parametrize("N", [70, 20003, 150001])
def test_bad_device_of_a_single_stage(L, N):
    from paper_2204_10562_amd import binding as pp
    from paper_2204_10562_amd.problem import GpuProblem
    w = workloads.random_small(8500 + L, L, 3, 1, N)
    bad = np.arange(3, N, 7)
    w.orderings[bad, 0] = np.where(bad % 2, 3, -1)
    g = GpuProblem(w)
    assert g.prefix() == 0
    print("[case]", L, N, flush=True)
    st, C, b = g.dp()
    want = np.full(N, int((w.fwd + w.bwd).sum()))
    want[bad] = np.iinfo(np.int64).max
    assert st == pp.PP_FAULT_ORDERING
    np.testing.assert_array_equal(C, want)
