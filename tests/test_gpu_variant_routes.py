"""The comparison schedules on both sides of where the kernels that spread a plan over lanes take over from
the general one (number of stages, updates per plan), against the oracle (bit for bit)."""
import numpy as np
import pytest

from paper_2204_10562_amd import workloads
from test_gpu_makespan_split import plans

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S,M", [(1, 1), (1, 24), (1, 25), (1, 300), (2, 4), (2, 5), (3, 2), (3, 3), (6, 1), (7, 1)])
def test_variants_around_the_rule(ppo, S, M):
    from paper_2204_10562_amd.problem import GpuProblem
    L, D, N = S + 9, max(S, 4), 150
    for zero in (0.0, 0.3):
        w = workloads.random_small(8800 + S + M, L, D, S, N, zero_frac=zero, hi_time=60, hi_act=6000)
        if not zero:
            w.actf[:], w.actb[:] = np.maximum(w.actf, 1), np.maximum(w.actb, 1)
        bounds = plans(np.random.Generator(np.random.PCG64(S)), N, S, L)
        rc, PF, PB, XF, XB = ppo.prefix_costs(w.fwd, w.bwd, w.actf, w.actb, w.bw)
        assert rc == 0
        g = GpuProblem(w)
        g.set_tables(PF, PB, XF, XB)
        for v in range(5):
            print("[case]", v, S, M, zero, flush=True)
            st, T = g.makespan_variant(v, M, bounds)
            rc, T0 = ppo.schedule_makespan_variant(v, L, D, S, N, M, PF, PB, XF, XB, w.orderings, bounds)
            assert st == 0 and rc == 0
            np.testing.assert_array_equal(T, T0)
