"""The readiness order (PP_SCHED_FIFO) of more candidates than one launch of 32 lanes each can hold:
a thousand plans over and over, each copy against the oracle's schedule of the plan."""
import numpy as np
import pytest
import torch

from paper_2204_10562_amd import workloads
from test_gpu_makespan_split import plans

pytestmark = pytest.mark.gpu


def test_readiness_order_of_a_long_list(ppo):
    from paper_2204_10562_amd import binding as pp
    from paper_2204_10562_amd.problem import GpuProblem
    S, L, D, M, n, N = 9, 16, 9, 2, 1000, (1 << 27) + 70
    w = workloads.random_small(8400, L, D, S, n, hi_time=60, hi_act=6000)
    w.actf[:], w.actb[:] = np.maximum(w.actf, 1), np.maximum(w.actb, 1)
    bounds = plans(np.random.Generator(np.random.PCG64(S)), n, S, L)
    rc, PF, PB, XF, XB = ppo.prefix_costs(w.fwd, w.bwd, w.actf, w.actb, w.bw)
    assert rc == 0
    g = GpuProblem(w)
    g.set_tables(PF, PB, XF, XB)
    rc, T0 = ppo.schedule_makespan_variant(ppo.SCHED_FIFO, L, D, S, n, M, PF, PB, XF, XB, w.orderings, bounds)
    assert rc == 0
    copies = -(-N // n)
    many = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).to(g.dev).repeat(copies, 1)[:N].reshape(-1)  # noqa: E731
    T = torch.zeros(copies * n, dtype=torch.int64, device=g.dev)
    print("[case]", S, N, flush=True)
    pp.pp_schedule_makespan_variant(pp.PP_SCHED_FIFO, L, D, S, N, M, g.PF, g.PB, g.XF, g.XB, many(w.orderings), many(bounds),
                                    T[:N], g.status)
    assert g.take_status() == 0
    T[N:] = torch.from_numpy(T0).to(g.dev)[N - (copies - 1) * n:]
    assert bool((T.reshape(copies, n) == torch.from_numpy(T0).to(g.dev)[None]).all())
