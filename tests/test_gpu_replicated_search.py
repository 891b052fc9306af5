"""pp_plan_replicated at the edges of its int32 form: the scan and the search for a cell's split
(chunks of 64 positions, runs of equal quotients, fewer layers than stages) and the quotients by double
arithmetic (exact multiples, sizes next to 2^53, where the int64 form takes over).  The values are
whole numbers, so all of them must be the oracle's."""
import numpy as np
import pytest

from paper_2204_10562_amd import workloads
from test_gpu_parity import sub_workload
from test_gpu_replicated import G, check, say  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("seed,L,D,N", [
    (601, 2, 8, 6), (602, 8, 8, 12), (603, 63, 3, 6), (604, 64, 5, 8), (605, 65, 8, 8), (606, 127, 4, 8), (610, 39, 6, 8),
    (611, 40, 6, 8), (607, 128, 6, 8), (608, 129, 3, 6), (609, 193, 4, 4),
    (612, 962, 2, 2), (613, 1021, 2, 2),
])
def test_search_edges(ppo, G, seed, L, D, N):
    rng = np.random.Generator(np.random.PCG64(seed))
    # times: few distinct values (runs of equal quotients), long runs of zeros, one huge layer
    for kind in ("narrow", "zeros", "peak", "sizes only"):
        w = workloads.random_small(seed, L, D, D, N, zero_frac=0.6 if kind == "zeros" else 0.1,
                                   hi_time=4 if kind == "narrow" else 1000, hi_act=900)
        if kind == "peak":
            w.fwd[L // 2] = 100000
        if kind == "sizes only":
            w.fwd[:] = 0
            w.bwd[:] = 0
        alpha = rng.integers(0, 4000 if kind == "peak" else 30, size=L).astype(np.int64)
        say("search", seed, L, D, kind)
        check(ppo, G, w, alpha, 5)


@pytest.mark.parametrize("act", [(1 << 53) - 1, 1 << 53, (1 << 53) + 1])
def test_quotients_next_to_the_exact_range(ppo, G, act):
    w = workloads.random_small(620, 20, 4, 4, 12, hi_time=50, hi_act=900)
    rng = np.random.Generator(np.random.PCG64(620))
    w.bw[:] = rng.integers((1 << 26) + 1, 1 << 27, size=w.bw.shape)
    np.fill_diagonal(w.bw, 0)
    w.actf[:] = act - rng.integers(0, 3, size=w.actf.shape)
    w.actf[0] = act
    w.actb[:] = rng.integers(1, 8, size=w.actb.shape) * w.bw[0, 1] * 12  # multiples of r r' b
    for total in ((1 << 53) // 8 - 1, (1 << 53) // 8, 0):
        alpha = np.full(20, total // 20, np.int64)
        alpha[0] += total - int(alpha.sum())
        say("quotients", act, total)
        check(ppo, G, w, alpha, 2)
