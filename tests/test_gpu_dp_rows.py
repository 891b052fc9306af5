"""The row-by-row partition DP (a search per cell) at the edges of its chunks of 64 cells and on
transfer times that make its crossings fall on peaks, against the oracle (bit for bit)."""
import numpy as np
import pytest

from paper_2204_10562_amd import workloads

pytestmark = pytest.mark.gpu


def shaped(kind, seed, L, D, S, N):
    w = workloads.random_small(seed, L, D, S, N, hi_time=300, hi_act=3000)
    rng = np.random.Generator(np.random.PCG64(seed))
    if kind == "rising":        # links never bind
        w.actf[:] = rng.integers(1, 40, size=L)
    elif kind == "peaks":       # every few cuts one that costs more than a stage
        w.actf[::5] = 40000
        w.actb[::7] = 90000
    elif kind == "falling":     # each cut cheaper than the one before, links always bind
        w.actf[:] = np.arange(L, 0, -1) * 400
        w.actb[:] = np.arange(L, 0, -1) * 300
    elif kind == "zero":        # runs of zero-length layers: equal prefix sums
        w.fwd[rng.random(L) < 0.6] = 0
        w.bwd[w.fwd == 0] = 0
        w.actf[::4] = 50000
    elif kind == "skewed":      # most layers in a small share of the time: windows far above L / stages
        w.fwd[: 3 * L // 4] = 1
        w.bwd[: 3 * L // 4] = 0
    return w


@pytest.mark.parametrize("kind", ["rising", "peaks", "falling", "zero", "skewed"])
@pytest.mark.parametrize("L,D,S,N", [(88, 6, 6, 40), (89, 6, 3, 40), (96, 5, 2, 40), (97, 70, 34, 70), (127, 9, 9, 40), (128, 64, 64, 34), (128, 4, 1, 9),
                                     (129, 5, 2, 20), (191, 7, 7, 30), (192, 6, 3, 30), (193, 9, 8, 30), (256, 4, 4, 24),
                                     (257, 12, 12, 20), (320, 65, 6, 20), (449, 20, 17, 12), (512, 8, 5, 20),
                                     (1025, 40, 33, 6), (2048, 64, 64, 3)])
def test_partition_rows(ppo, kind, L, D, S, N):
    from paper_2204_10562_amd.problem import GpuProblem
    w = shaped(kind, 7000 + L + S, L, D, S, N)
    rc, PF, PB, XF, XB = ppo.prefix_costs(w.fwd, w.bwd, w.actf, w.actb, w.bw)
    assert rc == 0
    g = GpuProblem(w)
    g.set_tables(PF, PB, XF, XB)
    print("[case]", kind, L, D, S, N, flush=True)
    st, C, b = g.dp()
    rc, C0, b0 = ppo.partition_dp(L, D, S, w.N, PF, PB, XF, XB, w.orderings)
    assert st == 0 and rc == 0
    np.testing.assert_array_equal(C, C0)
    np.testing.assert_array_equal(b, b0)
