"""pp_plan_replicated from the bands: 8, 16 and 32 cells per state at their edges (all cells of few layers, one layer
more), both ways to share the states among waves, lists that do not fill a wave, orderings that are none."""
import numpy as np
import pytest

from paper_2204_10562_amd import workloads
from test_gpu_parity import sub_workload
from test_gpu_replicated import G, check, say  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("seed,L,D,N,M,times", [
    (701, 9, 3, 5, 3, 40), (702, 10, 8, 9, 40, 40), (703, 17, 8, 8, 3, 40), (704, 18, 9, 4, 30, 40),
    (705, 33, 5, 3, 4, 400), (706, 34, 5, 3, 4, 400), (707, 40, 16, 3, 60, 90), (708, 96, 8, 7, 64, 20),
    (709, 96, 8, 1, 5, 200), (710, 70, 12, 2, 24, 900), (711, 120, 4, 17, 64, 500), (712, 64, 6, 9, 12, 90),
    (713, 12, 12, 6, 9, 30), (717, 90, 3, 5, 3, 50), (718, 90, 3, 5, 2, 50),
])
def test_bands(ppo, G, seed, L, D, N, M, times):
    rng = np.random.Generator(np.random.PCG64(seed))
    w = workloads.random_small(seed, L, D, D, N, zero_frac=0.05, hi_time=times, hi_act=900)
    for kind in ("near", "far"):
        if kind == "far":  # links that bind, AllReduces that do not fit
            w.bw[:] = np.maximum(w.bw // 8, 1)
        alpha = rng.integers(0, 30 if kind == "near" else 3000, size=L).astype(np.int64)
        say("bands", seed, L, D, M, kind)
        check(ppo, G, w, alpha, M)


@pytest.mark.parametrize("seed,L,D,N,M,times", [
    (730, 40, 5, 12301, 32, 90), (731, 20, 4, 6149, 3, 5000), (732, 24, 9, 6149, 16, 60), (733, 31, 5, 3077, 4, 400),
    (734, 40, 6, 1003, 32, 90)])
def test_long_lists(ppo, G, seed, L, D, N, M, times):
    """Nine orderings, each many times over, and some rows that are none: those have no plan, the others are not
    disturbed."""
    rng = np.random.Generator(np.random.PCG64(seed))
    few = workloads.random_small(seed, L, D, D, 9, hi_time=times, hi_act=900)
    alpha = rng.integers(0, 100, size=L).astype(np.int64)
    rc, _, T0, W0, b0, r0 = ppo.spp_replicated(L, D, 9, M, few.fwd, few.bwd, few.actf, few.actb, alpha, few.bw, few.orderings)
    assert rc == 0
    at = rng.integers(0, 9, size=N)
    w = sub_workload(few, at)
    none = rng.choice(N, 7, replace=False)
    for wrong in (False, True):
        say("bands, long lists", seed, L, D, N, "wrong rows" if wrong else "")
        if wrong:
            w.orderings[none[:4], 1] = w.orderings[none[:4], 0]
            w.orderings[none[4:], D - 1] = D + 3
        st, _, T, W, b, r = G(w).plan_replicated(M, alpha)
        assert (st != 0) == wrong
        good = np.ones(N, bool)
        if wrong:
            good[none] = False
            assert (W[none] == np.iinfo(np.int64).max).all()
        for got, want in ((W, W0), (b, b0), (r, r0), (T, T0)):
            np.testing.assert_array_equal(got[good], want[at][good])
