"""Schedules of more than 16 stages, whose resources are spread over several lanes: every number of
places per lane, pipelines that never fill and pipelines that do, times on both sides of the limit
of the 30-bit kernel, against the oracle (bit for bit)."""
import numpy as np
import pytest

from paper_2204_10562_amd import workloads

pytestmark = pytest.mark.gpu


def plans(rng, N, S, L):
    """N random plans: S - 1 distinct cuts each."""
    cuts = np.sort(np.argsort(rng.random((N, L - 1)), axis=1)[:, :S - 1] + 1, axis=1)
    return np.concatenate([cuts, np.full((N, 1), L)], axis=1).astype(np.int32)


def check(ppo, w, bounds, Ms):
    from paper_2204_10562_amd.problem import GpuProblem
    rc, PF, PB, XF, XB = ppo.prefix_costs(w.fwd, w.bwd, w.actf, w.actb, w.bw)
    assert rc == 0
    g = GpuProblem(w)
    g.set_tables(PF, PB, XF, XB)
    print("[case]", w.L, w.D, w.S, w.N, Ms, flush=True)
    st, T = g.makespan_multi(Ms, bounds)
    assert st == 0
    for q, M in enumerate(Ms):
        rc, T0 = ppo.schedule_makespan(w.L, w.D, w.S, w.N, M, PF, PB, XF, XB, w.orderings, bounds)
        assert rc == 0
        np.testing.assert_array_equal(T[q], T0)


@pytest.mark.parametrize("S", [17, 18, 24, 25, 29, 32, 33, 40, 41, 48, 49, 55, 56, 57, 64])
def test_makespan_many_stages(ppo, S):
    # 4S-3 + 31 is the longest fill there is
    L, D = S + 9, max(S, 66 if S % 2 else S)
    w = workloads.random_small(8000 + S, L, D, S, 150, zero_frac=0.2, hi_time=40, hi_act=6000)
    check(ppo, w, plans(np.random.Generator(np.random.PCG64(S)), 150, S, L), [1, 2, 7, 4 * S - 4, 4 * S - 3, 4 * S - 2, 4 * S + 40])


@pytest.mark.parametrize("S,N", [(17, 66000), (24, 66001), (31, 33000), (33, 33001), (44, 33003)])
def test_makespan_many_stages_many_candidates(ppo, S, N):
    # few lanes per candidate: more places per lane
    L = S + 3
    w = workloads.random_small(8100 + S, L, S, S, N, hi_time=40, hi_act=6000)
    check(ppo, w, plans(np.random.Generator(np.random.PCG64(S)), N, S, L), [3])


@pytest.mark.parametrize("S,M", [(17, 5), (32, 130), (50, 20)])
def test_makespan_many_stages_around_the_limit(ppo, S, M):
    # blocks of 64 candidates just below the limit and just above it; then all far above
    L, D, N = S + 1, S, 192
    w = workloads.random_small(8200 + S, L, D, S, N, hi_time=9, hi_act=10)
    cap = (1 << 30) // (M + 4 * S + 64)
    bounds = np.tile(np.concatenate([[1], np.arange(3, S + 2)]).astype(np.int32), (N, 1))
    bounds[64:128, 0] = 2             # layers 0 and 1 in the first stage
    w.fwd[0], w.bwd[0], w.fwd[1], w.bwd[1] = cap - 20, 0, 40, 0
    check(ppo, w, bounds, [M])
    w.fwd[0] = 8 * cap
    check(ppo, w, bounds, [M, 1])


@pytest.mark.parametrize("times", ["positive", "zeros", "wide", "mixed"])
@pytest.mark.parametrize("S,M", [(1, 3), (2, 1), (3, 40), (8, 64), (9, 5), (16, 70), (17, 9), (32, 20), (33, 6), (64, 4)])
def test_variants_over_lanes(ppo, S, M, times):
    # the comparison schedules: positive times go over lanes, zero-length items under FIFO and times
    # beyond 30 bits to the general kernel, candidate by candidate
    from paper_2204_10562_amd.problem import GpuProblem
    L, D, N = S + 7, max(S, 4), 130
    w = workloads.random_small(8300 + S, L, D, S, N, zero_frac=0.3 if times == "zeros" else 0.0, hi_time=60, hi_act=6000)
    w.actf[:] = np.maximum(w.actf, 0 if times == "zeros" else 1)
    w.actb[:] = np.maximum(w.actb, 0 if times == "zeros" else 1)
    if times == "mixed":
        w.fwd[L - 1] = w.bwd[L - 1] = 0   # some plans have a stage of nothing else
    if times == "wide":
        w.fwd[0] = 1 << 33
    bounds = plans(np.random.Generator(np.random.PCG64(S)), N, S, L)
    rc, PF, PB, XF, XB = ppo.prefix_costs(w.fwd, w.bwd, w.actf, w.actb, w.bw)
    assert rc == 0
    g = GpuProblem(w)
    g.set_tables(PF, PB, XF, XB)
    for v in range(5):
        print("[case]", v, S, M, times, flush=True)
        st, T = g.makespan_variant(v, M, bounds)
        rc, T0 = ppo.schedule_makespan_variant(v, L, D, S, N, M, PF, PB, XF, XB, w.orderings, bounds)
        assert st == 0 and rc == 0
        np.testing.assert_array_equal(T, T0)
