"""The partition from a few cells of every row: lists on each side of where it is tried (length, devices, layers),
links that never reach into a value, do so in a few rows and bind nearly everywhere, layers of length zero and bad
orderings, for S stages and for every number of stages, against the oracle (bit for bit)."""
import numpy as np
import pytest

from paper_2204_10562_amd import workloads

pytestmark = pytest.mark.gpu

SIZES = [
    # tested inside the register-tiled and the row kernel; in launches of its own; around a wave of candidates
    (88, 8, 8, 2600), (90, 9, 7, 9000), (128, 8, 8, 6000), (48, 24, 24, 10000), (90, 40, 12, 12001), (128, 64, 33, 900),
    (129, 6, 5, 63), (129, 6, 5, 64), (150, 9, 9, 65), (257, 12, 11, 3000), (200, 20, 20, 4500), (300, 64, 64, 300)]


def problem(kind, seed, L, D, S, N):
    w = workloads.random_small(seed, L, D, S, N, zero_frac=0.2 if kind == "zeros" else 0.0, hi_time=300)
    stage = int((w.fwd + w.bwd).sum()) // S
    # times at 100 bytes per microsecond against a stage's: hidden, now and then longer, mostly longer
    most = {"free": 0.4, "zeros": 0.8, "some": 1.3, "most": 3.0}[kind]
    rng = np.random.Generator(np.random.PCG64(seed))
    w.actf = rng.integers(0, int(most * stage * 50) + 1, size=L)
    w.actb = rng.integers(0, int(most * stage * 50) + 1, size=L)
    w.bw = rng.integers(100, 130, size=(D, D)).astype(np.int64)
    np.fill_diagonal(w.bw, 0)
    return w


@pytest.mark.parametrize("L,D,S,N", SIZES)
@pytest.mark.parametrize("kind", ["free", "zeros", "some", "most"])
def test_partition_from_few_cells(ppo, kind, L, D, S, N):
    from paper_2204_10562_amd.problem import GpuProblem
    w = problem(kind, 9100 + L + S + N, L, D, S, N)
    rc, PF, PB, XF, XB = ppo.prefix_costs(w.fwd, w.bwd, w.actf, w.actb, w.bw)
    assert rc == 0
    g = GpuProblem(w)
    g.set_tables(PF, PB, XF, XB)
    print("[case]", kind, L, D, S, N, flush=True)
    st, C, b = g.dp()
    rc, C0, b0 = ppo.partition_dp(L, D, S, N, PF, PB, XF, XB, w.orderings)
    assert st == 0 and rc == 0
    np.testing.assert_array_equal(C, C0)
    np.testing.assert_array_equal(b, b0)
    st, Cs, bs = g.dp_stages()
    assert st == 0
    Cs, bs = np.asarray(Cs).reshape(N, S), np.asarray(bs).reshape(N, -1)
    for x in {2, S // 2, S}:
        if x < 1:
            continue
        rc, C0, b0 = ppo.partition_dp(L, D, x, N, PF, PB, XF, XB, np.ascontiguousarray(w.orderings[:, :x]))
        assert rc == 0
        np.testing.assert_array_equal(Cs[:, x - 1], C0)
        np.testing.assert_array_equal(bs[:, x * (x - 1) // 2:x * (x + 1) // 2], b0)
    # bad rows are reported and leave the others alone
    rows = [1, 62, N - 1]
    w.orderings[rows[0], 0] = D
    w.orderings[rows[1], S - 1] = w.orderings[rows[1], 0]
    w.orderings[rows[2], S // 2] = -1
    g = GpuProblem(w)
    g.set_tables(PF, PB, XF, XB)
    st, C1, b1 = g.dp()
    assert st == ppo.FAULT_ORDERING
    keep = np.ones(N, bool)
    keep[rows] = False
    np.testing.assert_array_equal(C1[keep], C[keep])
    np.testing.assert_array_equal(b1[keep], b[keep])


def test_all_orderings_inside_and_outside_a_launch_of_their_own(ppo):
    from paper_2204_10562_amd.problem import GpuProblem
    for L in (97, 150):
        w = problem("some", 9300 + L, L, 8, 8, 1)
        w.orderings, w.N = None, 40320
        rc, PF, PB, XF, XB = ppo.prefix_costs(w.fwd, w.bwd, w.actf, w.actb, w.bw)
        assert rc == 0
        g = GpuProblem(w)
        g.set_tables(PF, PB, XF, XB)
        print("[case] all 8! orderings", L, flush=True)
        st, C, b = g.dp()
        rc, C0, b0 = ppo.partition_dp(L, 8, 8, w.N, PF, PB, XF, XB, workloads.all_orderings(8))
        assert st == 0 and rc == 0
        np.testing.assert_array_equal(C, C0)
        np.testing.assert_array_equal(b, b0)


def test_work_counters(ppo):
    """Links that reach into no value: no pair is evaluated; links that bind nearly everywhere: most rows are whole."""
    from paper_2204_10562_amd import binding as pp
    from paper_2204_10562_amd.problem import GpuProblem
    for kind in ("free", "most"):
        w = problem(kind, 9500, 128, 8, 8, 1)
        w.orderings, w.N = None, 40320
        g = GpuProblem(w)
        g.prefix()
        print("[case] work counters", kind, flush=True)
        assert g.dp()[0] == 0
        s = pp.read_workspace_stats(g.ws)
        assert s["rows_executed"] > 0 and s["band_pairs"] <= s["pairs_executed"]
        if kind == "free":
            assert s["pairs_executed"] == 0 and s["free_rows"] == s["rows_executed"]
        else:
            assert s["pairs_executed"] > s["rows_executed"] > 2 * (s["free_rows"] + s["band_rows"])


@pytest.mark.parametrize("L,D,S,N,looks", [(150, 9, 8, 300, 1), (300, 16, 16, 2000, 1), (400, 64, 64, 64, 1), (1024, 9, 8, 64, 1),
                                           (88, 8, 8, 2600, 0), (128, 8, 8, 900, 0), (60, 40, 33, 3000, 0), (97, 12, 11, 7000, 1),
                                           (40, 8, 8, 60000, 1), (128, 16, 16, 9000, 1)])
def test_short_lists_whose_links_bind(ppo, L, D, S, N, looks):
    """Nothing is tried that cannot be worth it there: the recursion over bands nowhere, and the plan of the program without
    transfer times only where a list is long enough for it and links seldom bind."""
    from paper_2204_10562_amd import binding as pp
    from paper_2204_10562_amd.problem import GpuProblem
    for kind in ("free", "most"):
        w = problem(kind, 9600 + L + S + N, L, D, S, N)
        g = GpuProblem(w)
        g.prefix()
        for stages in (False, True):
            print("[case] short list", kind, L, D, S, N, stages, flush=True)
            assert (g.dp_stages() if stages else g.dp())[0] == 0
            s = pp.read_workspace_stats(g.ws)
            assert s["band_pairs"] == s["band_rows"] == 0
            if kind == "most":
                assert s["free_rows"] == 0
            elif not stages:
                assert (s["free_rows"] > 0) == bool(looks)
