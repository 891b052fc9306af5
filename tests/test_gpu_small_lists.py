"""Lists so short that one workgroup schedules them and picks the winners itself: numbers of candidates around one, two
and three waves with one to five microbatch counts, plans that the schedule builds itself (equal activation sizes)
and plans from the dynamic program, lists with rows that are no orderings."""
import numpy as np
import pytest

from paper_2204_10562_amd import workloads
from test_gpu_parity import G, check_best_multi, oracle_tables, say  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [1, 2, 63, 64, 65, 127, 128, 129, 191, 192, 193])
@pytest.mark.parametrize("same_act", [False, True])
def test_short_lists(ppo, G, N, same_act):
    for S in (1, 2, 3, 8):
        w = workloads.random_small(900 + N + S, 24, 8, S, N, hi_time=60, hi_act=500, same_act=same_act)
        g, tables = G(w), oracle_tables(ppo, w)
        g.set_tables(*tables)
        for Ms in ([7], [20, 3], [1, 30, 5], [4, 9, 2, 9], [4, 9, 2, 9, 31]):
            say("short list", N, S, "same_act" if same_act else "", Ms)
            check_best_multi(ppo, g, w, Ms, tables)


@pytest.mark.parametrize("D", [2, 4, 5])
def test_all_orderings(ppo, G, D):
    w = workloads.random_small(950 + D, 17, D, D, 1, hi_time=60, hi_act=500)
    w.orderings, w.N = None, [1, 1, 2, 6, 24, 120][D]
    g, tables = G(w), oracle_tables(ppo, w)
    g.set_tables(*tables)
    for Ms in ([5], [8, 4], [3, 2, 1, 9]):
        say("all orderings", D, Ms)
        check_best_multi(ppo, g, w, Ms, tables)


@pytest.mark.parametrize("same_act", [False, True])
def test_rows_that_are_no_orderings(ppo, G, same_act):
    """They have no plan, the winner comes from the others; with none left there is no winner."""
    w = workloads.random_small(960, 24, 6, 5, 70, hi_time=60, hi_act=500, same_act=same_act)
    tables = oracle_tables(ppo, w)
    for all_bad in (False, True):
        rows = slice(0, 70) if all_bad else slice(3, 66, 7)
        bad = np.zeros(70, bool)
        bad[rows] = True
        w.orderings[rows, 1] = w.orderings[rows, 0]
        say("no orderings", "all" if all_bad else "some", "same_act" if same_act else "")
        g = G(w)
        g.set_tables(*tables)
        st, res, T, C = g.best_multi([6, 11])
        assert st != 0
        good = np.flatnonzero(~bad)
        for q, M in enumerate((6, 11)):
            assert (T[q][bad] == np.iinfo(np.int64).max).all()
            if all_bad:
                assert res[q]["best_index"] == -1
                continue
            rc, res0, T0, C0 = ppo.best_plan(w.L, w.D, w.S, len(good), M, *tables, np.ascontiguousarray(w.orderings[good]))
            assert rc == 0
            np.testing.assert_array_equal(T[q][good], T0)
            np.testing.assert_array_equal(C[good], C0)
            assert res[q] == dict(res0, best_index=int(good[res0["best_index"]]))
