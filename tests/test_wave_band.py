"""The partition from a few cells of every row, run lane by lane on the CPU (its own sources, with
UndefinedBehaviorSanitizer) against the recursion over all splits: every candidate it finishes has the true
values and the lowest split among equal ones, with and without the links' words, for every number of stages."""
import os
import subprocess

import pytest

from test_wave_makespan import build

pytestmark = pytest.mark.skipif(__import__("shutil").which("g++") is None, reason="needs g++")

FREE, ZEROS, TIES, OUTLIER, EQUAL, SOME, MOST, HIGH = range(8)
SIZES = [(3, 2, 2, 64), (5, 5, 5, 70), (17, 8, 8, 65), (64, 9, 2, 64), (40, 33, 33, 66), (88, 12, 11, 64), (128, 8, 8, 130),
         (200, 7, 7, 64), (321, 20, 16, 64), (130, 64, 64, 64)]


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    exe = build(tmp_path_factory.mktemp("band"), "band_driver")

    def ask(cases, *args):
        env = dict(os.environ)
        env.pop("LD_PRELOAD", None)  # the sanitizer's runtime must come first in the library list
        res = subprocess.run([exe, *args], input="".join(" ".join(str(x) for x in c) + "\n" for c in cases),
                             stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True, timeout=600, env=env)
        assert res.returncode == 0 and "runtime error" not in res.stderr, res.stderr[-2000:]
        out = [[int(x) for x in l.split()] for l in res.stdout.splitlines()]
        assert len(out) == len(cases)
        return out
    return ask


@pytest.mark.parametrize("kind", [FREE, ZEROS, TIES, OUTLIER, EQUAL, SOME, MOST, HIGH])
def test_bands_lane_by_lane(driver, kind):
    cases = [(L, D, S, N, L + S, kind, stages, words) for L, D, S, N in SIZES for stages in (0, 1) for words in (0, 1)
             if not (stages and S > 33)]
    ended = 0
    for case, (rc, status, differ, done, reported) in zip(cases, driver(cases)):
        N = case[3]
        assert rc == 0 and differ == 0, case
        if kind == FREE:
            # links that never bind: every candidate ends; the bad ordering is reported
            assert (done, reported) == (N - 1, 1) and status != 0, case
        else:
            assert status == 0, case
        ended += done
    # links that bind in some rows or all leave candidates to the other kernels, but not all of them
    assert ended > 0
    if kind in (SOME, MOST):
        assert ended < sum(c[3] for c in cases)


@pytest.mark.parametrize("kind", [FREE, SOME, MOST, HIGH])
def test_work_counters(driver, kind):
    """What did not run is not counted: no pair and no computed row for candidates with the channel-free plan or a bad
    ordering, pairs of bands only where there was a recursion (also one that ended nothing)."""
    cases = [(L, D, S, N, L + S, kind, stages, words) for L, D, S, N in SIZES[1:8] for stages in (0, 1) for words in (0, 1)
             if not (stages and S > 12)]
    for case, (_, _, _, done, _, pairs, rows, band_pairs, band_rows, free_rows) in zip(cases, driver(cases, "work")):
        L, D, S, N, _, _, stages, words = case
        assert pairs == band_pairs and rows == band_rows + free_rows, case
        per = S * (S - 1) // 2 if stages else S - 1
        assert free_rows <= done * (S - 1) and band_rows % per == 0 and band_rows <= done * per, case
        if not words:
            assert free_rows == 0 and band_rows == done * per and pairs >= band_rows, case
        elif kind == FREE:
            # every link is hidden: nothing is evaluated
            assert pairs == 0 and free_rows >= N - 1, case
        if pairs == 0:
            assert band_rows == 0, case


@pytest.mark.parametrize("kind", [FREE, ZEROS, TIES, OUTLIER, SOME, MOST])
def test_scheduled_where_they_are_found(driver, kind):
    """One to four counts; a group of 64 in part and several; rows of two to 64 devices, multiples of four and not; and in the first
    kind a bad ordering."""
    cases = [(L, D, S, N, seed, kind, 0, 1) for L, D, S, N in SIZES + [(30, 3, 3, 191), (60, 5, 5, 257), (64, 8, 4, 129), (97, 6, 6, 300)]
             for seed in (L + S, L + S + 1, L + S + 3)]
    found = 0
    for case, (rc, _, differ, done, reported, scheduled, times, minima, both) in zip(cases, driver(cases, "free")):
        S, N = case[2:4]
        assert (rc, differ, times, minima, both) == (0, 0, 0, 0, 0), case
        if kind == FREE:
            # (a link may reach into the values of a row without binding in the plan: with as many stages as 64, now and then)
            assert (done, reported) == (N - 1, 1) and (scheduled == N - 1 if S < 64 else 2 * scheduled > N), case
        found += scheduled
        assert scheduled <= done
    assert found > 0


@pytest.mark.parametrize("kind", [FREE, ZEROS, SOME, HIGH])
def test_short_lists(driver, kind):
    """A list too short for the recursion is looked at for the channel-free plan alone, and not at all where links bind so
    often that hardly a candidate has it."""
    cases = [(L, D, S, N, L + S, kind, stages, words) for L, D, S, N in SIZES[1:8] for stages in (0, 1) for words in (0, 1)
             if not (stages and S > 12)]
    ended = 0
    for case, (rc, _, differ, done, reported, pairs, rows, _, _, free_rows) in zip(cases, driver(cases, "short")):
        L, D, S, N, _, _, _, words = case
        assert rc == 0 and differ == 0 and pairs == 0 and rows == free_rows, case
        assert (rows > 0) == (done > 0) and (words or not done), case
        if kind == FREE and words:
            assert (done, reported) == (N - 1, 1), case
        if kind == HIGH and L > 4 * S > 8:
            assert done == reported == 0, case
        ended += done
    assert ended > 0 or kind in (SOME, HIGH)


def test_places_of_the_channel_free_plans(driver):
    cases = [(L, D, S, N) for L in (2, 16, 88, 128, 129, 131, 400, 1025) for D in (2, 3, 8, 33, 47, 63, 64)
             for S in sorted({2, min(3, D, L), min(D, L, 64)}) for N in list(range(64, 200)) + [252, 253, 999, 4095, 4097, 200003, 1 << 20]
             if S <= min(L, D)]
    for (L, D, S, N), (room, clash) in zip(cases, driver(cases, "layout")):
        # (a list of 64 or more; L <= 128: what the bands' own launches are made for has a thousand candidates)
        assert not clash and (room or (L <= 128 and N < 253)), (L, D, S, N)
