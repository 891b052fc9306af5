"""The replicated planner from the bands, run lane by lane on the CPU (its own sources, with UndefinedBehaviorSanitizer)
against the oracle: times from a few microseconds to the limit of 32-bit values, links that bind, layers of length zero,
both ways to share the states among waves."""
import os
import subprocess

import numpy as np
import pytest

from paper_2204_10562_amd import workloads
from test_wave_makespan import build

pytestmark = pytest.mark.skipif(__import__("shutil").which("g++") is None, reason="needs g++")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    exe = build(tmp_path_factory.mktemp("prm"), "prm_driver")

    def ask(problems):
        env = dict(os.environ)
        env.pop("LD_PRELOAD", None)  # the sanitizer's runtime must come first in the library list
        text = "".join(" ".join(str(int(x)) for x in p) + "\n" for p in problems)
        res = subprocess.run([exe], input=text, stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True, timeout=600, env=env)
        assert res.returncode == 0 and "runtime error" not in res.stderr, res.stderr[-2000:]
        out = [np.array([int(x) for x in l.split()], np.int64) for l in res.stdout.splitlines()]
        assert len(out) == len(problems)
        return out
    return ask


def problem(seed, L, D, N, M, times, kind):
    w = workloads.random_small(seed, L, D, D, N, zero_frac=0.05, hi_time=times, hi_act=90 * times)
    rng = np.random.Generator(np.random.PCG64(seed))
    if kind == "far":  # links that bind
        w.bw[:] = np.maximum(w.bw // 8, 1)
    if kind == "one slow":
        w.bw[0, D - 1] = w.bw[D - 1, 0] = 1
    alpha = rng.integers(0, 3 * times, size=L).astype(np.int64)
    return w, alpha, M


def numbers(w, alpha, M, team):
    return np.concatenate([[w.L, w.D, w.N, M, team], w.fwd, w.bwd, w.actf, w.actb, alpha, w.bw.ravel(), w.orderings.ravel()])


def split(out, N, D):
    tri = D * (D + 1) // 2
    W, b, r = out[5:5 + N * D], out[5 + N * D:5 + N * (D + tri)], out[5 + N * (D + tri):]
    return W.reshape(N, D), b.reshape(N, tri), r.reshape(N, tri)


# (the largest times: sums next to 2^29 / M, where the bound's arithmetic in 32-bit floats is coarsest)
SIZES = [(9, 3, 9, 3, 40), (17, 8, 9, 64, 40), (30, 4, 5, 16, 300), (34, 5, 9, 30, 5000), (60, 6, 3, 60, 900), (26, 9, 5, 24, 60),
         (40, 3, 17, 40, 120000), (90, 5, 2, 64, 40000), (70, 4, 3, 20, 160000), (33, 13, 3, 40, 200)]


@pytest.mark.parametrize("kind", ["near", "far", "one slow"])
def test_plans_from_the_bands(ppo, driver, kind):
    problems = [problem(900 + i, L, D, N, M, times, kind) for i, (L, D, N, M, times) in enumerate(SIZES)]
    used = 0
    for team in (1, 0):
        for (w, alpha, M), out in zip(problems, driver([numbers(*p, team) for p in problems])):
            status, parts, lanes, widest, tried = out[:5]
            assert status == 0 and (tried or not parts) and widest <= parts * lanes
            if not parts:
                continue
            used += 1
            rc, _, _, W0, b0, r0 = ppo.spp_replicated(w.L, w.D, w.N, M, w.fwd, w.bwd, w.actf, w.actb, alpha, w.bw, w.orderings)
            assert rc == 0
            W, b, r = split(out, w.N, w.D)
            np.testing.assert_array_equal(W, W0)
            np.testing.assert_array_equal(b, b0)
            np.testing.assert_array_equal(r, r0)
    assert used >= 10 if kind == "near" else used > 0


def test_slow_links_end_the_look_for_bands(driver):
    """A link so slow that a plan of one GPU a stage cannot have enough cuts within any of the times that would do."""
    for seed, L, D, M in ((960, 60, 4, 16), (961, 40, 5, 32), (962, 75, 12, 24)):
        w, alpha, M = problem(seed, L, D, 2, M, 300, "near")
        w.actf = w.actb = np.full(L, 20000, np.int64)
        w.bw[:] = 2000
        for slow in (False, True):
            if slow:
                w.bw[0, 1] = 1
            out, = driver([numbers(w, alpha, M, 1)])
            assert out[4] != slow and (not slow or out[1] == 0), (seed, slow)


def test_room_for_bands(driver):
    """Up to which number of layers there are bands, workgroups of four waves, and three workgroups (of 16 lanes a candidate)
    to a compute unit: what the tables of a workgroup and the states of its waves take of the LDS decides it."""
    rooms = {6: (667, 433, 433, 516), 8: (545, 353, 353, 420), 12: (396, 255, 255, 305),
             14: (197, 0, 194, 197), 16: (175, 0, 171, 175)}
    for (D, room), out in zip(rooms.items(), driver([[0, D, 0, 0, 0] for D in rooms])):
        assert tuple(out) == room, D
