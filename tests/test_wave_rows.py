"""The partition DP's kernels that search for a cell's split, run lane by lane on the CPU (their own sources,
with UndefinedBehaviorSanitizer) against the recursion over all splits: values, the lowest split among
equal ones, every number of stages.  The LDS is filled with different bytes beforehand: neither results nor
any vote of a wave may depend on what an earlier launch left there."""
import os
import subprocess

import pytest

from test_wave_makespan import build

pytestmark = pytest.mark.skipif(__import__("shutil").which("g++") is None, reason="needs g++")

KINDS = {"free": 0, "one zero layer": 1, "half zero layers": 2, "last layer outweighs": 3, "skewed": 4,
         "falling transfers": 5, "random transfers": 6, "all zero": 7,
         "few slow cuts": 8, "few slow cuts, half zero layers": 9}


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    exe = build(tmp_path_factory.mktemp("rows"), "rows_driver")

    def ask(cases, *args):
        env = dict(os.environ)
        env.pop("LD_PRELOAD", None)  # the sanitizer's runtime must come first in the library list
        res = subprocess.run([exe, *args], input="".join(" ".join(str(x) for x in c) + "\n" for c in cases),
                             stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True, timeout=300, env=env)
        assert res.returncode == 0 and "runtime error" not in res.stderr, res.stderr[-2000:]
        out = [[int(x) for x in l.split()] for l in res.stdout.splitlines()]
        assert len(out) == len(cases)
        return out
    return ask


@pytest.mark.parametrize("kind", KINDS)
def test_rows_lane_by_lane(driver, kind):
    sizes = [(89, 4, 2, 6), (89, 3, 3, 6), (90, 7, 1, 5), (97, 12, 11, 9), (100, 5, 5, 14), (111, 17, 16, 6),
             (127, 8, 8, 12), (128, 8, 8, 12), (128, 33, 32, 4), (113, 40, 33, 4), (128, 64, 64, 3),
             (129, 5, 5, 6), (192, 6, 5, 6), (200, 9, 8, 5), (256, 4, 4, 6), (321, 7, 7, 4)]
    cases = [(L, D, S, N, L + S, KINDS[kind], stages, fill) for L, D, S, N in sizes for stages in (0, 1) for fill in (0, 255, 85)]
    out = driver(cases)
    for case, got in zip(cases, out):
        assert got[:3] == [0, 0, 0], case
    # the same way there whatever the LDS held
    for i in range(0, len(out), 3):
        assert out[i] == out[i + 1] == out[i + 2], cases[i]


@pytest.mark.parametrize("L,D,S,N", [(97, 12, 11, 30), (128, 8, 8, 40), (128, 17, 16, 20), (300, 9, 8, 12), (192, 17, 16, 12)])
def test_steps_do_not_depend_on_binding_links(driver, L, D, S, N):
    # all trips of the searches are counted, those of repeated rounds too: links that bind at every cut
    # may widen the windows (and longer rows take shorter steps then), but never make a cell look at its
    # splits one by one
    free, falling, wild = (driver([(L, D, S, N, 5, k, 0, 0)])[0][3] for k in (0, 5, 6))
    most = 1.7 if L <= 128 else 3.5
    assert falling < most * free and wild < most * free, (free, falling, wild)


@pytest.mark.parametrize("L,D,S,N", [(89, 4, 2, 900), (97, 6, 5, 603), (128, 5, 3, 450), (90, 3, 3, 192), (128, 34, 33, 200)])
def test_candidates_that_are_finished_already(driver, L, D, S, N):
    """Chunks of several pieces, of which some candidates, all or none are left: those are right, and the kernel keeps its
    hands off the others also behind a piece where most are left."""
    cases = [(L, D, S, N, L + S, kind, stages, 85) for kind in (0, 6) for stages in (0, 1)]
    for case, got in zip(cases, driver(cases, "left")):
        assert got[:3] == [0, 0, 0], case


@pytest.mark.parametrize("L,D,S,N", [(89, 4, 2, 900), (89, 4, 3, 900), (97, 6, 5, 600), (128, 5, 3, 450), (150, 5, 3, 300)])
def test_bad_orderings_wherever_they_stand(driver, L, D, S, N):
    """Also behind as many finished candidates as a wave keeps before it writes their plans out."""
    cases = [(L, D, S, N, seed, kind, stages, 85) for seed in (2, 3) for kind in (0, 6) for stages in (0, 1)]
    for case, (rc, status, differ, _, _) in zip(cases, driver(cases, "bad")):
        assert rc == 0 and status != 0 and differ == 0, case
