"""The closed form of the schedules, run lane by lane on the CPU from the kernel's own source: several microbatch
counts, plans of every stage count, sums that leave 32 bits, and the minimum over the plans."""
import os
import subprocess

import pytest

from test_wave_makespan import ADDITIVE, DUPLEX, GPIPE, PE, build, pytestmark  # noqa: F401


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    return build(tmp_path_factory.mktemp("path"), "path_driver")


def ask(exe, lines):
    env = dict(os.environ)
    env.pop("LD_PRELOAD", None)  # the sanitizer's runtime must come first in the library list
    res = subprocess.run([exe], input="".join(l + "\n" for l in lines), stdout=subprocess.PIPE,
                         stderr=subprocess.PIPE, text=True, timeout=300, env=env)
    assert res.returncode == 0, res.stderr[-2000:]
    assert "runtime error" not in res.stderr, res.stderr[-2000:]
    out = [[int(x) for x in l.split()] for l in res.stdout.splitlines()]
    assert len(out) == len(lines)
    return out


# pipelines that fill and that do not, on both sides of M = 2R and M = K + 1; times with many zeros and
# equal values, of 20 bits (32-bit sums), and up to 2^50 (64-bit sums)
@pytest.mark.parametrize("variant,counts", [(PE, "1 2 3 4 5 6 7 8"), (PE, "9 14 29 30 31 64 200"), (PE, "1 40"), (DUPLEX, "1"),
                                            (DUPLEX, "13"), (DUPLEX, "200"), (GPIPE, "7"), (ADDITIVE, "1"), (ADDITIVE, "11"), (ADDITIVE, "99")])
def test_against_the_schedule(exe, variant, counts):
    nM = len(counts.split())
    lines = ["%d %d %d %d 0 %d 0 %d %s" % (variant, S, N, S + hi % 97, hi, nM, counts)
             for S, N in ((1, 3), (2, 64), (3, 65), (4, 130), (5, 70), (8, 260), (15, 20), (33, 9), (64, 2)) for hi in (1, 4, 10**6, 2**50)]
    for line, got in zip(lines, ask(exe, lines)):
        assert got == [0, 0, 0, 0], line


# times next to the largest that 32-bit sums and 24-bit products take (2^30 over M + 4 S + 64, twice M and 4 S more in
# GPipe's order), where the largest forward and the largest backward time lie on different resources
@pytest.mark.parametrize("variant,counts", [(PE, "1"), (PE, "3 40"), (PE, "2 5 9 70"), (DUPLEX, "2"), (DUPLEX, "31"), (GPIPE, "1"), (GPIPE, "2"),
                                            (GPIPE, "3"), (GPIPE, "5"), (GPIPE, "8"), (GPIPE, "12"), (GPIPE, "33"), (ADDITIVE, "2"),
                                            (ADDITIVE, "25")])
def test_times_next_to_the_limit(exe, variant, counts):
    Ms = [int(m) for m in counts.split()]
    lines = []
    for S, N in ((1, 2), (2, 20), (3, 40), (4, 64), (6, 65), (9, 20), (20, 10)):
        n = max(Ms) * (2 if variant == GPIPE else 1) + 4 * S * (2 if variant == GPIPE else 1) + 64
        limit = (2**30 - 1) // n
        lines += ["%d %d %d %d -1 %d 0 %d %s" % (variant, S, N, seed, hi, len(Ms), counts)
                  for seed in range(1, 6) for hi in (limit // 2, limit - 1, limit, limit + 1)]
    for line, got in zip(lines, ask(exe, lines)):
        assert got == [0, 0, 0, 0], line


@pytest.mark.parametrize("S,N", [(1, 70), (2, 5), (7, 66), (8, 64), (9, 20), (17, 3)])
def test_every_stage_count(exe, S, N):
    lines = ["%d %d %d %d 0 %d 1 3 2 17 70" % (PE, S, N, S, hi) for hi in (1, 10**5, 2**45)]
    for line, got in zip(lines, ask(exe, lines)):
        assert got == [0, 0, 0, 0], line


@pytest.fixture(scope="module")
def replicated(tmp_path_factory):
    return build(tmp_path_factory.mktemp("rep"), "rep_driver")


# (the smallest and largest numbers of GPUs of every instance of the kernel, fewer layers than GPUs, pipelines that fill
# and that do not; quotients of a few units, of 30 bits and beyond)
@pytest.mark.parametrize("D,L,N", [(2, 3, 70), (4, 9, 20), (5, 4, 30), (8, 20, 66), (9, 11, 9), (12, 30, 5), (13, 40, 4), (16, 50, 3)])
def test_replicated_stages(replicated, D, L, N):
    lines = ["%d %d %d %d %d %d" % (D, L, M, N, D + M, hi) for M in (1, 2, 7, 25, 80) for hi in (1, 30, 10**5, 2**44)]
    for line, got in zip(lines, ask(replicated, lines)):
        assert got == [0, 0, 0, 0], line
