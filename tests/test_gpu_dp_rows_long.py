"""Lists on both sides of where the row kernel takes over from the register-tiled one (88 < L <= 128: list
length, stages, layers), links that never and always bind and layers of length zero, against the oracle
(bit for bit)."""
import numpy as np
import pytest

from paper_2204_10562_amd import workloads
from test_gpu_dp_rows import shaped

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,D,S,N", [
    (89, 4, 2, 6144), (89, 5, 3, 6143), (89, 5, 3, 6144), (97, 12, 11, 6200), (104, 13, 12, 6144), (104, 17, 16, 6200),
    (105, 6, 6, 4095), (105, 6, 6, 4096), (112, 14, 13, 4100), (120, 13, 13, 2048), (128, 8, 8, 4096), (128, 9, 9, 20011),
    (128, 20, 18, 2100), (128, 40, 40, 2050), (89, 70, 24, 2100), (128, 70, 64, 2048)])
@pytest.mark.parametrize("kind", ["rising", "falling", "zero"])
def test_partition_rows_of_long_lists(ppo, kind, L, D, S, N):
    from paper_2204_10562_amd.problem import GpuProblem
    w = shaped(kind, 8600 + L + S, L, D, S, N)
    # half of the candidates share their first devices with the one before
    rng = np.random.Generator(np.random.PCG64(N))
    for c in np.flatnonzero(rng.random(N - 1) < 0.5) + 1:
        k = int(rng.integers(0, S))
        head = w.orderings[c - 1, :k]
        w.orderings[c] = np.concatenate([head, rng.permutation(np.setdiff1d(np.arange(D), head))[:S - k]])
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
    np.testing.assert_array_equal(Cs[:, S - 1], C0)
    np.testing.assert_array_equal(bs[:, S * (S - 1) // 2:], b0)
    x = S // 2
    if x > 1:
        rc, C0, b0 = ppo.partition_dp(L, D, x, N, PF, PB, XF, XB, np.ascontiguousarray(w.orderings[:, :x]))
        assert rc == 0
        np.testing.assert_array_equal(Cs[:, x - 1], C0)
        np.testing.assert_array_equal(bs[:, x * (x - 1) // 2:x * (x + 1) // 2], b0)


@pytest.mark.parametrize("L", [128, 191, 192, 193, 256, 1024])
def test_last_layer_that_outweighs_the_others(ppo, L):
    # cell L rests on its last split: nothing stands right of it in the row
    from paper_2204_10562_amd.problem import GpuProblem
    w = workloads.random_small(8700 + L, L, 6, 5, 40, hi_time=300, hi_act=3000)
    w.fwd[L - 1] = 2 * int((w.fwd + w.bwd).sum())
    rc, PF, PB, XF, XB = ppo.prefix_costs(w.fwd, w.bwd, w.actf, w.actb, w.bw)
    assert rc == 0
    g = GpuProblem(w)
    g.set_tables(PF, PB, XF, XB)
    print("[case]", L, flush=True)
    st, C, b = g.dp()
    rc, C0, b0 = ppo.partition_dp(L, 6, 5, 40, PF, PB, XF, XB, w.orderings)
    assert st == 0 and rc == 0
    np.testing.assert_array_equal(C, C0)
    np.testing.assert_array_equal(b, b0)
