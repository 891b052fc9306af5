"""Candidates with the channel-free plan are scheduled where they are found: lists in which all, some or none of the
candidates have it, in launches of their own (L <= 128, also where the makespan kernel could build plans itself) and in front
of the sort (L > 128), with every number of counts a lane works on and one more, with and without the T of all, against the
oracle (bit for bit)."""
import numpy as np
import pytest

from test_gpu_dp_band import problem

pytestmark = pytest.mark.gpu

SIZES = [
    (60, 8, 8, 60001), (97, 11, 3, 200003), (97, 12, 11, 30011), (100, 9, 7, 150000), (128, 16, 16, 20000), (77, 33, 31, 9001),
    (129, 6, 5, 64), (150, 9, 9, 65), (257, 12, 11, 3000), (200, 20, 18, 4500), (300, 64, 64, 300), (140, 4, 2, 777)]
# (the kernel of the rows looks for them itself, or candidates share their program)
ELSEWHERE = [(97, 11, 3, 200003), (97, 12, 11, 30011), (128, 16, 16, 20000), (129, 6, 5, 64), (140, 4, 2, 777)]


@pytest.mark.parametrize("L,D,S,N", SIZES)
@pytest.mark.parametrize("kind", ["free", "zeros", "some", "most"])
def test_free_plans(ppo, kind, L, D, S, N):
    from paper_2204_10562_amd import binding as pp
    from paper_2204_10562_amd.problem import GpuProblem
    w = problem(kind, 9700 + L + S + N, L, D, S, N)
    rc, PF, PB, XF, XB = ppo.prefix_costs(w.fwd, w.bwd, w.actf, w.actb, w.bw)
    assert rc == 0
    rc, C0, b0 = ppo.partition_dp(L, D, S, N, PF, PB, XF, XB, w.orderings)
    assert rc == 0
    Ms = [2, 19, 5, 40, 11]
    T0 = []
    for M in Ms:
        rc, T = ppo.schedule_makespan(L, D, S, N, M, PF, PB, XF, XB, w.orderings, b0)
        assert rc == 0
        T0.append(T)
    rows = [1, N // 2, N - 1]
    for bad in (False, True):
        if bad:
            w.orderings[rows[0], 0] = D
            w.orderings[rows[1], S - 1] = w.orderings[rows[1], 0]
            w.orderings[rows[2], S // 2] = -1
        g = GpuProblem(w)
        g.set_tables(PF, PB, XF, XB)
        keep = np.ones(N, bool)
        if bad:
            keep[rows] = False
        for nM in (1, 2, 4, 5):
            for want in (True, False):
                print("[case] free plans", kind, L, D, S, N, bad, nM, want, flush=True)
                st, res, T, C = g.best_multi(Ms[:nM], want_all=want)
                assert st == (ppo.FAULT_ORDERING if bad else 0)
                looked = int(g.ws[pp.PP_WS_SHARE + 40:pp.PP_WS_SHARE + 44].cpu().numpy().view(np.int32)[0])
                assert looked == (nM < 5 and (L, D, S, N) not in ELSEWHERE) or kind != "free"
                for q in range(nM):
                    t = np.where(keep, T0[q], np.iinfo(np.int64).max)
                    c = int(np.argmin(t))
                    assert (res[q]["best_index"], res[q]["T"], res[q]["C"]) == (c, t[c], C0[c])
                    assert res[q]["bounds"] == b0[c].tolist() and res[q]["order"] == w.orderings[c].tolist()
                    if want:
                        np.testing.assert_array_equal(T[q], t)
                if want:
                    np.testing.assert_array_equal(C[keep], C0[keep])


@pytest.mark.parametrize("L,D,S,N,looks", [(150, 9, 3, 400, False), (300, 32, 3, 400, False), (300, 33, 3, 400, True), (200, 10, 4, 400, False),
                                           (200, 11, 4, 400, True), (129, 64, 2, 64, False), (128, 11, 9, 150000, True)])
def test_no_launch_for_nothing(L, D, S, N, looks):
    """The look for channel-free plans to schedule (up to four counts) is not launched where candidates share their
    program whatever the links are: D * D kinds of links make at most 2^20 sequences."""
    import ctypes

    import torch
    from paper_2204_10562_amd import binding as pp
    from paper_2204_10562_amd.problem import GpuProblem
    g = GpuProblem(problem("free", L + D, L, D, S, N))
    assert g.prefix() == 0
    out = torch.zeros(5 * pp.RESULT_BYTES, dtype=torch.uint8, device=g.dev)
    ws = g.workspace()
    hip = ctypes.CDLL("libamdhip64.so")
    launches = []
    for nM in (4, 5):
        print("[case] launches", L, D, S, N, nM, flush=True)
        graph = torch.cuda.CUDAGraph(keep_graph=True)
        with torch.cuda.graph(graph):
            pp.pp_best_plan_multi(L, D, S, N, [2, 19, 5, 40, 11][:nM], g.PF, g.PB, g.XF, g.XB, g.orderings, out, None, None, ws, g.status)
        n = ctypes.c_size_t(0)
        assert hip.hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(n)) == 0
        launches.append(n.value)
    assert launches[0] - launches[1] == looks, launches
