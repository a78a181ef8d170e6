"""f_color where the class masks of a member take several pieces, and where the counts go pair by pair instead, and the
time of the counts with many classes."""
import numpy as np
import pytest

import oracle
from tcolgen import FP4, KCOL, KPART, GraphCase

from gpu_util import host, torch_mod
from test_gpu_call_times import solver, us_of

pytestmark = pytest.mark.gpu


# masks: one piece, two, several; compares: one strip, strips of every remainder, classes past the vertices, the last
# words of the rows
@pytest.mark.parametrize("problem", [KCOL, KPART])
@pytest.mark.parametrize("n,k,D", [(1, 1, 1), (64, 40, 3), (500, 320, 3), (700, 320, 40), (1025, 130, 37), (1025, 500, 80),
                                   (65, 1300, 2), (257, 700, 5), (513, 400, 3), (1000, 500, 4), (1023, 1300, 8),
                                   (1300, 4096, 1), (2000, 900, 2)])
def test_counts_of_many_classes(n, k, D, problem):
    import paper_1909_02261_amd as pk
    torch = torch_mod()
    if problem == KPART and k > n:
        pytest.skip("more parts than vertices")
    case = GraphCase("counts", problem, n, k, D, FP4, "gnp", 0.5, graph_seed=n + k)
    A, W = case.adjacency(), case.weights()
    c = oracle.colors(W)
    ref = oracle.fcolor(A, c)
    if problem == KPART:
        ref = int(A.astype(np.int64).sum()) // 2 - ref
    a, w = torch.from_numpy(A).cuda(), torch.from_numpy(W).cuda()
    p = pk.Params(n=n, k=k, D=D, problem=problem, precision=FP4, stop_on_legal=0)
    s = pk.Solver([(a, w)], [p])
    got = s.conflicts(0)
    loss = host(s.loss_grad(0, want_gs=False, want_gw=False)[0])
    s.close()
    assert np.array_equal(host(got[0]), c) and np.array_equal(host(got[1]), ref)
    assert loss[1] == ref.sum()
    got = pk.conflicts_noalloc(a, w, p)
    torch.cuda.synchronize()
    assert np.array_equal(host(got[0]), c) and np.array_equal(host(got[1]), ref)


def test_counts_of_two_graphs():
    """Graphs of one context on either side of the rule: the blocks of each start where the last one's end."""
    import paper_1909_02261_amd as pk
    torch = torch_mod()
    cases = [GraphCase("counts", KCOL, n, k, D, FP4, "gnp", 0.5, graph_seed=g)
             for g, (n, k, D) in enumerate([(300, 700, 3), (700, 20, 5), (640, 900, 2), (200, 10, 9)])]
    arrays = [(c.adjacency(), c.weights()) for c in cases]
    s = pk.Solver([(torch.from_numpy(A).cuda(), torch.from_numpy(W).cuda()) for A, W in arrays],
                  [pk.Params(n=c.n, k=c.k, D=c.D, precision=FP4, stop_on_legal=0) for c in cases])
    got = [host(s.conflicts(g)[1]) for g in range(len(cases))]
    s.close()
    for (A, W), f in zip(arrays, got):
        assert np.array_equal(f, oracle.fcolor(A, oracle.colors(W)))


@pytest.mark.parametrize("n,D", [(2000, 4), (4000, 4)])
def test_time_of_many_classes(n, D):
    """900 classes against 60 (as 32 and 63 pieces of masks the counts took 3.1 and 4.5 times as long)."""
    ss = [solver(n, k, D, FP4) for k in (60, 900)]
    us = us_of(lambda: ss[0].conflicts(0), lambda: ss[1].conflicts(0), reps=40)
    for s in ss:
        s.close()
    print(us)
    assert us[1] < 2.2 * us[0], us
