"""Calls whose time must not depend on the colouring, or grow with a batch or with few colours, beside another route of
the same build to the same numbers.  Each bound stands far from both sides: a route that loses its split loses several
times, and the routes compared share the box and the moment."""
import time

import numpy as np
import pytest

from paper_1909_02261_amd import FP4, FP32, KCOL, KPART, MCOL

from gpu_util import host, torch_mod

pytestmark = pytest.mark.gpu


def us_of(*calls, reps=10, rounds=9):
    """Microseconds of each call, in turn over `rounds`, the least of its runs of `reps`."""
    torch = torch_mod()
    best = [float("inf")] * len(calls)
    for f in calls:
        f(), f()
    for _ in range(rounds):
        for x, f in enumerate(calls):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            for _ in range(reps):
                f()
            torch.cuda.synchronize()
            best[x] = min(best[x], (time.perf_counter() - t0) / reps * 1e6)
    return best


def solver(n, k, D, prec, cols=None, G=1, problem=KCOL, A=None, **kw):
    """A solver whose colours stay as they are (a step moves the weights by about 1e-9)."""
    import paper_1909_02261_amd as pk
    torch = torch_mod()
    rng = np.random.default_rng(n + k)
    graphs, params = [], []
    for g in range(G):
        if A is None:
            a = np.triu(rng.random((n, n), dtype=np.float32) < 0.5, 1)
            a = (a | a.T).astype(np.uint8)
        else:
            a = A
        c = rng.integers(0, k, (D, n)) if cols is None else cols
        W = rng.normal(0.0, 0.01, (D, n, k)).astype(np.float32)
        np.put_along_axis(W, c[:, :, None], 1.0, axis=2)
        graphs.append((torch.from_numpy(a).cuda(), torch.from_numpy(W).cuda()))
        params.append(pk.Params(n=n, k=k, D=D, problem=problem, precision=prec, eta=1e-9, rho=1.0,
                                max_demand=1 if problem == MCOL else 0, **{"stop_on_legal": 0, **kw}))
    s = pk.Solver(graphs, params)
    for g in range(G):
        s.set_t(100, g)
    return s


def one_conflict(n, k, part):
    """A graph and a colouring with one conflicting (partitioning: cut) edge, between the vertices that a scan reaches
    last."""
    rng = np.random.default_rng(n)
    base = np.sort(np.arange(n) % k)
    a = np.triu(rng.random((n, n), dtype=np.float32) < 0.5, 1)
    same = base[:, None] == base[None, :]
    a &= same if part else ~same
    i, j = (n - 1, 0) if part else (n - 1, n - 2)
    a[min(i, j), max(i, j)] = True
    return (a | a.T).astype(np.uint8), base


@pytest.mark.parametrize("problem,n,k,D,prec", [(KCOL, 2700, 2, 8, FP4), (KCOL, 5000, 3, 8, FP4), (KPART, 2000, 4, 8, FP4),
                                                (KCOL, 1000, 3, 32, FP32)])
def test_stop_rule_of_nearly_legal_members(problem, n, k, D, prec):
    """Eight iterations with the stop rule on members one conflict away from legal against the same without it."""
    A, base = one_conflict(n, k, problem == KPART)
    ss = [solver(n, k, D, prec, cols=np.tile(base, (D, 1)), A=A, problem=problem, stop_on_legal=stop) for stop in (0, 1)]
    if problem == KPART:
        for s in ss:
            s.set_options(penalty=1)
    assert all(s.conflicts(0)[1].tolist() == [1] * D for s in ss)
    us = us_of(lambda: ss[0].step(8), lambda: ss[1].step(8))
    for s in ss:
        assert s.conflicts(0)[1].tolist() == [1] * D
        s.close()
    # (a scan of the pairs of the classes, one byte at a time, took 2.4 to 37 times)
    print(us)
    assert us[1] < 1.35 * us[0] + 40, us


@pytest.mark.parametrize("n,k,D", [(10000, 3, 10), (4000, 20, 64)])
def test_conflicts_of_few_colours(n, k, D):
    """The conflict counts from the adjacency bits against the contraction's gather (a multicolouring context's) where the
    contraction has few columns (pair by pair they took 3.2 and 2.1 times its time)."""
    ss = [solver(n, k, D, FP4, problem=problem) for problem in (KCOL, MCOL)]
    us = us_of(lambda: ss[0].conflicts(0), lambda: ss[1].conflicts(0), reps=40)
    assert np.array_equal(*(host(s.conflicts(0)[1]) for s in ss))
    for s in ss:
        s.close()
    print(us)
    assert us[0] < 1.1 * us[1], us


def test_conflicts_of_one_graph_of_a_batch():
    """conflicts() on a context of 128 small graphs: the graphs' fitness side by side.  Against the loss without gradients,
    which has the same launches and a block per graph (one block for all of them took 2.7 us a graph)."""
    s = solver(100, 10, 8, FP4, G=128)
    a, b = us_of(lambda: s.conflicts(3), lambda: s.loss_grad(3, want_gs=False, want_gw=False))
    f = host(s.conflicts(3)[1]).sum()
    assert f == host(s.loss_grad(3)[0])[1]
    s.close()
    print(a, b)
    assert a < 1.5 * b, (a, b)


@pytest.mark.parametrize("n,k,D,one", [(2000, 40, 8, True), (4000, 2, 20, False), (1000, 1, 8, True), (8000, 3, 8, False),
                                       (300, 500, 4, False), (500, 50, 64, True)])
def test_class_rows_of_few_or_large_classes(n, k, D, one):
    """fp32 iterations where a class holds every vertex, where there are few classes, and where there are more than
    vertices, against the plain schedule, whose contraction does not depend on the classes (a wave summing a whole class
    by itself took up to 2.4 times)."""
    cols = np.full((D, n), k // 2) if one else None
    ss = [solver(n, k, D, FP32, cols=cols) for _ in range(2)]
    for fused, s in enumerate(ss):
        s.set_options(fused=fused, penalty=1)
    us = us_of(lambda: ss[0].step(8), lambda: ss[1].step(8))
    for s in ss:
        s.close()
    print(us)
    assert us[1] < us[0], us
