"""The merged schedule of the fast path (one launch for everything that depends on the colours, with the
stop rule's answer; class-row sums instead of the fp32 contraction) against the plain schedule,
which launches each step of Algorithm 1 by itself.

The class-row sums add the same FP32 terms in the order of the fp32 contraction's accumulation, so
weights are compared bit for bit.  Stop decisions, group concentration and graph checks are integers.
"""
import numpy as np
import pytest

import tcolgen
from tcolgen import BF16, BKPART, ECP, FP4, FP32, KCOL, KPART, MSCP, GraphCase

from gpu_util import host, make_solver, torch_mod

pytestmark = pytest.mark.gpu


def weights_of(cols, k, seed=0):
    """Weights whose argmax is the colouring cols ([D, n])."""
    rng = np.random.default_rng(seed)
    W = rng.normal(0.0, 0.01, size=cols.shape + (k,)).astype(np.float32)
    np.put_along_axis(W, cols[:, :, None], 1.0, axis=2)
    return W


@pytest.mark.parametrize("problem", [KCOL, BKPART, MSCP])
@pytest.mark.parametrize("n,k,D", [(1, 1, 1), (16, 2, 1), (63, 5, 3), (64, 64, 2), (65, 33, 4), (129, 17, 5), (300, 90, 9),
                                   (515, 7, 3), (700, 200, 2), (200, 380, 2)])
def test_class_rows_bits_equal_the_fp32_contraction(problem, n, k, D):
    """6 iterations from t = 300 (all terms active), random weights; the class sizes pass through collapsed
    phases after the smoothing at t = 304."""
    case = GraphCase(f"cr_n{n}_k{k}_D{D}", problem, n, k, D, FP32, "gnp", 0.5, graph_seed=n, rho=10.0, lam=1e-3, mu=1e-4,
                     nu=1e-3 if problem != KCOL else 0.0, stop_on_legal=0, momentum=0.5 if D == 3 else 0.0)
    out = []
    for fused in (0, 1):
        s, _ = make_solver([case], fused=fused, penalty=1)
        assert s.options()["fused"] == fused
        s.set_t(300)
        done, _ = s.step(6)
        assert done == 6
        out.append(host(s.W[0]))
        s.close()
    assert np.array_equal(out[0], out[1])


@pytest.mark.parametrize("one", [False, True], ids=["spread", "one_class"])
def test_class_rows_loss_and_gradients_of_any_class_sizes(one):
    """gS and the loss through the class-row sums, every vertex in one class among empty ones or spread over all,
    against the plain schedule's contraction by way of one unsmoothed step: W - W' = eta gW."""
    n, k, D = 197, 40, 3
    cols = np.full((D, n), 17) if one else np.random.default_rng(1).integers(0, k, (D, n))
    W = weights_of(cols, k)
    case = GraphCase("cr_grad", KCOL, n, k, D, FP32, "gnp", 0.4, graph_seed=3, lam=1e-3, mu=1e-4, stop_on_legal=0)
    s, _ = make_solver([case], Ws=[W])
    s.set_t(50)
    _, _, gw = s.loss_grad(0)
    c, f, _ = s.conflicts(0)
    s.step(1)
    step = (W.astype(np.float64) - host(s.W[0])) / float(np.float32(1e-3))
    # the difference of two FP32 weights of magnitude up to 1: 2^-24 each, over eta
    assert np.abs(step - host(gw)).max() <= 2.0 ** -23 / 1e-3 + 1e-6 * np.abs(host(gw)).max()
    A = case.adjacency().astype(np.int64)
    ref = [int((A * (cols[d][:, None] == cols[d][None, :])).sum()) // 2 for d in range(D)]
    assert np.array_equal(host(c), cols) and host(f).tolist() == ref
    s.close()


def legal_setup(problem, n, k, D, legal):
    """A graph and D colourings of which members `legal` have fitness 0; the others have one bad pair."""
    rng = np.random.default_rng(n + k)
    base = rng.permutation(np.arange(n) % k)             # equitable classes
    u = np.triu(rng.random((n, n)) < 0.5, 1)
    same = base[:, None] == base[None, :]
    part = problem in (KPART, BKPART)
    A = u & (same if part else ~same)
    # one edge that colourings other than `base` get wrong
    i = 0
    j = int(np.flatnonzero(same[0])[1]) if part else int(np.flatnonzero(~same[0])[0])
    A[min(i, j), max(i, j)] = True
    A = (A | A.T).astype(np.uint8)
    cols = np.tile(base, (D, 1))
    for d in range(D):
        if d not in legal:
            # swap the colours of j and of another vertex (sizes stay equitable)
            if part:
                x = int(np.flatnonzero(base != base[j])[0])
                cols[d, j], cols[d, x] = base[x], base[j]
            else:
                x = next(v for v in range(n) if base[v] == base[i] and v != i)
                cols[d, j], cols[d, x] = base[x], base[j]
    return A, cols


@pytest.mark.parametrize("prec", [FP32, FP4])
@pytest.mark.parametrize("problem", [KCOL, ECP, KPART, BKPART])
@pytest.mark.parametrize("n,k", [(65, 6), (254, 31)])
def test_merged_stop_rule(problem, n, k, prec):
    """The first launch's legality check: the lowest legal member stops the graph before its update, and
    members one bad pair away do not."""
    for legal in ((), (2,), (1, 3)):
        A, cols = legal_setup(problem, n, k, 4, legal)
        W = weights_of(cols, k)
        case = GraphCase("stop", problem, n, k, 4, prec, "gnp", 0.5, stop_on_legal=1, lam=1e-3, mu=1e-4, nu=1e-3)
        torch = torch_mod()
        res = []
        for fused in (0, 1):
            s, _ = make_solver([case], As=[A], Ws=[W], fused=fused, penalty=1)
            out = torch.full((n,), -1, dtype=torch.int16, device="cuda")
            done, ld = s.step(1, colors_out=[out])
            res.append((done, ld, host(out).tolist(), s.get_t(), host(s.W[0]).tobytes()))
            if legal:
                assert done == 0 and ld == [legal[0]] and np.array_equal(host(out), cols[legal[0]])
                assert np.array_equal(host(s.W[0]), W)
            else:
                assert done == 1 and ld == [-1]
            s.close()
        assert res[0] == res[1]


@pytest.mark.parametrize("n,k,D", [(33, 126, 1), (65, 127, 3), (40, 126, 5), (130, 3, 130), (2100, 2, 9), (70, 300, 67)])
def test_packed_group_concentration(n, k, D):
    rng = np.random.default_rng(D)
    cols = rng.integers(0, k, (D, n))
    cols[:, -1] = k - 1                                  # the largest colour of the packed form
    case = GraphCase("mt", KCOL, n, k, D, FP4, "gnp", 0.5)
    s, _ = make_solver([case], Ws=[weights_of(cols, k)])
    ref = sum((cols[d][:, None] == cols[d][None, :]).astype(np.int64) for d in range(D))
    assert np.array_equal(host(s.mtilde(0)), ref)
    s.close()


@pytest.mark.parametrize("n", [64, 65, 130])
def test_graph_check_over_tile_edges(n):
    """One flipped entry on either side of a tile edge, on the diagonal or above 1 is found."""
    import paper_1909_02261_amd as pk
    case = GraphCase("pack", KCOL, n, 3, 1, FP4, "gnp", 0.5)
    A0 = case.adjacency()
    make_solver([case], As=[A0])[0].close()
    for i, j, v in ((0, 63, None), (n - 1, 0, None), (0, n - 1, None), (n - 1, n - 1, 1), (1, 2, 2)):
        A = A0.copy()
        A[i, j] = (1 - A[i, j]) if v is None else v
        with pytest.raises(pk.TcolError):
            make_solver([case], As=[A])


@pytest.mark.parametrize("problem", [KCOL, ECP, BKPART, MSCP])
@pytest.mark.parametrize("n,k,D", [(1, 1, 1), (63, 32, 5), (65, 33, 4), (200, 64, 3), (300, 96, 5), (129, 97, 4), (257, 128, 3),
                                   (520, 45, 16), (190, 256, 6), (130, 200, 9), (1025, 90, 8), (2048, 85, 3)])
def test_contraction_with_row_update_bits(problem, n, k, D):
    """The merged contraction whose tiles hold whole members (and, where the shape rule leaves members to the update
    launch, that one) against the plain schedule, bit for bit, over 5 iterations from t = 203."""
    case = GraphCase(f"gr_n{n}_k{k}_D{D}", problem, n, k, D, FP4, "gnp", 0.5, graph_seed=n, rho=10.0, lam=1e-3, mu=1e-4,
                     nu=1e-3 if problem != KCOL else 0.0, stop_on_legal=0, momentum=0.5 if D in (5, 3) else 0.0)
    out = []
    for fused in (0, 1):
        s, _ = make_solver([case], fused=fused, penalty=1)
        s.set_t(203)
        done, _ = s.step(5)
        assert done == 5
        c, f, _ = s.conflicts(0)
        out.append((host(s.W[0]), host(c), host(f)))
        s.close()
    for a, b in zip(*out):
        assert np.array_equal(a, b)


def test_contraction_with_row_update_in_an_uneven_batch():
    """Graphs whose members fit the column tiles beside graphs that keep the update launch, stops included."""
    cases = [GraphCase(f"gb{i}", KCOL, n, k, 6, FP4, "gnp", p, graph_seed=i, lam=1e-3, mu=1e-4, rho=10.0,
                       stop_on_legal=1 if i == 2 else 0)
             for i, (n, k, p) in enumerate([(310, 90, 0.5), (90, 11, 0.1), (70, 60, 0.1), (400, 300, 0.9), (257, 128, 0.5)])]
    out = []
    for fused in (0, 1):
        s, _ = make_solver(cases, fused=fused, penalty=1)
        s.step(40)
        out.append(([host(w) for w in s.W], [s.get_t(g) for g in range(len(cases))]))
        s.close()
    assert out[0][1] == out[1][1]
    for a, b in zip(out[0][0], out[1][0]):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("prec", [FP32, FP4])
@pytest.mark.parametrize("n,k,D,one", [(1, 1, 1, False), (64, 2, 3, False), (65, 9, 2, False), (257, 129, 4, False), (258, 300, 3, False),
                                       (600, 5, 2, True), (1100, 40, 67, False)])
def test_conflict_counts_without_a_contraction(n, k, D, one, prec):
    """tcol_conflicts, the loss without gradients and the class-conflict matrices against integers, for spread
    colours and all vertices in one class; a row of equal weights takes its lowest colour."""
    rng = np.random.default_rng(n)
    cols = np.full((D, n), k - 1) if one else rng.integers(0, k, (D, n))
    W = weights_of(cols, k)
    W[0, 0, :] = 0.25
    cols[0, 0] = 0
    case = GraphCase("cf", KCOL, n, k, D, prec, "gnp", 0.5, graph_seed=n)
    s, (A,) = make_solver([case], Ws=[W])
    A = A.astype(np.int64)
    f = [int((A * (cols[d][:, None] == cols[d][None, :])).sum()) // 2 for d in range(D)]
    for _ in range(2):                                   # the counters are cleared by each call
        c, fm, fs = s.conflicts(0)
        assert np.array_equal(host(c), cols) and host(fm).tolist() == f and not host(fs).any()
        loss, _, _ = s.loss_grad(0, want_gs=False, want_gw=False)
        assert host(loss)[1] == sum(f)
    C = host(s.class_conflicts(0))
    for d in range(D):
        S = np.zeros((n, k), np.int64)
        S[np.arange(n), cols[d]] = 1
        assert np.array_equal(C[d], S.T @ A @ S)
    s.close()


@pytest.mark.parametrize("prec", [FP32, BF16])
@pytest.mark.parametrize("n,k,D,cm,stop", [(31, 5, 1, 2, 0), (130, 17, 4, 3, 0), (70, 200, 3, 8, 0), (5, 5, 3, 2, 1), (90, 96, 5, 2, 1)])
def test_multicolouring_merged_steps_equal_the_plain_schedule(n, k, D, cm, stop, prec):
    """The update that selects the next colours and ends the iteration against the plain schedule (fused = 0): weights,
    selections, counts and stops, bit for bit, over two calls of 7 iterations."""
    import paper_1909_02261_amd as pk
    torch = torch_mod()
    rng = np.random.default_rng(k)
    A = np.triu(rng.random((n, n)) < (0.5 if not stop else 0.05), 1)
    A = (A | A.T).astype(np.uint8)
    if n == 5:
        A = np.zeros((5, 5), np.uint8)
        for i in range(5):
            A[i, (i + 1) % 5] = A[(i + 1) % 5, i] = 1
    W = rng.normal(0.0, 0.01, (D, n, k)).astype(np.float32)
    W[0, 0, :] = -0.0
    W[0, 0, k // 2] = 0.0                                # -0 and 0 tie: the lowest colours
    dem = rng.integers(1, cm + 1, n)
    out = []
    for fused in (0, 1):
        p = pk.Params(n=n, k=k, D=D, problem=pk.MCOL, precision=prec, lam=1e-3, mu=1e-4, rho=10.0, max_demand=cm,
                      stop_on_legal=stop)
        s = pk.Solver([(torch.from_numpy(A).cuda(), torch.from_numpy(W.copy()).cuda())], [p])
        s.set_options(fused=fused)
        s.set_demand(dem)
        s.set_t(40)
        sel0 = host(s.selection(0))
        res = [s.step(7), s.step(7)]
        c, f, _ = s.conflicts(0)
        out.append((host(s.W[0]), host(s.selection(0)), host(c), host(f), np.array([res[0][0], res[1][0], s.get_t()]),
                    np.array(res[0][1] + res[1][1]), host(s.loss_grad(0)[0])))
        assert sel0[0, 0, 0] == 0
        s.close()
    for a, b in zip(*out):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("prec", [FP32, FP4])
def test_merged_non_finite_update_ends_the_run_there(prec):
    """An update that overflows (at t = 0, in the first of nine iterations, over several replays) stops the graph with an
    error before the next iteration, as the plain schedule does: the same weights and t."""
    import paper_1909_02261_amd as pk
    case = GraphCase("bad", KCOL, 70, 5, 2, prec, "gnp", 0.5, graph_seed=1, stop_on_legal=0)
    W = case.weights()
    W[1, 3, :] = [3e38, 3e38, 3e38, 3.0e38, -3e38]
    case.eta = 3e38
    out = []
    for fused in (0, 1):
        s, _ = make_solver([case], Ws=[W], fused=fused, unroll=4)
        with pytest.raises(pk.TcolError):
            s.step(9)
        out.append((s.get_t(), host(s.W[0]).tobytes()))
        s.close()
    assert out[0] == out[1]
