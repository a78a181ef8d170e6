"""The fp32 class-row sums: they take the adjacency from the signs of the penalty operand, so the signs have to
hold for every parameter set that is accepted, and their time must not depend on how the colours are spread."""
import numpy as np
import pytest

from tcolgen import FP32, KCOL, KPART, GraphCase

from gpu_util import host, make_solver, torch_mod

pytestmark = pytest.mark.gpu

# the exponent of a term whose weight is 0 is free: its table entries would be -0 (a negative exponent) or, where the
# power overflows, NaN; with a weight, infinite entries times t = 0 are NaN
PARAMS = {"alpha_negative": dict(lam=0.0, alpha=-1.0, mu=1e-4, beta=1.2),
          "beta_negative": dict(lam=1e-3, alpha=2.5, mu=0.0, beta=-1.0),
          "both_negative": dict(lam=0.0, alpha=-1.0, mu=0.0, beta=-2.0),
          "alpha_overflow": dict(lam=0.0, alpha=900.0, mu=1e-4, beta=1.2),
          "both_overflow": dict(lam=0.0, alpha=900.0, mu=0.0, beta=900.0),
          "infinite_table": dict(lam=1e-3, alpha=900.0, mu=1e-3, beta=900.0)}


@pytest.mark.parametrize("problem", [KCOL, KPART])
@pytest.mark.parametrize("name", list(PARAMS))
def test_adjacency_signs_of_any_parameters(name, problem):
    """Steps, gradients and conflicts against the plain schedule's contraction, which reads A itself: the same bits."""
    kw = PARAMS[name]
    case = GraphCase("signs", problem, 150, 7, 9, FP32, "gnp", 0.5, graph_seed=4, rho=10.0, stop_on_legal=0, **kw)
    cols = np.random.default_rng(2).integers(0, 7, (9, 150))
    W = np.random.default_rng(3).normal(0.0, 0.01, (9, 150, 7)).astype(np.float32)
    np.put_along_axis(W, cols[:, :, None], 1.0, axis=2)
    # the infinite entries are finite sums only while the penalty is inactive, at t = 0
    t = 0 if name == "infinite_table" else 7
    out = []
    for fused in (0, 1):
        s, (A,) = make_solver([case], Ws=[W], fused=fused, penalty=1)
        s.set_t(t)
        loss, gs, _ = s.loss_grad(0)
        s.step(1 if name == "infinite_table" else 3)
        out.append(host(s.W[0]))
        gs, f = host(gs), host(loss)[1]
        s.close()
    assert np.array_equal(out[0], out[1])
    # the conflicts of the loss and, where the penalty is inactive, the gradient are whole numbers
    A = A.astype(np.int64)
    S = (cols[:, :, None] == np.arange(7)).astype(np.int64)
    AS = np.stack([A @ S[d] for d in range(9)])
    ref = [int((AS[d] * S[d]).sum()) // 2 for d in range(9)]
    assert f == (sum(ref) if problem == KCOL else 9 * int(A.sum()) // 2 - sum(ref))
    if (kw["lam"] == 0.0 and kw["mu"] == 0.0) or t == 0:
        assert np.array_equal(gs, (AS if problem == KCOL else -AS).astype(np.float32))


@pytest.mark.parametrize("t", [0, 9])
@pytest.mark.parametrize("sizes", [(256, 257), (252, 253, 300), (1, 320, 0, 321, 5), (600,), (1025, 3), (0, 383, 384, 385, 2),
                                   (511, 512, 513, 514), (260, 0, 0, 1900), (257, 1, 0, 0, 0, 0, 0, 0, 3)], ids=str)
def test_large_classes_bits(sizes, t):
    """Classes about and beyond the size from which a block's waves count them together (lists past 256 entries), with
    one member that has every vertex in one class: steps against the plain schedule and gradients against the fp32 contraction
    of a multicolouring context with one colour per vertex, bit for bit."""
    import paper_1909_02261_amd as pk
    torch = torch_mod()
    n, k, D = sum(sizes), len(sizes) + 3, 3
    rng = np.random.default_rng(n)
    cols = np.stack([rng.permutation(np.repeat(np.arange(len(sizes)), sizes)) + 1, np.full(n, k - 1),
                     rng.permutation(np.repeat(np.arange(len(sizes)), sizes))])
    W = rng.normal(0.0, 0.01, (D, n, k)).astype(np.float32)
    np.put_along_axis(W, cols[:, :, None], 1.0, axis=2)
    A = np.triu(rng.random((n, n), dtype=np.float32) < 0.5, 1)
    A = (A | A.T).astype(np.uint8)
    case = GraphCase("large", KCOL, n, k, D, FP32, "gnp", 0.5, lam=1e-3, mu=1e-4, stop_on_legal=0)
    out = []
    for fused in (0, 1):
        s, _ = make_solver([case], As=[A], Ws=[W], fused=fused, penalty=1)
        s.set_t(t)
        if fused:
            loss, gs, gw = (host(x) for x in s.loss_grad(0))
        s.step(2)
        out.append(host(s.W[0]))
        s.close()
    assert np.array_equal(out[0], out[1])
    p = pk.Params(n=n, k=k, D=D, problem=pk.MCOL, precision=FP32, lam=1e-3, mu=1e-4, max_demand=1, stop_on_legal=0)
    s = pk.Solver([(torch.from_numpy(A).cuda(), torch.from_numpy(W).cuda())], [p])
    s.set_t(t)
    ref = [host(x) for x in s.loss_grad(0)]
    s.close()
    assert np.array_equal(gs, ref[1]) and np.array_equal(gw, ref[2]) and loss[1] == ref[0][1]


@pytest.mark.parametrize("n,k,D", [(40, 9, 3), (65, 31, 2), (300, 33, 3), (300, 65, 4), (500, 97, 5), (510, 120, 16), (700, 129, 9),
                                   (777, 193, 16), (600, 290, 32), (800, 385, 33), (900, 576, 16), (2000, 30, 3), (1500, 3, 20)])
def test_class_rows_bits_of_every_row_width(n, k, D):
    """Sizes on the sums' side of the rule, one for each width of the row update and its edges, empty classes among
    them, against the plain schedule over 3 iterations from t = 203 (the smoothing at t = 204 among them)."""
    case = GraphCase("width", KCOL, n, k, D, FP32, "gnp", 0.5, graph_seed=n, rho=10.0, lam=1e-3, mu=1e-4, stop_on_legal=0)
    out = []
    for fused in (0, 1):
        s, _ = make_solver([case], fused=fused, penalty=1)
        s.set_t(203)
        s.step(3)
        out.append(host(s.W[0]))
        s.close()
    assert np.array_equal(out[0], out[1])
