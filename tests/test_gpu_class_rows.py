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
