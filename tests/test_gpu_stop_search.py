"""The merged schedule's search for legal members over the edges of its split: several blocks a member (1024 vertices
each), class masks in several pieces (many colours), words of one vertex, and one conflicting (or cut) pair at either
end, inside a word and across pieces."""
import numpy as np
import pytest

from tcolgen import BKPART, ECP, FP4, FP32, KCOL, KPART, GraphCase

from gpu_util import host, make_solver, torch_mod
from test_gpu_merged import weights_of

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("problem", [KCOL, ECP, KPART, BKPART])
@pytest.mark.parametrize("n,k,prec", [(2, 1, FP4), (65, 5, FP4), (64, 30, FP32), (1024, 8, FP4), (1025, 5, FP32), (1026, 513, FP4),
                                      (2112, 300, FP4), (3000, 3, FP4)])
def test_one_bad_pair_anywhere(problem, n, k, prec):
    torch = torch_mod()
    rng = np.random.default_rng(n + k)
    base = np.arange(n) % k                              # equitable; i, j share a class when k divides i - j
    part = problem in (KPART, BKPART)
    far = (n - 1) // k * k
    if part:
        pairs = [(0, 1), (n - 1, n - 2), (0, n - 1 if (n - 1) % k else n - 2), (n // 2, n // 2 + 1)] if k > 1 else []
    else:
        pairs = [(0, k), (0, far), (n - 1, n - 1 - k), (n // 2, n // 2 + k)] if n > k + n // 2 else [(0, k), (n - 1, n - 1 - k)]
    same = base[:, None] == base[None, :]
    u = np.triu(rng.random((n, n), dtype=np.float32) < 0.3, 1) & (same if part else ~same)
    for pair in pairs + [None]:
        A = u.copy()
        if pair is not None:
            i, j = min(pair), max(pair)
            assert i != j and same[i, j] != part
            A[i, j] = True
        A = (A | A.T).astype(np.uint8)
        W = weights_of(np.tile(base, (2, 1)), k)
        case = GraphCase("search", problem, n, k, 2, prec, "gnp", 0.5, stop_on_legal=1, eta=1e-9, rho=1.0, nu=1e-3)
        s, _ = make_solver([case], As=[A], Ws=[W], fused=1, penalty=1)
        out = torch.full((n,), -1, dtype=torch.int16, device="cuda")
        done, ld = s.step(3, colors_out=[out])
        if pair is None:
            assert (done, ld) == (0, [0]) and np.array_equal(host(out), base)
        else:
            assert (done, ld) == (3, [-1]), pair
            # one vertex of the pair moved away in member 1 (its class sizes then differ: not with an added fitness)
            if problem == KCOL and k > 1:
                cols = np.tile(base, (2, 1))
                free = [c for c in range(k) if not A[i][base == c].any()]
                if free:
                    cols[1, i] = free[0]
                    s.W[0].copy_(torch.from_numpy(weights_of(cols, k)))
                    assert s.step(2)[1] == [1]
        s.close()
