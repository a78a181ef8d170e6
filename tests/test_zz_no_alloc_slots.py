"""tcol_conflicts_noalloc where the conflict slots (64 int32 per member) are more than an S^T operand of the
same graph would be: one colour, many members, few vertices.  Against tcol_conflicts, bit-exact."""
import numpy as np
import pytest

from tcolgen import BF16, BKPART, FP4, KCOL, MSCP, GraphCase

from test_zz_no_alloc import noalloc, with_context

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("problem", [KCOL, BKPART, MSCP])
@pytest.mark.parametrize("n,k,D", [(256, 1, 1024), (200, 1, 600), (256, 1, 584), (256, 1, 585), (3, 1, 1024), (250, 2, 1024),
                                   (257, 1, 1024)])
def test_noalloc_slots_beside_the_colours(problem, n, k, D):
    torch = __import__("torch")
    case = GraphCase("slots", problem, n, k, D, FP4 if n % 2 else BF16, "gnp", 0.5, graph_seed=n,
                     nu=1e-3 if problem != KCOL else 0.0)
    A, W = case.adjacency(), case.weights()
    want = with_context(case, A, W)
    if k == 1:                                           # every edge conflicts in every member
        assert want[1].tolist() == [0 if problem == BKPART else int(A.sum()) // 2] * D
    for _ in range(3):
        got = noalloc(case, torch.from_numpy(A).cuda(), torch.from_numpy(W).cuda())
        for g, w, what in zip(got, want, ("colours", "main fitness", "added fitness")):
            assert np.array_equal(g, w), (case.name, what)
