"""f_color through the contraction's gather for every instantiated tile shape: a multicolouring context with one colour
per vertex counts its conflicts that way (other contexts count them from the adjacency bits)."""
import numpy as np
import pytest

import oracle
from tcolgen import BF16, FP4, FP8, FP32, KCOL, GraphCase

from gpu_util import host, torch_mod
from test_gpu_parity import SHAPES

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [FP32, BF16, FP8, FP4])
def test_gather_every_tile_shape(prec):
    import paper_1909_02261_amd as pk
    torch = torch_mod()
    case = GraphCase("gather", KCOL, 1000, 28, 40, prec, "gnp", 0.5, graph_seed=13)
    A, W = case.adjacency(), case.weights()
    ref = oracle.fcolor(A, oracle.colors(W))
    p = pk.Params(n=case.n, k=case.k, D=case.D, problem=pk.MCOL, precision=prec, max_demand=1, stop_on_legal=0)
    s = pk.Solver([(torch.from_numpy(A).cuda(), torch.from_numpy(W).cuda())], [p])
    bad = []
    for bm, ntw in SHAPES:
        s.set_options(tile_bm=bm, tile_ntw=ntw)
        o = s.options()
        assert (o["tile_bm"], o["tile_ntw"]) == (bm, ntw)
        for rep in range(4):    # a stage-buffer race shows up only now and then
            got = host(s.conflicts(0)[1])
            if not np.array_equal(got, ref):
                bad.append(((bm, ntw), rep, np.nonzero(got != ref)[0].tolist()[:8]))
            loss = host(s.loss_grad(0)[0])
            if loss[1] != ref.sum():
                bad.append(((bm, ntw), rep, "loss", loss[1], int(ref.sum())))
    s.close()
    assert not bad, bad
