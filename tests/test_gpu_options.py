"""Tile options: a tile that the caller names is the one that runs, also where it is the one that the automatic
choice shows; options that are changed one at a time leave the others as the caller left them."""
import pytest

from tcolgen import FP4, KCOL, GraphCase

from gpu_util import make_solver

pytestmark = pytest.mark.gpu


def tile(s):
    o = s.options()
    return o["tile_bm"], o["tile_ntw"]


def test_named_tile_stays_named():
    case = GraphCase("tile", KCOL, 1000, 28, 128, FP4, "gnp", 0.5, graph_seed=13, stop_on_legal=0)
    s, _ = make_solver([case])
    auto = tile(s)
    # the epilogue path's own choice, and with the shown tile by name
    s.set_options(fused=2)
    own = tile(s)
    assert own != auto, "the case has to tell the two apart"
    s.set_options(fused=1)
    assert tile(s) == auto                               # automatic again
    s.set_options(fused=2, tile_bm=auto[0], tile_ntw=auto[1])
    assert tile(s) == auto
    s.set_options(fused=1)
    s.set_options(fused=2, penalty=1)
    assert tile(s) == auto                               # still the named one
    s.set_options(tile_bm=0, tile_ntw=0)
    assert tile(s) == own
    s.set_options(fused=1)
    s.set_options(tile_bm=auto[0])                       # one half named: the other as shown
    assert tile(s) == auto
    s.set_options(fused=2)
    assert tile(s) == auto
    s.close()


@pytest.mark.parametrize("n,k,D", [(1000, 90, 64), (500, 50, 64), (1000, 28, 128)])
def test_shown_tile_is_the_one_of_the_storing_contractions(n, k, D):
    """Where the contraction of an iteration takes the row update in a tile of its own, the tile shown, which the gradients and the
    class conflicts take, is the choice for storing G: the plain schedule's."""
    case = GraphCase("shown", KCOL, n, k, D, FP4, "gnp", 0.5, graph_seed=13, stop_on_legal=0)
    s, _ = make_solver([case])
    shown = tile(s)
    s.set_options(fused=0)
    assert tile(s) == shown
    s.close()
