"""Two grids: which nodes the FP64 guard redoes.  A cell is judged where its projection can still lower
the bound, taken in the order of the key-0 cells and then of the table by 16 rows, whatever the
layout projects beside it: identical doses on one grid (every bound is 0 at the start) guard
no node however steep they are, and the automatic layout guards the nodes that 16 lanes per node
guard, with the same gamma, runs repeatable.  Steep doses on anisotropic grids, thresholds at
which few and most of the neighbourhoods hold an ill-conditioned tetrahedron."""
import numpy as np
import pytest

from dosegen import make_pair_3d
from gpu_util import dev, host
from test_gpu_grids_queue import _sample

pytestmark = pytest.mark.gpu


def _steep(v, k):
    return (1.0 / (1.0 + np.exp(-k * (v.astype(np.float64) - 0.4)))).astype(np.float32)


@pytest.mark.parametrize("cond", [1.0, 100.0])
def test_no_cell_can_lower_a_bound_of_zero(cond):
    import paper_1012_1900_amd as gx
    p = make_pair_3d(57, shape=(12, 14, 13), spacing=(2.5, 1.0, 2.0))
    d = dev(_steep(p.ref, 40.0))
    g, r = gx.gammax_map_grids(d, d.clone(), p.spacing, p.spacing, (0.0, 0.0, 0.0), 0.01, 1.0, 0.1, cond_threshold=cond)
    assert r.n_evaluated > 0 and r.n_pass == r.n_evaluated and np.all(host(g)[host(g) >= 0] == 0.0)
    assert r.n_guarded == 0


@pytest.mark.parametrize("cond", [30.0, 1e4, 1e5])
@pytest.mark.parametrize("shape,sp,ratio,local", [((24, 48, 50), (2.5, 0.8, 0.8), 1.0, True),
                                                  ((20, 40, 44), (2.0, 2.0, 2.0), 0.5, False),
                                                  ((40, 60, 60), (2.0, 1.0, 1.5), 0.8, False)])
def test_layouts_guard_the_same_nodes(shape, sp, ratio, local, cond):
    import paper_1012_1900_amd as gx
    p = make_pair_3d(33, shape, sp)
    esp, org = tuple(ratio * h for h in sp), tuple(0.3 * h for h in sp)
    ev = _sample(_steep(p.eval, 25.0), sp, tuple(int((n - 1) / ratio) + 1 for n in shape), esp, org)
    a = (dev(_steep(p.ref, 25.0)), dev(ev), sp, esp, org, 0.01, 1.0, 0.1, local)
    want, rw = gx.gammax_map_grids(*a, tail_lanes=16, cond_threshold=cond)
    for again in range(2):
        got, rg = gx.gammax_map_grids(*a, cond_threshold=cond)
        assert np.array_equal(host(got), host(want)), again
        assert (rg.n_guarded, rg.n_pass, rg.n_borderline, rg.max_gamma) == (rw.n_guarded, rw.n_pass, rw.n_borderline,
                                                                            rw.max_gamma), again
    print(shape, cond, rw.n_guarded, "of", rw.n_evaluated, flush=True)
    if cond == 30.0:
        assert 0 < rw.n_guarded < rw.n_evaluated
