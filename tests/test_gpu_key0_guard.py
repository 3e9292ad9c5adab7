"""The guard's judgement in the 3D key-0 pass: steep neighbourhoods are judged by the denominators of
their whole cells' tetrahedra.  The guarded nodes and every gamma are those of one lane per
cell, which projects all cells with the judgement in it, for thresholds from every neighbourhood
steep to none, doses rough and smooth, grids that are all boundary; and judging every
neighbourhood takes less than half as long again as judging none (projecting the cells again for
it took 1.8 times; the least of 10 maps each)."""
import numpy as np
import pytest

from dosegen import make_pair_3d
from gpu_util import dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cond", [1.0, 30.0, 300.0, 1e4])
@pytest.mark.parametrize("shape,sp,local", [((2, 2, 2), (2.0, 2.0, 2.0), False), ((3, 7, 70), (3.0, 0.8, 1.4), True),
                                            ((17, 33, 35), (2.5, 2.5, 2.5), False)])
def test_same_nodes_as_one_lane_per_cell(shape, sp, local, cond):
    import paper_1012_1900_amd as gx
    rng = np.random.default_rng(shape[2])
    p = make_pair_3d(5, shape, sp)
    for ref, ev in ((p.ref, p.eval),
                    (rng.uniform(0.2, 1.0, size=shape), rng.uniform(0.2, 1.0, size=shape))):
        a = (dev(ref), dev(ev), sp, 0.02, 2.0, 0.1, local)
        want, rw = gx.gammax_map(*a, cell_lanes=8, tail_lanes=1, cond_threshold=cond)
        got, rg = gx.gammax_map(*a, tail_lanes=1, cond_threshold=cond)
        assert np.array_equal(host(got), host(want))
        for f in ("n_evaluated", "n_pass", "n_tail", "n_cells", "n_guarded", "n_fp64_tets", "max_gamma"):
            assert getattr(rg, f) == getattr(rw, f), f


def test_judging_costs_less_than_the_pass():
    import paper_1012_1900_amd as gx
    p = make_pair_3d(31, (96, 128, 128), (2.5, 2.5, 2.5))
    a = (dev(p.ref), dev(p.eval), p.spacing, 0.03, 3.0, 0.1, False)
    ctx = gx.Context(0)

    def key0_ms(**opt):
        return min(gx.gammax_map(*a, ctx=ctx, timing=True, **opt)[1].ms_search for _ in range(10))

    none, every = key0_ms(), key0_ms(cond_threshold=100.0)
    print(f"key-0 pass {1e3 * none:.1f} us, every neighbourhood judged {1e3 * every:.1f} us", flush=True)
    assert every < 1.5 * none
