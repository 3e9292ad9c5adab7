"""FP64 precision in 3D (the key-0 pass and the queued walk in double) against the FP64 oracle:
grids that are all boundary, odd sizes, anisotropic spacing, local normalisation with long
walks, a tail in which few groups have a node and one of more than 16384 nodes.  The result is
the oracle's gamma rounded to float (2^-24 relative; the two add their terms in different
orders in 64 bits, far below that), so 1e-7 max(1, gamma) as the other FP64 tests; visited cells
as the exact walk's but for keys rounded to float (1e-4)."""
import numpy as np
import pytest

import oracle
from dosegen import make_pair_3d
from gpu_util import dev, host

pytestmark = pytest.mark.gpu


def _rough(seed, shape):
    rng = np.random.default_rng(seed)
    ref = rng.uniform(0.2, 1.0, size=shape)
    return ref.astype(np.float32), (ref + 0.3 * rng.standard_normal(shape)).astype(np.float32)


@pytest.mark.parametrize("shape,spacing,local", [((2, 2, 2), (2.0, 2.0, 2.0), False), ((5, 9, 66), (3.0, 0.8, 1.4), False),
                                                 ((7, 33, 31), (1.0, 1.0, 1.0), True)])
def test_fp64_rough_doses(shape, spacing, local):
    import paper_1012_1900_amd as gx
    ref, ev = _rough(shape[2], shape)
    o = oracle.gamma(ref, ev, spacing, 0.05, 2.0, 0.1, local)
    g, r = gx.gammax_map(dev(ref), dev(ev), spacing, 0.05, 2.0, 0.1, local, precision="fp64")
    gh = host(g).astype(np.float64)
    assert np.array_equal(gh >= 0, o.gamma >= 0)
    m = o.gamma >= 0
    assert np.all(np.abs(gh[m] - o.gamma[m]) <= 1e-7 * np.maximum(1.0, o.gamma[m]))
    assert abs(int(r.n_cells) - o.cells_visited) <= 1e-4 * o.cells_visited + 1


@pytest.mark.parametrize("shape,h,crit,local,error", [((24, 41, 43), 1.5, (0.02, 2.0), False, -0.04),
                                                      ((40, 48, 50), 1.0, (0.02, 2.0), True, 0.0),
                                                      ((20, 30, 35), 2.5, (0.03, 3.0), False, 0.0)])
def test_fp64_walks(shape, h, crit, local, error):
    import paper_1012_1900_amd as gx
    p = make_pair_3d(11, shape=shape, spacing=(h,) * 3)
    ev = (p.eval + np.where(p.ref >= 0.1 * p.ref.max(), np.float32(error), np.float32(0))).astype(np.float32)
    o = oracle.gamma(p.ref, ev, p.spacing, *crit, 0.1, local)
    g, r = gx.gammax_map(dev(p.ref), dev(ev), p.spacing, *crit, 0.1, local, precision="fp64")
    gh = host(g).astype(np.float64)
    m = o.gamma >= 0
    assert np.array_equal(gh >= 0, m)
    assert np.all(np.abs(gh[m] - o.gamma[m]) <= 1e-7 * np.maximum(1.0, o.gamma[m]))
    assert abs(int(r.n_cells) - o.cells_visited) <= 1e-4 * o.cells_visited + 1
    assert r.n_tail > 0
