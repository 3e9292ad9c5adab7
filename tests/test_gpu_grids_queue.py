"""Two grids: the automatic layout (queued projections in the key-0 pass and in the walk) against
16 lanes per node in the walk, and against the oracle's bar: gamma bit for bit the same between
the layouts, counts equal, runs repeatable.  Evaluation grids of two nodes along an axis, finer,
coarser and offset ones, long walks (local normalisation), steep doses that the guard judges."""
import numpy as np
import pytest

import oracle
from dosegen import make_pair_2d, make_pair_3d
from gpu_util import assert_parity, dev, host

pytestmark = pytest.mark.gpu


def _sample(vol, spacing, shape, sp, org):
    """The volume at the nodes of another grid (linear, clamped)."""
    from scipy import ndimage
    ax = [(org[i] + np.arange(shape[i]) * sp[i]) / spacing[i] for i in range(vol.ndim)]
    return ndimage.map_coordinates(vol, np.meshgrid(*ax, indexing="ij"), order=1, mode="nearest").astype(np.float32)


@pytest.mark.parametrize("shape,eshape,esp,org,local,dd,dta", [
    ((12, 30, 33), (24, 61, 70), (1.0, 1.0, 1.0), (0.3, 0.1, 0.7), False, 0.03, 3.0),
    ((12, 30, 33), (2, 15, 17), (20.0, 4.0, 4.0), (0.5, 0.0, 0.0), False, 0.02, 2.0),
    ((20, 40, 41), (20, 40, 41), (2.0, 2.0, 2.0), (1.0, 1.0, 1.0), True, 0.01, 2.0),
    ((9, 35, 64), (9, 71, 30), (2.0, 1.0, 4.0), (0.0, 0.5, 1.5), True, 0.03, 3.0),
])
def test_layouts_agree_and_meet_the_bar(shape, eshape, esp, org, local, dd, dta):
    import paper_1012_1900_amd as gx
    sp = (2.0, 2.0, 2.0)
    p = make_pair_3d(17, shape=shape, spacing=sp)
    ev = _sample(p.eval, sp, eshape, esp, org)
    a = (dev(p.ref), dev(ev), sp, esp, org, dd, dta, 0.1, local)
    got, rg = gx.gammax_map_grids(*a)
    o = oracle.gamma_grids(p.ref, ev, sp, esp, org, dd, dta, 0.1, local)
    assert_parity(host(got), o.gamma, str(shape))
    for lanes in (16, 64):
        want, rw = gx.gammax_map_grids(*a, tail_lanes=lanes)
        if rg.n_guarded == rw.n_guarded == 0:
            assert np.array_equal(host(got), host(want))
        assert (rg.n_evaluated, rg.n_pass) == (rw.n_evaluated, rw.n_pass)
    again, ra = gx.gammax_map_grids(*a)
    assert np.array_equal(host(got), host(again)) and ra.n_cells == rg.n_cells and ra.n_guarded == rg.n_guarded
    for opt in (dict(cond_threshold=30.0), dict(cond_threshold=1.0), dict(precision="fp32")):
        g, r = gx.gammax_map_grids(*a, **opt)
        assert_parity(host(g), o.gamma, f"{shape} {opt}")
        assert r.n_evaluated == rg.n_evaluated
        if opt.get("cond_threshold"):
            assert r.n_guarded > 0


def test_2d_extruded():
    import paper_1012_1900_amd as gx
    p = make_pair_2d(3, (70, 90), (1.0, 1.0))
    ev = _sample(p.eval, (1.0, 1.0), (35, 47), (2.0, 1.9), (0.5, 0.25))
    a = (dev(p.ref), dev(ev), (1.0, 1.0), (2.0, 1.9), (0.5, 0.25), 0.02, 2.0)
    got, rg = gx.gammax_map_grids(*a)
    want, rw = gx.gammax_map_grids(*a, tail_lanes=16)
    assert np.array_equal(host(got), host(want)) and rg.n_pass == rw.n_pass
