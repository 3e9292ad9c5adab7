"""Doses at the ends of the float range.  FP64 maps do not depend on the doses' unit: scaled by a power of two
down to where 1 / dD is past the float range (all values still normal floats), gamma is the same bit
for bit, whatever the walk's screening does in floats.  Two grids in FP32: a node whose reference
dose is 1e-30 of its surroundings (local normalisation without a threshold) is infinitely far from
the evaluation surface and does not pass."""
import numpy as np
import pytest

from dosegen import make_pair_3d
from gpu_util import dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("local", [True, False])
@pytest.mark.parametrize("shape,sp", [((9, 14, 15), (1.0, 1.0, 2.5)), ((24, 40, 41), (1.0, 1.0, 1.0))])
def test_fp64_does_not_depend_on_the_unit(shape, sp, local):
    import paper_1012_1900_amd as gx
    rng = np.random.default_rng(shape[2])
    ref = rng.uniform(0.2, 1.0, size=shape).astype(np.float32)
    ev = (ref * rng.uniform(0.9, 1.1, size=shape)).astype(np.float32)
    unit = np.float32(2.0 ** -123)
    assert (ref * unit).min() > np.finfo(np.float32).tiny and np.all(ref * unit / unit == ref)
    with np.errstate(over="ignore"):
        assert np.isinf(np.float32(1.0) / (np.float32(0.03) * (ref * unit).max()))
    want, rw = gx.gammax_map(dev(ref), dev(ev), sp, 0.03, 3.0, 0.0, local, precision="fp64", ctx=gx.Context(0))
    got, rg = gx.gammax_map(dev(ref * unit), dev(ev * unit), sp, 0.03, 3.0, 0.0, local, precision="fp64",
                            ctx=gx.Context(0))
    assert rw.n_tail > 0
    assert np.array_equal(host(got), host(want))
    for f in ("n_evaluated", "n_pass", "n_borderline", "n_tail", "n_cells", "max_gamma"):
        assert getattr(rg, f) == getattr(rw, f), f


@pytest.mark.parametrize("opt", [dict(precision="fp32"), dict(), dict(precision="fp32", tail_lanes=16)],
                         ids=["fp32", "guarded", "16 lanes"])
def test_two_grids_infinite_first_bounds(opt):
    import paper_1012_1900_amd as gx
    shape, sp = (8, 11, 12), (2.0, 2.0, 2.0)
    rng = np.random.default_rng(3)
    p = make_pair_3d(7, shape, sp)
    ref = (0.5 + 0.5 * p.ref).astype(np.float32)
    ev = rng.uniform(0.5, 1.0, size=shape).astype(np.float32)
    low = rng.uniform(size=shape) < 0.05
    ref[low] = 1e-30
    low &= np.all([i < n - 1 for i, n in zip(np.indices(shape), shape)], axis=0)   # (the last nodes lie outside)
    a = (dev(ref), dev(ev), sp, sp, (0.7, 0.9, 1.1), 0.03, 3.0, 0.0, True)
    ctx = gx.Context(0)
    for again in range(2):
        g, r = gx.gammax_map_grids(*a, ctx=ctx, **opt)
        gh = host(g)
        inside = gh >= 0
        assert np.all(np.isinf(gh[low & inside])) and (low & inside).sum() > 20
        # the others as a map in which those nodes are not evaluated
        ref2 = np.where(ref < 1e-20, np.float32(-1.0), ref).astype(np.float32)
        g2, r2 = gx.gammax_map_grids(dev(ref2), *a[1:], ctx=gx.Context(0), **opt)
        rest = inside & ~(ref < 1e-20)
        assert np.array_equal(gh[rest], host(g2)[rest]) and r.n_pass == r2.n_pass, again
