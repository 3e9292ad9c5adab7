"""The one-launch compaction of small grids against the three-launch one: a context's first map
of a geometry compacts before its cell table exists (three launches, scalars read in between),
its second on the table takes the one launch.  Gamma and every count are the same, at the edges
of a block, of a loop step and of the size range; masks that select nothing but the maximum,
everything, and ragged runs; both normalisations; a radius that outgrows the table; doses that
are not finite, at the first and the last node."""
import numpy as np
import pytest

from gpu_util import dev, host

pytestmark = pytest.mark.gpu

FIELDS = ("n_evaluated", "n_pass", "n_borderline", "n_tail", "n_cells", "n_guarded", "max_gamma", "pass_rate",
          "dose_max", "search_radius")
SHAPES = [(2, 2), (31, 33), (32, 32), (25, 41), (64, 64), (64, 128), (2731, 3), (192, 256), (219, 224), (2, 24577),
          (2, 2, 2), (12, 64, 64), (7, 31, 37)]


def _doses(shape, seed):
    rng = np.random.default_rng(seed)
    ref = rng.uniform(0.0, 1.0, size=shape)
    ref.flat[rng.integers(ref.size)] = 1.25
    ev = ref + 0.02 * rng.standard_normal(shape)
    return ref.astype(np.float32), ev.astype(np.float32)


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("threshold", [0.0, 0.4, 0.9])
def test_small_compaction_is_the_general_one(shape, threshold):
    import paper_1012_1900_amd as gx
    ref, ev = _doses(shape, len(shape) + shape[-1])
    spacing = (2.5, 2.0, 3.0)[:len(shape)]
    for local in (False, True):
        ctx = gx.Context(0)
        a = (dev(ref), dev(ev), spacing, 0.03, 3.0, threshold, local)
        want, rw = gx.gammax_map(*a, ctx=ctx, tail_lanes=16)
        got, rg = gx.gammax_map(*a, ctx=ctx, tail_lanes=16)
        assert np.array_equal(host(got), host(want)), local
        for f in FIELDS:
            assert getattr(rg, f) == getattr(rw, f), (local, f)


def test_radius_that_outgrows_the_table():
    import paper_1012_1900_amd as gx
    ref, ev = _doses((40, 50), 3)
    ev2 = (ref + 12 * (ev - ref)).astype(np.float32)
    ctx, fresh = gx.Context(0), gx.Context(0)
    gx.gammax_map(dev(ref), dev(ev), (2.0, 2.0), 0.03, 3.0, 0.1, ctx=ctx)
    want, rw = gx.gammax_map(dev(ref), dev(ev2), (2.0, 2.0), 0.03, 3.0, 0.1, ctx=fresh, tail_lanes=16)
    got, rg = gx.gammax_map(dev(ref), dev(ev2), (2.0, 2.0), 0.03, 3.0, 0.1, ctx=ctx, tail_lanes=16)
    assert np.array_equal(host(got), host(want))
    for f in FIELDS:
        assert getattr(rg, f) == getattr(rw, f), f


@pytest.mark.parametrize("which", ["ref", "ev"])
@pytest.mark.parametrize("at", [0, -1])
@pytest.mark.parametrize("value", [np.nan, np.inf, -np.inf])
def test_doses_that_are_not_finite_are_refused(which, at, value):
    import paper_1012_1900_amd as gx
    ref, ev = _doses((45, 47), 4)
    ctx = gx.Context(0)
    gx.gammax_map(dev(ref), dev(ev), (2.0, 2.0), 0.03, 3.0, 0.1, ctx=ctx)
    bad = {"ref": ref.copy(), "ev": ev.copy()}
    bad[which].flat[at] = value
    with pytest.raises(gx.GammaxError, match="NaN or infinite"):
        gx.gammax_map(dev(bad["ref"]), dev(bad["ev"]), (2.0, 2.0), 0.03, 3.0, 0.1, ctx=ctx)
    gx.gammax_map(dev(ref), dev(ev), (2.0, 2.0), 0.03, 3.0, 0.1, ctx=ctx)


def test_maximum_of_doses_that_are_all_negative():
    """Local normalisation evaluates no node there, and reports the maximum."""
    import paper_1012_1900_amd as gx
    ref, ev = _doses((33, 70), 5)
    ctx = gx.Context(0)
    gx.gammax_map(dev(ref), dev(ev), (2.0, 2.0), 0.03, 3.0, 0.1, True, ctx=ctx)
    for k in (1, 2):
        _, r = gx.gammax_map(dev(-ref - np.float32(k)), dev(ev), (2.0, 2.0), 0.03, 3.0, 0.1, True, ctx=ctx)
        assert (r.n_evaluated, r.dose_max) == (0, np.float32(-ref - np.float32(k)).max())
