"""The queued walk of long tails (automatic layout) against the one-lane-per-node walk, which
visits the rows one by one: gamma bit for bit the same (the minimum does not depend on its
order and a skipped cell cannot lower it), the same passes, tail nodes, visited cells (those
with key below the final gamma) and guarded nodes.  Sizes where it can go wrong: a tail just
past the least the queued walk takes (groups without a node), odd grids with their boundary
in the dose, anisotropic cells, walks of thousands of rows, every cell suspected of
ill-conditioning, cell ranges on (the context's earlier map had a long tail) and off, 2D."""
import numpy as np
import pytest

from dosegen import make_pair_2d, make_pair_3d
from gpu_util import dev, host

pytestmark = pytest.mark.gpu
MIN_TAIL = 16384


CASES = {
    # name: (pair, spacing, dd, dta, threshold, local, options)
    "shifted": lambda: (make_pair_3d(3, (41, 53, 67), (1.5, 1.5, 1.5)), 0.02, 2.0, 0.1, False, {}),
    "local, long walks": lambda: (make_pair_3d(40064, (48, 64, 64), (1.0, 1.0, 1.0)), 0.01, 1.0, 0.05, True, {}),
    "anisotropic": lambda: (make_pair_3d(5, (37, 61, 59), (3.0, 1.0, 1.7)), 0.01, 2.0, 0.1, False, {}),
    "fp32": lambda: (make_pair_3d(6, (40, 64, 64), (1.25, 1.25, 1.25)), 0.02, 2.0, 0.1, False, dict(precision="fp32")),
    "guard suspects": lambda: (make_pair_3d(7, (33, 47, 51), (1.5, 1.5, 1.5)), 0.01, 2.0, 0.1, True,
                               dict(cond_threshold=300.0)),
    "2d": lambda: (make_pair_2d(8, (601, 633), (0.25, 0.25)), 0.01, 2.0, 0.05, True, {}),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_queued_walk_is_the_sequential_walk(name):
    import paper_1012_1900_amd as gx
    p, dd, dta, thr, local, opt = CASES[name]()
    ev = p.eval + np.where(p.ref >= 0.1 * p.ref.max(), np.float32(-0.04), np.float32(0.0))   # most nodes walk
    a = (dev(p.ref), dev(ev), p.spacing, dd, dta, thr, local)
    want, rw = gx.gammax_map(*a, tail_lanes=1, ctx=gx.Context(0), **opt)
    assert rw.n_tail >= MIN_TAIL, rw.n_tail
    ctx = gx.Context(0)
    for again in range(3):   # the second and third map know the tail: cell ranges
        got, rg = gx.gammax_map(*a, ctx=ctx, **opt)
        assert np.array_equal(host(got), host(want)), (name, again)
        for f in ("n_evaluated", "n_pass", "n_borderline", "n_tail", "n_cells", "n_guarded", "max_gamma"):
            assert getattr(rg, f) == getattr(rw, f), (name, again, f)


@pytest.mark.parametrize("shape", [(16, 32, 32), (5, 29, 113), (17, 31, 33), (20, 32, 32)])
def test_tail_just_past_the_least(shape):
    """A noisy offset: every node walks, so the grid gives the tail's length (16384, 16385,
    17391 and 20480 nodes; the launch holds more groups than that)."""
    import paper_1012_1900_amd as gx
    rng = np.random.default_rng(shape[2])
    ref = np.full(shape, 0.75, dtype=np.float32)
    ev = (ref + 0.04 + 0.004 * rng.standard_normal(shape)).astype(np.float32)
    a = (dev(ref), dev(ev), (1.0, 1.0, 1.0), 0.03, 3.0, 0.0, False)
    want, rw = gx.gammax_map(*a, tail_lanes=1, ctx=gx.Context(0))
    assert rw.n_tail == ref.size >= MIN_TAIL
    ctx = gx.Context(0)
    for again in range(2):
        got, rg = gx.gammax_map(*a, ctx=ctx)
        assert np.array_equal(host(got), host(want)), again
        assert (rg.n_cells, rg.n_tail, rg.n_pass) == (rw.n_cells, rw.n_tail, rw.n_pass), again


def test_sorted_tail_takes_the_queued_walk_too():
    import paper_1012_1900_amd as gx
    p, dd, dta, thr, local, _ = CASES["shifted"]()
    a = (dev(p.ref), dev(p.eval - np.float32(0.04)), p.spacing, dd, dta, thr, local)
    want, rw = gx.gammax_map(*a)
    got, rg = gx.gammax_map(*a, sort="dd")
    assert rw.n_tail >= MIN_TAIL
    assert np.array_equal(host(got), host(want)) and rg.n_cells == rw.n_cells


@pytest.mark.parametrize("shape", [(63, 65, 64), (64, 64, 64), (71, 67, 61), (541, 541)])
def test_tail_whose_nodes_are_claimed(shape):
    """Every node walks again: lists of less than eight entries per group of the launch (dealt
    out), of eight, and of ragged lengths past that (the rest claimed by the waves), 3D and 2D,
    in list order and sorted."""
    import paper_1012_1900_amd as gx
    rng = np.random.default_rng(shape[1])
    ref = np.full(shape, 0.75, dtype=np.float32)
    ev = (ref + 0.04 + 0.004 * rng.standard_normal(shape)).astype(np.float32)
    a = (dev(ref), dev(ev), (1.0,) * len(shape), 0.03, 3.0, 0.0, False)
    want, rw = gx.gammax_map(*a, tail_lanes=1, ctx=gx.Context(0))
    assert rw.n_tail == ref.size
    ctx = gx.Context(0)
    for opt in ({}, {}, dict(sort="bound")):
        got, rg = gx.gammax_map(*a, ctx=ctx, **opt)
        assert np.array_equal(host(got), host(want)), opt
        assert (rg.n_cells, rg.n_tail, rg.n_pass) == (rw.n_cells, rw.n_tail, rw.n_pass), opt
