"""Long tail lists on every path that walks them by the queue: FP64 lists whose entries are claimed
(262144 and more), maps with and without cell ranges on one context, pairs of a batch.  Every
node walks (a noisy offset), so the grid gives the list's length.  FP64 against the oracle at the bar of
the other FP64 tests (1e-7 max(1, gamma); cells 1e-4, keys being rounded to float); the others bit
for bit against one lane per node.  That a later map has ranges is asserted from its first one:
at least 16384 walking nodes and two visited cells per grid node."""
import numpy as np
import pytest

import oracle
from gpu_util import dev, host

pytestmark = pytest.mark.gpu
FIELDS = ("n_evaluated", "n_pass", "n_borderline", "n_tail", "n_cells", "n_guarded", "max_gamma")


def _offset_pair(shape):
    rng = np.random.default_rng(shape[-1])
    ref = np.full(shape, 0.75, dtype=np.float32)
    return ref, (ref + 0.04 + 0.004 * rng.standard_normal(shape)).astype(np.float32)


def _ranges_follow(r, ref):
    return r.n_tail >= 16384 and r.n_cells - 2 ** ref.ndim * r.n_evaluated >= 2 * ref.size


@pytest.mark.parametrize("shape", [(63, 65, 64), (64, 64, 64), (71, 67, 61)])
def test_fp64_lists_dealt_and_claimed(shape):
    import paper_1012_1900_amd as gx
    ref, ev = _offset_pair(shape)
    sp = (2.0, 2.0, 2.0)
    o = oracle.gamma(ref, ev, sp, 0.03, 3.0, 0.0)
    a = (dev(ref), dev(ev), sp, 0.03, 3.0, 0.0, False)
    ctx = gx.Context(0)
    first, r = gx.gammax_map(*a, ctx=ctx, precision="fp64")
    gh = host(first).astype(np.float64)
    assert np.all(np.abs(gh - o.gamma) <= 1e-7 * np.maximum(1.0, o.gamma))
    assert abs(int(r.n_cells) - o.cells_visited) <= 1e-4 * o.cells_visited + 1
    assert r.n_tail == ref.size and _ranges_follow(r, ref)
    for again in range(2):   # with ranges
        got, rg = gx.gammax_map(*a, ctx=ctx, precision="fp64")
        assert np.array_equal(host(got), host(first)), again
        for f in FIELDS:
            assert getattr(rg, f) == getattr(r, f), (again, f)


@pytest.mark.parametrize("shape,opt", [((40, 48, 50), {}), ((40, 48, 50), dict(precision="fp32")), ((64, 64, 65), {}),
                                       ((541, 541), {}), ((400, 300), dict(sort="bound")),
                                       ((40, 48, 50), dict(sort="dd"))])
def test_maps_with_ranges_and_batches_equal_one_lane_per_node(shape, opt):
    import paper_1012_1900_amd as gx
    ref, ev = _offset_pair(shape)
    sp = (1.0,) * len(shape)
    a = (dev(ref), dev(ev), sp, 0.03, 3.0, 0.0, False)
    plain = {k: v for k, v in opt.items() if k != "sort"}
    want, rw = gx.gammax_map(*a, tail_lanes=1, ctx=gx.Context(0), **plain)
    assert rw.n_tail == ref.size and _ranges_follow(rw, ref)
    pair = [dict(ref=a[0], ev=a[1], spacing=sp, dd=0.03, dta=3.0, threshold=0.0)] * 2
    ctx, bctx, mctx = gx.Context(0), gx.Context(0), gx.Context(0)
    for again in range(3):
        runs = [gx.gammax_map(*a, ctx=ctx, **opt)]
        for fn, c in ((gx.gammax_batch, bctx), (gx.gammax_map_many, mctx)):
            gs, rs = fn(pair, ctx=c, **opt)
            runs += list(zip(gs, rs))
        for g, r in runs:
            assert np.array_equal(host(g), host(want)), again
            for f in FIELDS:
                assert getattr(r, f) == getattr(rw, f), (again, f)
