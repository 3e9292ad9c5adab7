"""The queued walk where nodes with long walks lie together in the list: 81 thousand nodes with
walks of up to 105 thousand rows.  The automatic layout takes less than three quarters of the time
of 64 lanes per node, which gives every node a wave of its own (waves that walked eight of the
long ones in turn took 1.7 to 1.9 times that time, now it is 0.5); gamma and counts as one lane per
node finds them, whether the context knows the walks (later maps) or not (the first), and in a
batch."""
import numpy as np
import pytest

from dosegen import batch_specs, make_batch_pair
from gpu_util import dev, host

pytestmark = pytest.mark.gpu
FIELDS = ("n_evaluated", "n_pass", "n_borderline", "n_tail", "n_cells", "n_guarded", "max_gamma")


def _pair():
    s = batch_specs(43000, 16, 0.5)[7]
    p = make_batch_pair(s)
    return (dev(p.ref), dev(p.eval), p.spacing, s.dd, s.dta, 0.1, s.local)


def test_long_walks_side_by_side():
    import paper_1012_1900_amd as gx
    a = _pair()
    auto, wide = gx.Context(0), gx.Context(0)

    def tail_ms(ctx, **opt):
        return min(gx.gammax_map(*a, ctx=ctx, timing=True, **opt)[1].ms_tail for _ in range(5))

    _, r = gx.gammax_map(*a, ctx=auto)
    assert r.n_tail >= 16384 and r.long_walk_rows > 50000
    got, want = tail_ms(auto), tail_ms(wide, tail_lanes=64)
    print(f"tail {got:.3f} ms, 64 lanes per node {want:.3f} ms", flush=True)
    assert got < 0.75 * want


def test_same_results_and_batch():
    import paper_1012_1900_amd as gx
    a = _pair()
    want, rw = gx.gammax_map(*a, tail_lanes=1, ctx=gx.Context(0))
    ctx, bctx = gx.Context(0), gx.Context(0)
    pair = dict(ref=a[0], ev=a[1], spacing=a[2], dd=a[3], dta=a[4], local=a[6])
    for again in range(3):
        got, rg = gx.gammax_map(*a, ctx=ctx)
        gb, rb = gx.gammax_batch([pair], ctx=bctx)
        for g, r in ((got, rg), (gb[0], rb[0])):
            assert np.array_equal(host(g), host(want)), again
            for f in FIELDS:
                assert getattr(r, f) == getattr(rw, f), (again, f)
