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


@pytest.mark.parametrize("precision", ["guarded", "fp32"])
@pytest.mark.parametrize("shape,ratio,sp,local", [((40, 64, 64), 0.5, 1.5, False), ((48, 80, 80), 1.0, 1.0, False),
                                                  ((36, 50, 52), 1.0, 1.0, True)])
def test_either_walk_gives_the_same_map(shape, ratio, sp, local, precision):
    """A context's first map walks its tail by 16 lanes per node; the next ones by the queued
    walk where the first found many nodes for its longest walk (the first two cases; the last
    one has walks of hundreds of rows for its few nodes): the same bits and counts."""
    import paper_1012_1900_amd as gx
    sp = (sp,) * 3
    p = make_pair_3d(33, shape, sp)
    esp, org = tuple(ratio * h for h in sp), tuple(0.3 * h for h in sp)
    ev = _sample(p.eval, sp, tuple(int((n - 1) / ratio) + 1 for n in shape), esp, org)
    a = (dev(p.ref), dev(ev), sp, esp, org, 0.02, 2.0, 0.1, local)
    ctx = gx.Context(0)
    first, r0 = gx.gammax_map_grids(*a, ctx=ctx, precision=precision)
    lanes, rl = gx.gammax_map_grids(*a, ctx=gx.Context(0), precision=precision, tail_lanes=16)
    assert np.array_equal(host(first), host(lanes)) and abs(int(r0.n_cells) - int(rl.n_cells)) <= 16 * r0.n_evaluated
    for _ in range(3):
        g, r = gx.gammax_map_grids(*a, ctx=ctx, precision=precision)
        assert np.array_equal(host(g), host(first))
        for f in ("n_evaluated", "n_pass", "n_borderline", "n_cells", "n_guarded", "max_gamma"):
            assert getattr(r, f) == getattr(r0, f), f


def test_long_walks_keep_the_lane_groups():
    """A tail whose longest walk has thousands of rows takes no longer in the automatic layout than
    by 16 lanes per node (the queued walk took 1.2 times the whole map's time, in other cases up to 4
    times; the least of 12 maps each, with 10 % to spare)."""
    import time

    import torch

    import paper_1012_1900_amd as gx
    shape, sp = (48, 96, 96), (5.0, 1.2, 1.2)
    p = make_pair_3d(33, shape, sp)
    org = tuple(0.3 * h for h in sp)
    a = (dev(_steep(p.ref, 40.0)), dev(_sample(_steep(p.eval, 40.0), sp, shape, sp, org)), sp, sp, org, 0.02, 2.0, 0.1)

    def least(**opt):
        ctx, t = gx.Context(0), []
        for _ in range(15):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            gx.gammax_map_grids(*a, ctx=ctx, **opt)
            t.append(time.perf_counter() - t0)
        return min(t[3:])

    auto, lanes = least(), least(tail_lanes=16)
    print(f"automatic {1e6 * auto:.0f} us, 16 lanes {1e6 * lanes:.0f} us", flush=True)
    assert auto < 1.1 * lanes
