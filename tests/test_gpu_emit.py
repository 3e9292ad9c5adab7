"""The compaction of large grids, eight tiles per block, against one tile per block (which batches
use): the same gamma and counts.  Tile counts that are and are not a multiple of eight, a grid
that ends inside a tile, runs without a masked node, every node masked, almost none."""
import numpy as np
import pytest

from gpu_util import dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(3, 1024, 1024), (3, 1025, 1025), (1773, 1777)])
@pytest.mark.parametrize("fill", ["runs", "all", "few"])
def test_wide_compaction_is_the_tiled_one(shape, fill):
    import paper_1012_1900_amd as gx
    rng = np.random.default_rng(shape[-1])
    n = int(np.prod(shape))
    ref = rng.uniform(0.5, 1.0, size=n)
    if fill == "runs":
        ref[(np.arange(n) // 3333) % 3 != 0] = 0.01
    elif fill == "few":
        ref[rng.uniform(size=n) > 1e-4] = 0.01
    ref = ref.astype(np.float32).reshape(shape)
    ev = (ref + 0.01 * rng.standard_normal(shape)).astype(np.float32)
    spacing = (2.0,) * len(shape)
    pair = dict(ref=dev(ref), ev=dev(ev), spacing=spacing, dd=0.03, dta=3.0, threshold=0.1, local=False)
    want, rw = gx.gammax_batch([pair], ctx=gx.Context(0))
    ctx = gx.Context(0)
    for again in range(2):   # before and after the cell table exists
        got, rg = gx.gammax_map(pair["ref"], pair["ev"], spacing, 0.03, 3.0, 0.1, ctx=ctx)
        assert np.array_equal(host(got), host(want[0])), again
        for f in ("n_evaluated", "n_pass", "n_borderline", "n_tail", "n_guarded", "max_gamma", "search_radius"):
            assert getattr(rg, f) == getattr(rw[0], f), (again, f)
