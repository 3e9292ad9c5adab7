"""The cell ranges of long tails are only an accelerator (8 bytes per grid node, kept by the context): calls
whose walk cannot read them do not allocate them, and a map that cannot have them runs without."""
import numpy as np
import pytest

from gpu_util import dev, host

pytestmark = pytest.mark.gpu
RANGE_BYTES = 8


def _walking_pair(shape, seed=1):
    """Every node walks, and visits many more than two cells: the ranges are wanted from the second map on."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    ref = torch.full(shape, 0.75, dtype=torch.float32, device="cuda")
    ev = ref + 0.04 + 0.004 * torch.randn(shape, generator=g, device="cuda")
    return ref, ev


def _wanted(r, n):
    return r.n_tail >= 16384 and r.n_cells - 8 * r.n_evaluated >= 2 * n


@pytest.mark.parametrize("opt", [dict(tail_lanes=16), dict(tail_lanes=1), "batch", dict()],
                         ids=["16 lanes", "one lane", "batch", "automatic"])
def test_only_calls_that_read_them_allocate_them(opt):
    import torch

    import paper_1012_1900_amd as gx
    shape = (160, 224, 224)   # 64 MB of ranges
    ref, ev = _walking_pair(shape)
    ctx = gx.Context(0)

    def run():
        if opt == "batch":
            gs, rs = gx.gammax_batch([dict(ref=ref, ev=ev, spacing=(1.5,) * 3, dd=0.03, dta=3.0, threshold=0.0)], ctx=ctx)
            return gs[0], rs[0]
        return gx.gammax_map(ref, ev, (1.5,) * 3, 0.03, 3.0, 0.0, ctx=ctx, **opt)

    first, r = run()
    assert _wanted(r, ref.numel())
    torch.cuda.synchronize()
    torch.cuda.empty_cache()   # (what torch keeps for itself is not counted, before or after)
    before = torch.cuda.mem_get_info()[0]
    for _ in range(2):
        got, r2 = run()
        assert np.array_equal(host(got), host(first)) and r2.n_cells == r.n_cells
        got = None
    torch.cuda.empty_cache()
    took = before - torch.cuda.mem_get_info()[0]
    if opt == {}:
        assert took >= RANGE_BYTES * ref.numel() // 2
    else:
        assert took < RANGE_BYTES * ref.numel() // 2


def test_map_without_memory_for_the_ranges():
    """The second map of a pair wants 1 GB of ranges where less is free: it runs without them, as do
    later ones."""
    import torch

    import paper_1012_1900_amd as gx
    shape = (512, 512, 512)
    n = 512 ** 3
    ref, ev = _walking_pair(shape)
    out = torch.empty_like(ref)
    ctx = gx.Context(0)
    a = (ref, ev, (1.5,) * 3, 0.03, 3.0, 0.0)
    _, r = gx.gammax_map(*a, ctx=ctx, out=out)
    assert _wanted(r, n)
    first = out.clone()
    assert torch.equal(out.zero_(), torch.zeros_like(out))   # (what the loop below uses is loaded while there is memory)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    hold, left = [], RANGE_BYTES * n * 5 // 10
    while torch.cuda.mem_get_info()[0] > left + (64 << 20):
        hold.append(torch.empty(torch.cuda.mem_get_info()[0] - left, dtype=torch.uint8, device="cuda"))
    try:
        for _ in range(2):
            out.zero_()
            _, r2 = gx.gammax_map(*a, ctx=ctx, out=out)
            assert torch.equal(out, first)
            assert (r2.n_cells, r2.n_pass, r2.n_tail) == (r.n_cells, r.n_pass, r.n_tail)
        assert torch.cuda.mem_get_info()[0] < RANGE_BYTES * n * 6 // 10   # (it stayed that way)
    finally:
        hold.clear()
        torch.cuda.empty_cache()
