"""The network's input features by rows, bit for bit against the formula in float32 rounded to
bfloat16: rows of one node block, of exactly one and just past one step of 256 nodes, longer
ones, more rows than the launch has waves; doses that are not finite are still refused."""
import numpy as np
import pytest
import torch

from gpu_util import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(2, 2, 2), (3, 5, 248), (3, 4, 249), (2, 3, 700), (90, 93, 5)])
def test_features_are_the_formula(shape):
    import paper_1012_1900_amd as gx
    rng = np.random.default_rng(shape[-1])
    ref = rng.uniform(0.0, 2.0, size=shape).astype(np.float32)
    ev = (ref + 0.05 * rng.standard_normal(shape)).astype(np.float32)
    got = gx.model_features(dev(ref), dev(ev), (2.5, 2.5, 2.5), 0.03).cpu()
    dmax = ref.max()
    f = np.stack([ref * (np.float32(1) / dmax), (ev - ref) * (np.float32(1) / (np.float32(0.03) * dmax))], -1)
    want = torch.zeros(tuple(n + 8 for n in shape) + (2,), dtype=torch.bfloat16)
    want[4:-4, 4:-4, 4:-4] = torch.from_numpy(f).to(torch.bfloat16)
    assert torch.equal(got.view(torch.int16), want.view(torch.int16))
    bad = ev.copy()
    bad.flat[-1] = np.nan
    with pytest.raises(gx.GammaxError, match="NaN or infinite"):
        gx.model_features(dev(ref), dev(bad), (2.5, 2.5, 2.5), 0.03)
