"""Weight gradients of one training step at the sizes where the bwd-weight tiles can go wrong:
a single node, ragged boxes across tile edges, and more tiles than workgroups (each workgroup
then sums several tiles into one partial).  Tolerance as the gradient parity test of the same
network: bf16 operands on both sides, so the error per layer (relative L2) stays below 2^-6
and every element below 5 % of the layer's largest gradient."""
import numpy as np
import pytest

from gpu_util import dev
from oracle import cnn
from test_gpu_cnn import _feat_tensor, _labels, _oracle_batch_grad, _random_crops, _theta

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nvol,crop", [(1, (1, 1, 1)), (2, (2, 4, 10)), (3, (5, 9, 17)), (400, (2, 2, 2))])
def test_weight_gradients_at_tile_edges(nvol, crop):
    import paper_1012_1900_amd as gx
    th = _theta(31)
    bits = _random_crops(32, nvol, crop)
    labels = _labels(33, nvol, crop)
    labels[0].flat[0] = 0.3          # at least one labelled node
    m = gx.Model(th.astype(np.float32))
    loss = m.train_step(_feat_tensor(bits), dev(labels), lr=0.0)
    got = m.grad().astype(np.float64)
    want_loss, want = _oracle_batch_grad(th, bits, labels)
    assert abs(loss - want_loss) <= 1e-3 * max(want_loss, 1e-3)
    off = 0
    for l, (ws, bs) in enumerate(cnn.layer_shapes()):
        n = int(np.prod(ws)) + bs[0]
        a, b = got[off:off + n], want[off:off + n]
        assert np.linalg.norm(a - b) <= 2.0 ** -6 * np.linalg.norm(b), l
        assert np.max(np.abs(a - b)) <= 0.05 * np.max(np.abs(b)), l
        off += n
    # two steps on the same inputs give the same bits (fixed summation order)
    m2 = gx.Model(th.astype(np.float32))
    m2.train_step(_feat_tensor(bits), dev(labels), lr=0.0)
    assert np.array_equal(m.grad(), m2.grad())
