"""The training kernels at batch sizes around their tiles (32 samples a
workgroup, 256 slots a loss sum, 1024 samples a gradient chunk) against the
FP64 oracle.  Tolerances as for the gradients elsewhere: loss 2%, gradient
blocks 5% in norm (five BF16 products of 2^-9 each on inputs and weights)."""
import numpy as np
import pytest

from oracle import learned as ol
from test_gpu_learned import _net, _records

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 31, 257, 1300, 3073])
def test_train_sizes(n):
    import torch
    import paper_2204_10871_amd as irs
    fr, th = _net(seed=6)
    rec = _records(np.random.default_rng(n), n)
    loss, g = irs.mlp_loss_grad(fr, th, torch.tensor(rec, device="cuda:0"), n)
    lo, go = ol.loss_and_grad(th.astype(np.float64), fr.astype(np.float64),
                              rec[0:2].T.astype(np.float64),
                              (rec[2:18:2] + 1j * rec[3:18:2]).T.astype(np.complex128),
                              (rec[18] + 1j * rec[19]).astype(np.complex128))
    assert abs(loss - lo) <= 0.02 * lo
    off = 0
    for shp in ol._SHAPES:
        m = int(np.prod(shp))
        a, b = g[off:off + m].astype(np.float64), go[off:off + m]
        assert np.linalg.norm(a - b) < 0.05 * np.linalg.norm(b)
        off += m
