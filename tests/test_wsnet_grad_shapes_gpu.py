"""Weight gradients of the warm-start network at the edges of the position
chunks (128) and of the partial groups (128 and 256), against the FP64 oracle
with the BF16 bars of test_wsnet_gpu.py (5e-2, cosine 0.998)."""
import numpy as np
import pytest

import oracle.wsnet as NET
from tests.gpu_util import rel, say
from tests.test_wsnet_gpu import _batch, _cos, _net

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,m", [(1, 3), (2, 40), (1, 128), (2, 129), (1, 257), (129, 96),
                                 (87, 260)])
def test_gradient_chunk_edges(lib, B, m):
    import torch
    say(f"case: wsnet gradient chunk edges B={B} m={m}")
    net = _net(lib, seed=7)
    feat, target, xb, tb = _batch(B, m, 8)
    loss, grad = net.loss_grad(feat, target)
    torch.cuda.synchronize()
    params = lib.wsnet_unpack(net.params.cpu().numpy())
    out, acts = NET.forward(params, xb)
    lref, gout = NET.mse_loss(out, tb)
    assert abs(loss.item() - lref) <= 3e-2 * lref
    gref = NET.backward(params, acts, gout)
    for (gw, gb), (rw, rb) in zip(lib.wsnet_unpack(grad.cpu().numpy()), gref):
        assert rel(gw, rw) <= 5e-2 and _cos(gw, rw) >= 0.998
        assert rel(gb, rb) <= 5e-2
