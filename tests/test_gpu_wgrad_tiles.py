"""Weight gradients at the edges of the kernel's bricks (32 x 4 x 2 voxels) against the oracle.

Grids whose rows are shorter than a brick, end inside one, or are of odd length at quarter resolution, and
enough bricks that a block takes several.  The oracle runs with the network's own BF16 roundings; what is left
is the order of FP32 sums and the activations that this order puts on the other side of a rounding,
2^-8 of an element each and spread by the later layers: 2e-2 (five of them at most) of the
largest gradient of a layer.
"""
import numpy as np
import pytest

from oracle import nn
from tests.test_gpu_nn import flat, make_params, rounded, unflat

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(4, 4, 4), (4, 8, 12), (8, 4, 36), (12, 20, 28), (4, 12, 68), (16, 36, 32)])
def test_weight_gradients(shape):
    import torch

    import paper_1704_08521_amd as lk
    D, H, W = shape
    print(f"[case] {shape}", flush=True)
    p = make_params(21)
    net = lk.Net()
    net.set_params(flat(p))
    rng = np.random.default_rng(22)
    x, t = rng.standard_normal((D, H, W, 4)), rng.standard_normal((D, H, W))
    _, g = net.step(torch.from_numpy(x.astype(np.float32)).cuda(), torch.from_numpy(t.astype(np.float32)).cuda(),
                    grads=True)
    ref = nn.loss_and_grad(rounded(p), nn.bf16(x), t[..., None], q=nn.bf16)[1]
    got = unflat(g.astype(np.float64))
    for name, *_ in nn.LAYERS:
        for key in (name + ".w", name + ".b"):
            err = np.max(np.abs(np.ravel(got[key]) - np.ravel(ref[key]))) / max(np.max(np.abs(ref[key])), 1e-300)
            assert err < 2e-2, (key, err)
