"""The tile shapes of the U-Net's kernels, to the bit.

Every output of a convolution adds its products in the order (chunk of 32
input channels, tap) whatever tile it is computed in, so a sample gives the
same output in a batch and alone.  The parameter gradients are sums over
pixels whose float32 partial sums are cut differently: at most some 2^13
additions of either sign each, and a float64 sum of the partials; their
rounding stays below 2^-24 sqrt(2^13), 5e-6, of the sum's norm."""
import numpy as np
import pytest

from gpu_util import unet_params
from oracle import unet as ou

pytestmark = pytest.mark.gpu


def run(u, torch, x, gout):
    u.input().copy_(torch.from_numpy(x).to(torch.bfloat16).to(u.dev))
    u.pic_unet_forward()
    out = u.output().cpu().numpy()
    u.grad_output().copy_(torch.from_numpy(gout).to(u.dev))
    u.pic_unet_backward()
    return out, u.grads.cpu().numpy().astype(np.float64)


# the largest tiles; ragged ones at every level (232 x 184, 116 x 92, 58 x 46, 29 x 23); the smallest images, whose
# patches reach across both edges at once
@pytest.mark.parametrize("wrap", [False, True])
@pytest.mark.parametrize("B,H,W", [(4, 1024, 512), (6, 232, 184), (16, 96, 56), (64, 16, 8)])
def test_a_sample_is_the_same_in_a_batch_and_alone(B, H, W, wrap):
    import torch

    from paper_1610_03918_amd.unet import UNet
    ps = unet_params(33, ou.conv_shapes())
    flat = np.concatenate([p.reshape(-1) for p in ps]).astype(np.float32)
    r = np.random.default_rng(34)
    x = r.standard_normal((B, H, W, 3)).astype(np.float32)
    gout = r.standard_normal((B, H, W)).astype(np.float32)
    u = UNet(B, H, W, params=flat, periodic_w=wrap)
    out, grads = run(u, torch, x, gout)
    u.close()
    one = UNet(1, H, W, params=flat, periodic_w=wrap)
    total = np.zeros_like(grads)
    for b in range(B):
        o, g = run(one, torch, x[b:b + 1], gout[b:b + 1])
        assert np.array_equal(out[b:b + 1], o), b
        total += g
    one.close()
    assert np.isfinite(grads).all() and np.abs(grads).max() > 0
    off = 0
    for k, p in enumerate(ps):
        a, c = grads[off:off + p.size], total[off:off + p.size]
        off += p.size
        assert np.linalg.norm(a - c) <= 1e-5 * np.linalg.norm(c), k
