"""The tile shapes that the U-Net's convolutions and weight gradients take.

Which tile a layer runs with depends on how many there are: a large batch walks
several tiles a block with up to 64 output channels, one sample alone takes
smaller ones.  A batch therefore has to give, sample by sample, what each
sample gives alone: the output within the per-element bar of the comparison
with the oracle (8 bfloat16 steps of the element plus the RMS), the parameter
gradients, which are sums over samples, within its relative L2 error of 2e-2."""
import numpy as np
import pytest

from gpu_util import UNET_STEPS, unet_params
from oracle import unet as ou

pytestmark = pytest.mark.gpu


def run(u, torch, x, gout):
    u.input().copy_(torch.from_numpy(x).to(torch.bfloat16).to(u.dev))
    u.pic_unet_forward()
    out = u.output().cpu().numpy().astype(np.float64)
    u.grad_output().copy_(torch.from_numpy(gout).to(u.dev))
    u.pic_unet_backward()
    return out, u.grads.cpu().numpy().astype(np.float64)


# the largest tiles, and ragged ones at every level (232 x 184, 116 x 92, 58 x 46, 29 x 23)
@pytest.mark.parametrize("B,H,W", [(4, 1024, 512), (6, 232, 184)])
def test_batch_equals_its_samples_alone(B, H, W):
    import torch

    from paper_1610_03918_amd.unet import UNet
    shapes = ou.conv_shapes()
    ps = unet_params(31, shapes)
    flat = np.concatenate([p.reshape(-1) for p in ps]).astype(np.float32)
    r = np.random.default_rng(32)
    x = r.standard_normal((B, H, W, 3)).astype(np.float32)
    gout = r.standard_normal((B, H, W)).astype(np.float32)
    u = UNet(B, H, W, params=flat)
    out, grads = run(u, torch, x, gout)
    u.close()
    one = UNet(1, H, W, params=flat)
    total = np.zeros_like(grads)
    for b in range(B):
        o, g = run(one, torch, x[b:b + 1], gout[b:b + 1])
        rms = float(np.sqrt(np.mean(o * o)))
        assert np.all(np.abs(out[b:b + 1] - o) <= UNET_STEPS * 2.0 ** -8 * (np.abs(o) + rms)), b
        total += g
    one.close()
    assert np.isfinite(grads).all() and np.abs(grads).max() > 0
    off = 0
    for k, p in enumerate(ps):
        a, c = grads[off:off + p.size], total[off:off + p.size]
        off += p.size
        assert np.linalg.norm(a - c) <= 2e-2 * np.linalg.norm(c), k
