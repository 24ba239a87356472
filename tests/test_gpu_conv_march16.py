"""The 16 -> 16 convolution by columns (2M voxels and more) against the one by
bricks, which smaller volumes take: a large batch of small volumes equals
the volumes one by one, bit for bit, with every output the network uses."""

import numpy as np
import pytest

from gpu_common import log
from oracle import nn_oracle as nno
from test_gpu_nn import _net_inputs, he_params

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,D,H,W", [(65, 20, 33, 50), (1100, 3, 20, 33), (3000, 1, 27, 27)])
def test_batch_equals_its_volumes(B, D, H, W):
    import torch
    from paper_2511_03115_amd import nn
    assert B * D * H * W >= 1 << 21
    log(f"march16 batch {(B, D, H, W)}")
    gen = torch.Generator(device="cuda").manual_seed(D)
    x = torch.randn((B, D, H, W, 16), generator=gen, device="cuda").bfloat16()
    w = (0.1 * torch.randn((16, 27, 16), generator=gen, device="cuda")).bfloat16()
    b = torch.randn(16, generator=gen, device="cuda")
    empty = lambda n, dt: torch.full((n, D, H, W, 16), float("nan"), dtype=dt, device="cuda")
    y16, y32 = empty(B, torch.bfloat16), empty(B, torch.float32)
    only = empty(B, torch.bfloat16)
    nn.conv3d_fwd(x, w, b, act=True, alpha=0.1, out16=y16, out32=y32)
    nn.conv3d_fwd(x, w, b, act=True, alpha=0.1, out16=only)
    assert torch.equal(y16, only)
    dx, one = empty(B, torch.float32), empty(1, torch.float32)
    nn.conv3d_dgrad(x, w, dx)
    for k in (0, 1, B // 2, B - 1):
        s16, s32 = empty(1, torch.bfloat16), empty(1, torch.float32)
        nn.conv3d_fwd(x[k:k + 1], w, b, act=True, alpha=0.1, out16=s16, out32=s32)
        nn.conv3d_dgrad(x[k:k + 1], w, one)
        assert torch.equal(y16[k:k + 1], s16) and torch.equal(y32[k:k + 1], s32)
        assert torch.equal(dx[k:k + 1], one)


@pytest.mark.parametrize("levels,D,H,W", [(2, 16, 64, 64), (3, 20, 52, 64)])
def test_network_on_32_copies(levels, D, H, W):
    """32 copies of a volume: the same outputs as the volume alone; the loss
    gradient's terms are scaled by a power of two, so only the order of the
    FP32 weight-gradient sums differs."""
    import torch
    from paper_2511_03115_amd import nn
    B = 32
    assert B * D * H * W >= 1 << 21
    log(f"march16 network levels={levels} {(B, D, H, W)}")
    flat = nno.flatten(he_params(levels, 16, 16, seed=9), levels, 16, 16).astype(np.float32)
    one = _net_inputs(1, D, H, W, seed=8)
    outs, grads = [], []
    for n in (1, B):
        net = nn.Net(levels, 16, 16, 0.01, max_batch=n, max_dims=(D, H, W), train=True)
        net.set_params(flat)
        dev = [torch.from_numpy(np.repeat(a, n, axis=0)).cuda() for a in one]
        out = torch.zeros((n, D, H, W), dtype=torch.float32, device="cuda")
        net.forward(dev[0], dev[1], out)
        outs.append(out)
        net.loss_grad(*dev)
        grads.append(np.array(net.get_grads(), dtype=np.float64))
        net.close()
    for k in range(B):
        assert torch.equal(outs[1][k], outs[0][0])
    e = np.abs(grads[1] - grads[0]).max() / np.abs(grads[0]).max()
    log(f"  gradient rel diff {e:.2e}")
    assert np.abs(grads[0]).max() > 0 and e <= 1e-5
