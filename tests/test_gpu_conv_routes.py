"""A batch goes by other kernels, or in other blocks, than its volumes one by
one: the same outputs, bit for bit, and within FP32 rounding of the definition,
at sizes on both sides of the rules (volumes of few rows, few planes, few
columns).  16 -> 16 by columns needs 2M voxels: there a batch of small
volumes against the volumes by bricks, with every output the network uses."""

import numpy as np
import pytest

from gpu_common import log
from oracle import nn_oracle as nno
from test_gpu_nn import bf16_round, to_bf16_dev

pytestmark = pytest.mark.gpu


def _batch_equals_volumes(shape, ci, co):
    import torch
    from paper_2511_03115_amd import nn
    B = shape[0]
    log(f"conv routes shape={shape} ci={ci} co={co}")
    rng = np.random.default_rng(ci + co + shape[1])
    x = bf16_round(rng.normal(size=shape + (ci,)))
    w = bf16_round(rng.normal(scale=0.2, size=(co, 27, ci)))
    b = rng.normal(size=co).astype(np.float32)
    xd, wd, bd = to_bf16_dev(x), to_bf16_dev(w), torch.from_numpy(b).cuda()
    out = lambda n, dt: torch.full((n,) + shape[1:] + (co,), np.nan, dtype=dt, device="cuda")
    y16, y32, only = out(B, torch.bfloat16), out(B, torch.float32), out(B, torch.bfloat16)
    nn.conv3d_fwd(xd, wd, bd, act=True, alpha=0.1, out16=y16, out32=y32)
    nn.conv3d_fwd(xd, wd, bd, act=True, alpha=0.1, out16=only)
    assert torch.equal(y16, only) and torch.equal(y32.bfloat16(), y16)
    s16, s32 = out(1, torch.bfloat16), out(1, torch.float32)
    for k in (0, B // 2, B - 1):
        nn.conv3d_fwd(xd[k:k + 1], wd, bd, act=True, alpha=0.1, out16=s16, out32=s32)
        assert torch.equal(y16[k:k + 1], s16) and torch.equal(y32[k:k + 1], s32)
    k = B - 1
    ref = nno.conv3d(x[k:k + 1], w, b.astype(np.float64))
    tol = 1e-5 * (nno.conv3d(np.abs(x[k:k + 1]), np.abs(w), None) + np.abs(b)) + 1e-30   # FP32 sums
    ref = np.where(ref > 0, ref, 0.1 * ref)
    assert np.all(np.abs(s32.cpu().numpy() - ref) <= tol)


@pytest.mark.parametrize("shape,ci,co", [
    ((9, 30, 3, 33), 64, 64), ((40, 1, 17, 9), 96, 64), ((64, 4, 4, 4), 128, 128),
    ((30, 2, 9, 17), 64, 96), ((5, 60, 12, 10), 64, 32), ((3, 40, 1, 70), 96, 192),
    ((7, 33, 2, 18), 192, 64), ((17, 8, 8, 8), 64, 192)])
def test_wide_inputs(shape, ci, co):
    _batch_equals_volumes(shape, ci, co)


@pytest.mark.parametrize("shape,ci,co", [
    ((9, 30, 3, 33), 32, 32), ((12, 20, 4, 50), 32, 96), ((5, 200, 9, 3), 32, 64),
    ((9, 240, 10, 3), 32, 128), ((7, 20, 20, 19), 32, 32),
    ((9, 30, 3, 33), 16, 32), ((12, 20, 4, 50), 16, 96), ((5, 200, 9, 3), 16, 64),
    ((9, 240, 10, 2), 16, 128), ((7, 20, 20, 19), 16, 64)])
def test_few_inputs(shape, ci, co):
    _batch_equals_volumes(shape, ci, co)


@pytest.mark.parametrize("B,D,H,W,co", [(65, 21, 45, 47, 16), (160, 9, 31, 49, 16),
                                        (22, 21, 46, 47, 48), (25, 90, 20, 8, 48)])
def test_sixteen_inputs(B, D, H, W, co):
    import torch
    from paper_2511_03115_amd import nn
    assert B * D * H * W * (co // 16) >= 1 << 20
    log(f"conv routes 16 -> {co} {(B, D, H, W)}")
    gen = torch.Generator(device="cuda").manual_seed(D)
    x = torch.randn((B, D, H, W, 16), generator=gen, device="cuda").bfloat16()
    w = (0.1 * torch.randn((co, 27, 16), generator=gen, device="cuda")).bfloat16()
    b = torch.randn(co, generator=gen, device="cuda")
    empty = lambda n, dt: torch.full((n, D, H, W, co), float("nan"), dtype=dt, device="cuda")
    y16, y32, only = empty(B, torch.bfloat16), empty(B, torch.float32), empty(B, torch.bfloat16)
    nn.conv3d_fwd(x, w, b, act=True, alpha=0.1, out16=y16, out32=y32)
    nn.conv3d_fwd(x, w, b, act=True, alpha=0.1, out16=only)
    assert torch.equal(y16, only)
    for k in (0, 1, B // 2, B - 1):
        s16, s32 = empty(1, torch.bfloat16), empty(1, torch.float32)
        nn.conv3d_fwd(x[k:k + 1], w, b, act=True, alpha=0.1, out16=s16, out32=s32)
        assert torch.equal(y16[k:k + 1], s16) and torch.equal(y32[k:k + 1], s32)


@pytest.mark.parametrize("B,D,H,W", [(40, 22, 46, 62), (34, 30, 46, 46)])
def test_network_on_copies(B, D, H, W):
    """Copies of a volume: the same outputs as the volume alone, and its
    gradient up to the order of the FP32 sums."""
    import torch
    from paper_2511_03115_amd import nn
    from test_gpu_nn import _net_inputs, he_params
    log(f"conv routes network {(B, D, H, W)}")
    flat = nno.flatten(he_params(2, 16, 16, seed=9), 2, 16, 16).astype(np.float32)
    one = _net_inputs(1, D, H, W, seed=8)
    outs, grads = [], []
    for n in (1, B):
        net = nn.Net(2, 16, 16, 0.01, max_batch=n, max_dims=(D, H, W), train=True)
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
    # 1 / B in the loss is no power of two: the bf16 layer gradients round
    # differently, to 2^-9 each; their sums over B D H W voxels stay within that
    e = np.abs(grads[1] - grads[0]).max() / np.abs(grads[0]).max()
    log(f"  gradient rel diff {e:.2e}")
    assert e <= 2.0 ** -8


@pytest.mark.parametrize("B,D,H,W", [(1, 24, 258, 262), (8, 14, 90, 92), (1, 200, 72, 72),
                                     (1, 96, 130, 120), (2, 20, 8, 66), (1, 30, 82, 80)])
def test_concatenation(B, D, H, W):
    """The level-0 decoder convolution over the skip and the level below in
    place, in long and in short columns and by bricks, against the stored
    concatenation's: equal bit for bit."""
    import torch
    from paper_2511_03115_amd import nn
    from test_gpu_nn import _net_inputs, he_params
    log(f"conv routes concatenation {(B, D, H, W)}")
    flat = nno.flatten(he_params(2, 16, 16, seed=3), 2, 16, 16).astype(np.float32)
    dose, rho, _, _ = _net_inputs(B, D, H, W, seed=4)
    outs = []
    for stored in (False, True):
        net = nn.Net(2, 16, 16, 0.01, max_batch=B, max_dims=(D, H, W), train=False,
                     store_concat=stored)
        net.set_params(flat)
        out = torch.zeros((B, D, H, W), dtype=torch.float32, device="cuda")
        net.forward(torch.from_numpy(dose).cuda(), torch.from_numpy(rho).cuda(), out)
        outs.append(out.cpu().numpy())
        net.close()
    assert np.isfinite(outs[0]).all() and np.array_equal(*outs)


@pytest.mark.parametrize("levels,B,D,H,W", [(3, 2, 80, 8, 24), (4, 1, 16, 16, 104), (3, 5, 24, 16, 8)])
def test_training_of_few_rows(levels, B, D, H, W):
    """Networks whose lower levels have one to four rows: with the decoder's
    concatenations read in place and stored, equal bit for bit in outputs, loss and
    gradients."""
    import torch
    from paper_2511_03115_amd import nn
    from test_gpu_nn import _net_inputs, he_params
    log(f"conv routes training levels={levels} {(B, D, H, W)}")
    flat = nno.flatten(he_params(levels, 16, 16, seed=5), levels, 16, 16).astype(np.float32)
    dev = [torch.from_numpy(a).cuda() for a in _net_inputs(B, D, H, W, seed=6)]
    got = []
    for stored in (False, True):
        net = nn.Net(levels, 16, 16, 0.01, max_batch=B, max_dims=(D, H, W), train=True,
                     store_concat=stored)
        net.set_params(flat)
        out = torch.zeros((B, D, H, W), dtype=torch.float32, device="cuda")
        net.forward(dev[0], dev[1], out)
        loss = net.loss_grad(*dev)
        got.append((out.cpu().numpy(), loss, net.get_grads().copy()))
        net.close()
    (o0, l0, g0), (o1, l1, g1) = got
    assert np.isfinite(o0).all() and np.abs(g0).max() > 0
    assert np.array_equal(o0, o1) and l0 == l1 and np.array_equal(g0, g1)
