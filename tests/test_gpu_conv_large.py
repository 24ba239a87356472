"""Operands of 2 GiB and more, past the 32-bit offsets of the columns, blocks and
bricks: two volumes in one call against each of them alone, which those take."""

import pytest

from gpu_common import log

pytestmark = pytest.mark.gpu


def _tensors(vol, ci, co):
    import torch
    gen = torch.Generator(device="cuda").manual_seed(ci + co)
    x = torch.empty((2,) + vol + (ci,), dtype=torch.bfloat16, device="cuda")
    dz = torch.empty((2,) + vol + (co,), dtype=torch.bfloat16, device="cuda")
    for b in range(2):
        x[b] = torch.randn(vol + (ci,), generator=gen, device="cuda")
        dz[b] = torch.randn(vol + (co,), generator=gen, device="cuda")
    w = (0.2 * torch.randn((co, 27, ci), generator=gen, device="cuda")).bfloat16()
    assert x.numel() * 2 > 2 ** 31 and x.numel() < 2 ** 31 and dz.numel() < 2 ** 31
    return x, w, torch.randn(co, generator=gen, device="cuda"), dz


@pytest.mark.parametrize("vol,ci,co", [((131, 257, 260), 64, 32), ((90, 250, 250), 96, 64),
                                       ((131, 513, 260), 32, 32), ((131, 513, 513), 16, 16)])
def test_forward(vol, ci, co):
    import torch
    from paper_2511_03115_amd import nn
    log(f"large conv {vol} {ci} -> {co}")
    x, w, b, _ = _tensors(vol, ci, co)
    y = torch.full((2,) + vol + (co,), float("nan"), dtype=torch.float32, device="cuda")
    nn.conv3d_fwd(x, w, b, act=False, out32=y)
    one, size = torch.empty_like(y[:1]), torch.empty_like(y[:1])
    for k in range(2):
        nn.conv3d_fwd(x[k:k + 1], w, b, act=False, out32=one)
        nn.conv3d_fwd(x[k:k + 1].abs(), w.abs(), b.abs(), act=False, out32=size)
        # FP32 sums of the same products, perhaps in another order
        assert bool(((y[k:k + 1] - one).abs() <= 2e-5 * size).all())


@pytest.mark.parametrize("vol,ci,co", [((131, 257, 260), 64, 32), ((131, 513, 260), 32, 48)])
def test_weight_gradient(vol, ci, co):
    import torch
    from paper_2511_03115_amd import nn
    log(f"large wgrad {vol} {ci} -> {co}")
    x, _, _, dz = _tensors(vol, ci, co)
    dw = torch.empty((3, co, 27, ci), dtype=torch.float32, device="cuda")
    db = torch.empty((3, co), dtype=torch.float32, device="cuda")
    nn.conv3d_wgrad(dz, x, dw[2], db[2])
    for k in range(2):
        nn.conv3d_wgrad(dz[k:k + 1], x[k:k + 1], dw[k], db[k])
    for g in (dw.double(), db.double()):
        # FP32 sums in chunks: far within 1e-5 of the largest, as at other sizes
        assert float((g[2] - g[0] - g[1]).abs().max() / g[2].abs().max()) <= 1e-5
