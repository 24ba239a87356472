"""The convolutions' zero padding is multiplied like any other voxel: with
infinite and NaN weights the result is that of the volume with a border of
zeros stored around it, bit for bit (0 x Inf = NaN)."""

import numpy as np
import pytest

from gpu_common import log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ci,co", [(16, 16), (16, 32), (32, 16), (32, 32), (32, 96), (48, 16),
                                   (48, 32), (64, 32), (96, 64), (64, 128)])
@pytest.mark.parametrize("shape", [(1, 9, 12, 20), (2, 1, 3, 17), (1, 40, 16, 33)])
def test_nonfinite_weights(shape, ci, co):
    import torch
    from paper_2511_03115_amd import nn
    B, D, H, W = shape
    gen = torch.Generator(device="cuda").manual_seed(ci + co)
    x = torch.randn(shape + (ci,), generator=gen, device="cuda").bfloat16()
    w = (0.2 * torch.randn((co, 27, ci), generator=gen, device="cuda")).bfloat16()
    for k, (o, t, bad) in enumerate([(0, 0, np.nan), (1, 4, np.inf), (2, 13, -np.inf),
                                     (3, 22, np.nan), (5, 26, np.inf), (co - 1, 8, np.nan)]):
        w[o, t, (5 * k) % ci] = bad
    pad = torch.zeros((B, D + 2, H + 2, W + 2, ci), dtype=torch.bfloat16, device="cuda")
    pad[:, 1:-1, 1:-1, 1:-1] = x
    out = lambda n, d: torch.zeros(n + (co,), dtype=d, device="cuda")
    got, want = out(shape, torch.float32), out((B, D + 2, H + 2, W + 2), torch.float32)
    nn.conv3d_fwd(x, w, None, act=False, out32=got)
    nn.conv3d_fwd(pad, w, None, act=False, out32=want)
    log(f"conv padding shape={shape} ci={ci} co={co}")
    a, b = got.cpu().numpy(), want[:, 1:-1, 1:-1, 1:-1].cpu().numpy()
    assert np.isnan(a[..., 0]).all() and np.isfinite(a[..., 4]).all()
    assert np.array_equal(a, b, equal_nan=True)
