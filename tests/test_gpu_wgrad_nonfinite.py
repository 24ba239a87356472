"""Weight gradients of inputs and output gradients with infinite and NaN voxels:
finite, infinite and NaN where the definition's sums are, also beside the planes
and rows where the volume is cut into columns."""

import numpy as np
import pytest

from gpu_common import log
from oracle import nn_oracle as nno
from test_gpu_nn import bf16_round, to_bf16_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,ci,co", [((1, 12, 17, 20), 64, 48), ((2, 40, 24, 33), 32, 64),
                                         ((1, 3, 9, 5), 16, 64), ((3, 36, 20, 40), 16, 16)])
@pytest.mark.parametrize("where", ["x", "dz", "both"])
def test_nonfinite(shape, ci, co, where):
    import torch
    from paper_2511_03115_amd import nn
    rng = np.random.default_rng(ci + co + len(where))
    x = bf16_round(rng.normal(size=shape + (ci,)))
    dz = bf16_round(rng.normal(size=shape + (co,)))
    D, H, W = shape[1:]
    if where != "dz":       # a channel each: first and last plane, rows of a cut, anywhere
        x[0, 0, H // 2, W // 2, 0] = np.inf
        x[-1, D - 1, 0, 0, 1] = np.nan
        x[0, D // 2, min(7, H - 1), min(15, W - 1), 2] = -np.inf
        x[0, D // 2, min(8, H - 1), min(16, W - 1), 3] = np.inf
        for c in range(4, 12):
            x[tuple(rng.integers(0, n) for n in shape) + (c,)] = rng.choice([np.inf, -np.inf, np.nan])
    if where != "x":
        dz[0, D - 1, H - 1, W - 1, 0] = np.inf
        dz[0, D // 3, H // 2, 0, 1] = np.nan
    log(f"wgrad non-finite {where} shape={shape} ci={ci} co={co}")
    with np.errstate(invalid="ignore"):
        _, ref, db_ref = nno.conv3d_backward(dz, x, np.zeros((co, 27, ci)), need_dx=False)
    dw = torch.zeros((co, 27, ci), dtype=torch.float32, device="cuda")
    db = torch.zeros(co, dtype=torch.float32, device="cuda")
    nn.conv3d_wgrad(to_bf16_dev(dz), to_bf16_dev(x), dw, db)
    got, fin = dw.cpu().numpy(), np.isfinite(ref)
    assert fin.any() and not fin.all()
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    assert np.array_equal(got[np.isinf(ref)], ref[np.isinf(ref)])
    # FP32 sums of n products, as without the special values
    assert np.abs(got[fin] - ref[fin]).max() <= 1e-5 * np.abs(ref[fin]).max()
    assert np.array_equal(np.isnan(db.cpu().numpy()), np.isnan(db_ref))
