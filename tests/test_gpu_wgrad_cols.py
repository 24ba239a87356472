"""Weight gradients by columns against the FP64 oracle where the split can
go wrong: one voxel, one plane, one column without a partner, rows and
planes that do not fill a column, several columns per workgroup, batches,
widths that are no power of two; and the sums with and without the bias."""

import numpy as np
import pytest

from gpu_common import log
from oracle import nn_oracle as nno
from test_gpu_nn import bf16_round, to_bf16_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,ci,co", [
    ((1, 1, 1, 1), 64, 64), ((1, 1, 7, 15), 64, 48), ((1, 2, 8, 16), 64, 64),
    ((2, 3, 1, 33), 16, 80), ((3, 5, 9, 17), 96, 64), ((1, 3, 33, 5), 128, 64),
    ((2, 61, 17, 40), 16, 16), ((1, 161, 16, 33), 16, 16), ((5, 13, 25, 31), 16, 32),
    ((1, 70, 8, 50), 32, 32), ((2, 19, 24, 40), 64, 128), ((7, 4, 20, 20), 48, 64)])
def test_wgrad_by_columns(shape, ci, co):
    import torch
    from paper_2511_03115_amd import nn
    rng = np.random.default_rng(ci * 131 + co + shape[1])
    x = bf16_round(rng.normal(size=shape + (ci,)))
    dz = bf16_round(rng.normal(size=shape + (co,)))
    log(f"wgrad columns shape={shape} ci={ci} co={co}")
    _, dw_ref, db_ref = nno.conv3d_backward(dz, x, np.zeros((co, 27, ci)))
    xd, zd = to_bf16_dev(x), to_bf16_dev(dz)
    dw = torch.full((co, 27, ci), np.nan, dtype=torch.float32, device="cuda")
    db = torch.full((co,), np.nan, dtype=torch.float32, device="cuda")
    nn.conv3d_wgrad(zd, xd, dw, db)
    # FP32 accumulation of n products: far within 1e-5 of the largest sum,
    # as for every other split of these sums
    for name, got, ref in (("dw", dw, dw_ref), ("db", db, db_ref)):
        e = np.abs(got.cpu().numpy() - ref).max() / np.abs(ref).max()
        log(f"  {name} rel err {e:.3e}")
        assert e <= 1e-5, name
    dw2 = torch.full_like(dw, np.nan)
    nn.conv3d_wgrad(zd, xd, dw2)
    assert torch.equal(dw, dw2)
