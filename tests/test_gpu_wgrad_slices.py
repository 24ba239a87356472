"""Weight gradients from 64-voxel slices, which widths beside the powers of two
take on volumes that columns hardly cover, against the FP64 oracle: one voxel,
ragged slices and chunks, batches, many and few tap groups."""

import numpy as np
import pytest

from gpu_common import log
from oracle import nn_oracle as nno
from test_gpu_nn import bf16_round, to_bf16_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,ci,co", [
    ((2, 300, 1, 1), 16, 192), ((9, 50, 2, 4), 128, 96), ((16, 130, 1, 4), 32, 48),
    ((1, 300, 7, 1), 16, 96), ((3, 65, 2, 2), 64, 48), ((7, 33, 3, 1), 96, 96)])
def test_wgrad_from_slices(shape, ci, co):
    import torch
    from paper_2511_03115_amd import nn
    rng = np.random.default_rng(ci * 131 + co + shape[1])
    x = bf16_round(rng.normal(size=shape + (ci,)))
    dz = bf16_round(rng.normal(size=shape + (co,)))
    log(f"wgrad slices shape={shape} ci={ci} co={co}")
    _, dw_ref, db_ref = nno.conv3d_backward(dz, x, np.zeros((co, 27, ci)), need_dx=False)
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
