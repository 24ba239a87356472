"""The 32-channel convolution that marches along z, where its columns can go
wrong: one voxel, one plane, ragged rows and columns, groups of outputs,
batches, and the seams between columns of different length."""

import numpy as np
import pytest

from gpu_common import log
from oracle import nn_oracle as nno
from test_gpu_nn import bf16_round, to_bf16_dev

pytestmark = pytest.mark.gpu


def _data(shape, co, seed):
    rng = np.random.default_rng(seed)
    return (bf16_round(rng.normal(size=shape + (32,))),
            bf16_round(rng.normal(scale=0.2, size=(co, 27, 32))),
            rng.normal(size=co).astype(np.float32))


@pytest.mark.parametrize("shape,co", [((1, 1, 1, 1), 32), ((1, 1, 8, 16), 32), ((2, 3, 9, 17), 96),
                                      ((3, 2, 7, 5), 64), ((1, 9, 16, 33), 32),
                                      ((1, 40, 20, 36), 96)])
def test_march_against_the_oracle(shape, co):
    import torch
    from paper_2511_03115_amd import nn
    x, w, b = _data(shape, co, 7 * co + shape[1])
    log(f"march shape={shape} co={co}")
    ref = nno.conv3d(x, w, b.astype(np.float64))
    tol = 1e-5 * (nno.conv3d(np.abs(x), np.abs(w), None) + np.abs(b)) + 1e-30   # FP32 sums
    out = lambda dt: torch.full(shape + (co,), np.nan, dtype=dt, device="cuda")
    xd, wd, bd = to_bf16_dev(x), to_bf16_dev(w), torch.from_numpy(b).cuda()
    y32, both32 = out(torch.float32), out(torch.float32)
    y16, both16 = out(torch.bfloat16), out(torch.bfloat16)
    nn.conv3d_fwd(xd, wd, bd, act=False, out32=y32)
    nn.conv3d_fwd(xd, wd, bd, act=False, out16=both16, out32=both32)
    nn.conv3d_fwd(xd, wd, bd, act=False, out16=y16)
    assert np.all(np.abs(y32.cpu().numpy() - ref) <= tol)
    assert torch.equal(y32, both32) and torch.equal(y16, both16)
    assert torch.equal(y32.bfloat16(), y16)
    for alpha in (0.01, 1.5):
        nn.conv3d_fwd(xd, wd, bd, act=True, alpha=alpha, out16=y16)
        assert torch.equal(torch.where(y32 > 0, y32, alpha * y32).bfloat16(), y16)


@pytest.mark.parametrize("depth", [2, 3, 5, 17, 33])
def test_march_seams(depth):
    """Output planes away from the cut do not depend on where columns end."""
    import torch
    from paper_2511_03115_amd import nn
    x, w, b = _data((1, 40, 33, 100), 32, 5)
    xd, wd, bd = to_bf16_dev(x), to_bf16_dev(w), torch.from_numpy(b).cuda()
    whole = torch.zeros((1, 40, 33, 100, 32), dtype=torch.float32, device="cuda")
    nn.conv3d_fwd(xd, wd, bd, act=False, out32=whole)
    part = torch.zeros((1, depth, 33, 100, 32), dtype=torch.float32, device="cuda")
    nn.conv3d_fwd(xd[:, :depth].contiguous(), wd, bd, act=False, out32=part)
    log(f"march seams depth={depth}")
    assert torch.equal(whole[:, :depth - 1], part[:, :depth - 1])
