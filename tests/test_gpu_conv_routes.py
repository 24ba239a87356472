"""A batch goes by other kernels, or in other blocks, than its volumes one by
one: the same outputs, bit for bit, and within FP32 rounding of the definition,
at sizes on both sides of the rules (volumes of few rows, few planes, few
columns)."""

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
