"""The convolutions of 16 and 32 channels that march along z, and that of more in
passes over blocks of planes, where they can go wrong: one voxel, one plane,
ragged rows, columns and blocks, groups of outputs, batches, and the seams
between columns and blocks of different length."""

import numpy as np
import pytest

from gpu_common import log
from oracle import nn_oracle as nno
from test_gpu_nn import bf16_round, to_bf16_dev

pytestmark = pytest.mark.gpu


def _data(shape, ci, co, seed):
    rng = np.random.default_rng(seed)
    return (bf16_round(rng.normal(size=shape + (ci,))),
            bf16_round(rng.normal(scale=0.2, size=(co, 27, ci))),
            rng.normal(size=co).astype(np.float32))


@pytest.mark.parametrize("shape,ci,co", [
    ((1, 1, 1, 1), 32, 32), ((1, 1, 8, 16), 32, 32), ((2, 3, 9, 17), 32, 96),
    ((3, 2, 7, 5), 32, 64), ((1, 9, 16, 33), 32, 32), ((1, 40, 20, 36), 32, 96),
    ((1, 5, 12, 20), 32, 128),
    # two taps per step
    ((1, 1, 1, 1), 16, 32), ((1, 1, 8, 16), 16, 32), ((2, 3, 9, 17), 16, 96),
    ((3, 2, 7, 5), 16, 64), ((1, 40, 20, 36), 16, 32),
    ((1, 5, 12, 20), 16, 128),
    # blocks of one, two and four planes
    ((1, 1, 1, 1), 64, 32), ((2, 3, 9, 17), 96, 64), ((1, 40, 16, 33), 64, 64),
    ((2, 21, 25, 36), 64, 64), ((1, 66, 17, 50), 96, 32), ((1, 5, 9, 20), 128, 128)])
def test_against_the_oracle(shape, ci, co):
    import torch
    from paper_2511_03115_amd import nn
    x, w, b = _data(shape, ci, co, 7 * co + ci + shape[1])
    log(f"conv shape={shape} ci={ci} co={co}")
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


@pytest.mark.parametrize("ci", [16, 32, 64])
@pytest.mark.parametrize("depth", [2, 3, 5, 17, 33])
def test_seams(depth, ci):
    """Output planes away from the cut do not depend on where columns and
    blocks end."""
    import torch
    from paper_2511_03115_amd import nn
    x, w, b = _data((1, 40, 33, 100), ci, 32, 5)
    xd, wd, bd = to_bf16_dev(x), to_bf16_dev(w), torch.from_numpy(b).cuda()
    whole = torch.zeros((1, 40, 33, 100, 32), dtype=torch.float32, device="cuda")
    nn.conv3d_fwd(xd, wd, bd, act=False, out32=whole)
    part = torch.zeros((1, depth, 33, 100, 32), dtype=torch.float32, device="cuda")
    nn.conv3d_fwd(xd[:, :depth].contiguous(), wd, bd, act=False, out32=part)
    log(f"seams depth={depth} ci={ci}")
    assert torch.equal(whole[:, :depth - 1], part[:, :depth - 1])


@pytest.mark.parametrize("B,D,H,W", [(1, 10, 130, 130), (1, 40, 34, 34), (3, 2, 18, 16),
                                     (1, 2, 2, 2), (2, 64, 16, 32)])
def test_level0_concatenation(B, D, H, W):
    """The level-0 decoder convolution that marches along z over the skip and
    the level below in place, against the stored concatenation's: equal bit
    for bit, over columns of several lengths."""
    import torch
    from paper_2511_03115_amd import nn
    from test_gpu_nn import _net_inputs, he_params
    flat = nno.flatten(he_params(2, 16, 16, seed=3), 2, 16, 16).astype(np.float32)
    dose, rho, _, _ = _net_inputs(B, D, H, W, seed=4)
    log(f"level-0 concatenation {(B, D, H, W)}")
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


@pytest.mark.parametrize("ci,co", [(16, 32), (32, 32), (64, 64)])
def test_fp32_output_at_any_float(ci, co):
    """FP32 outputs and biases need no more than a float's alignment, and
    nothing is written beside them."""
    import torch
    from paper_2511_03115_amd import nn
    shape = (1, 9, 12, 20)
    x, w, b = _data(shape, ci, co, 6)
    xd, wd = to_bf16_dev(x), to_bf16_dev(w)
    bd = torch.from_numpy(np.concatenate([[0.0], b]).astype(np.float32)).cuda()[1:]
    n = int(np.prod(shape)) * co
    want = torch.zeros(shape + (co,), dtype=torch.float32, device="cuda")
    nn.conv3d_fwd(xd, wd, bd, act=False, out32=want)
    for off in (1, 2, 3):
        log(f"unaligned output ci={ci} co={co} off={off}")
        flat = torch.zeros(n + 8, dtype=torch.float32, device="cuda")
        nn.conv3d_fwd(xd, wd, bd, act=False, out32=flat[off:off + n].view(shape + (co,)))
        assert torch.equal(flat[off:off + n].view(shape + (co,)), want)
        assert not flat[:off].any() and not flat[off + n:].any()
