"""Grids that the gamma index takes in several passes (sde_gamma_noalloc: 2^20
voxels each) against the oracle's evaluation of the definition: voxels on both
sides of the cuts, more voxels to search than a pass's list could hold with the
others', and passes with none."""

import numpy as np
import pytest

import oracle
from gpu_common import log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(17, 256, 257), (3, 700, 1501)])
@pytest.mark.parametrize("hard", ["some", "around the cuts", "one pass"])
def test_counts_equal(shape, hard):
    import torch
    from paper_2511_03115_amd import sde
    n, cap = int(np.prod(shape)), 1 << 20
    assert n > cap
    rng = np.random.default_rng(shape[0])
    # flat in every plane: an altered voxel is all that has to be searched
    ref = np.ones(shape) + 0.2 * np.arange(shape[0])[:, None, None]
    ev, f = ref.copy(), rng.uniform(0.9, 1.1, n)
    if hard == "some":
        at = rng.choice(n, 40000, replace=False)
    elif hard == "around the cuts":
        cuts = np.arange(cap, n, cap)
        at = np.unique((cuts[:, None] + np.arange(-700, 700)[None]).ravel())
        at = at[at < n]
    else:
        at = np.arange(cap, min(n, cap + 30000))
    ev.ravel()[at] *= f[at]
    d = (0.1, 0.1, 0.1)
    r, e = torch.from_numpy(ref).cuda(), torch.from_numpy(ev).cuda()
    for local in (True, False):
        _, ne, npass = oracle.gamma_pass_rate(ref, ev, d, 0.02, 0.06, 0.01, 5, local)
        got = sde.gamma_noalloc(r, e, d, 0.02, 0.06, 0.01, 5, local)[1:]
        log(f"gamma passes {shape} {hard} local={local}: {(ne, npass)} {got}")
        assert got == (ne, npass) and 0 < npass < ne
