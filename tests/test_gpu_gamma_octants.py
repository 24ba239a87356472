"""The gamma search where each lane walks its own octant before the whole wave
takes what is left (the distance to agreement above a voxel, or few offsets per
axis), against the oracle's double-precision evaluation of the definition: pass
counts equal, exactly, from nearly all voxels passing to nearly none, with rows
that leave the octant's cell and the grid."""

import numpy as np
import pytest

import oracle
from gpu_common import log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,d,dta,interp", [
    ((14, 13, 12), (0.1, 0.1, 0.1), 0.3, 1), ((14, 13, 12), (0.1, 0.1, 0.1), 0.3, 2),
    ((9, 10, 11), (0.1, 0.15, 0.2), 0.3, 10), ((6, 7, 8), (0.2, 0.1, 0.3), 0.35, 50),
    ((14, 13, 12), (0.2, 0.2, 0.2), 0.05, 1), ((14, 13, 12), (0.2, 0.2, 0.2), 0.1, 2),
    ((14, 13, 12), (0.1, 0.1, 0.1), 0.1, 3), ((14, 13, 12), (0.1, 0.1, 0.1), 0.08, 4),
    ((3, 1, 60), (0.1, 0.1, 0.1), 0.25, 3), ((1, 1, 9), (0.1, 0.1, 0.1), 0.3, 2),
])
@pytest.mark.parametrize("local", [True, False])
def test_counts_equal(shape, d, dta, interp, local):
    import torch
    from paper_2511_03115_amd import sde
    rng = np.random.default_rng(interp * 10 + shape[0])
    ref = rng.uniform(0.2, 1.0, shape)
    for spread, dd in ((0.03, 0.02), (0.2, 0.02), (0.5, 0.003)):
        ev = ref * (1 + spread * rng.standard_normal(shape))
        _, ne, npass = oracle.gamma_pass_rate(ref, ev, d, dd, dta, 0.01, interp, local)
        r, e = torch.from_numpy(ref).cuda(), torch.from_numpy(ev).cuda()
        got = sde.gamma(r, e, d, dd, dta, 0.01, interp, local)[1:]
        log(f"gamma {shape} d={d} dta={dta} K={interp} local={local} {spread}: {(ne, npass)} {got}")
        assert got == (ne, npass)
