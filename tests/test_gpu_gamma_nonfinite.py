"""Evaluated maps with NaN and infinite voxels where the distance to agreement
is a voxel: the outermost offsets lie on the faces towards the next cell, whose
values hold whatever the octant's own cell does.  Pass counts equal to the
double-precision evaluation of the definition, exactly."""

import numpy as np
import pytest

import oracle
from gpu_common import log

pytestmark = pytest.mark.gpu


def _both(ref, ev, d, dta, interp, local):
    import torch
    from paper_2511_03115_amd import sde
    _, ne0, np0 = oracle.gamma_pass_rate(ref, ev, d, 0.02, dta, 0.01, interp, local)
    r, e = (torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (ref, ev))
    return (ne0, np0), sde.gamma(r, e, d, 0.02, dta, 0.01, interp, local)[1:]


@pytest.mark.parametrize("axis", [0, 1, 2])
@pytest.mark.parametrize("bad", [np.nan, np.inf, -np.inf])
def test_plateaus_a_voxel_away(axis, bad):
    """Alternating plateaus: every voxel agrees with nothing but its neighbours
    a voxel away, with non-finite voxels scattered among them."""
    rng = np.random.default_rng(17 + axis)
    shape = (14, 13, 12)
    k = np.arange(shape[axis]).reshape([-1 if a == axis else 1 for a in range(3)])
    ref = np.where(k % 2, 1.0, 5.0) * np.ones(shape)
    ev = np.where(k % 2, 5.0, 1.0) * np.ones(shape)
    n = rng.choice(ref.size, 150, replace=False)
    ev.ravel()[n] = bad
    for interp in (1, 4, 10):
        for local in (True, False):
            want, got = _both(ref, ev, (0.1, 0.1, 0.1), 0.1, interp, local)
            log(f"gamma plateaus axis={axis} bad={bad} K={interp} local={local}: {want} {got}")
            assert 0 < want[1] < want[0] and want == got
