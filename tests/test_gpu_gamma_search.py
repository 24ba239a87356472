"""The gamma search's octant and row bounds against the oracle's
double-precision evaluation of the definition: pass counts equal, exactly,
where the bounds could go wrong (the distance to agreement equal to a voxel
on some axes, lattices of one and of many offsets, grid faces, planes and
lines, doses spanning twelve decades with no threshold, steep and flat
neighbours, infinities and NaN beside ordinary voxels)."""

import numpy as np
import pytest

import oracle
from gpu_common import log

pytestmark = pytest.mark.gpu


def _both(ref, ev, d, dd, dta, thr, interp, local):
    import torch
    from paper_2511_03115_amd import sde
    _, ne0, np0 = oracle.gamma_pass_rate(ref, ev, d, dd, dta, thr, interp, local)
    r, e = (torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (ref, ev))
    a = sde.gamma(r, e, d, dd, dta, thr, interp, local)[1:]
    b = sde.gamma_noalloc(r, e, d, dd, dta, thr, interp, local)[1:]
    assert a == b
    return (ne0, np0), a


@pytest.mark.parametrize("local", [True, False])
@pytest.mark.parametrize("shape,d,dta,interp", [
    ((17, 15, 13), (0.1, 0.1, 0.1), 0.1, 10),     # dta equal to a voxel on every axis
    ((17, 15, 13), (0.1, 0.05, 0.2), 0.05, 7),    # on one axis
    ((17, 15, 13), (0.1, 0.2, 0.1), 0.11, 4),     # above a voxel on two: no bound
    ((17, 15, 13), (0.3, 0.2, 0.25), 0.05, 1),    # six offsets
    ((9, 8, 7), (0.2, 0.2, 0.2), 0.19, 27),
    ((1, 12, 11), (0.1, 0.1, 0.1), 0.1, 10),
    ((2, 2, 40), (0.1, 0.1, 0.1), 0.08, 10),
])
def test_counts_equal_at_bound_edges(shape, d, dta, interp, local):
    rng = np.random.default_rng(interp * 100 + shape[0])
    for spread in (0.02, 0.1, 0.6):
        ref = rng.uniform(0.2, 1.0, shape)
        ev = ref * (1 + spread * rng.standard_normal(shape))
        want, got = _both(ref, ev, d, 0.02, dta, 0.01, interp, local)
        log(f"gamma {shape} d={d} dta={dta} K={interp} local={local} spread={spread}: {want} {got}")
        assert want == got


@pytest.mark.parametrize("local", [True, False])
def test_counts_equal_over_twelve_decades(local):
    """No threshold and doses from 1e-12 to 1 side by side: the interpolated
    values' rounding is then far above the tolerance of the small voxels."""
    rng = np.random.default_rng(2)
    shape = (14, 13, 12)
    ref = 10.0 ** rng.uniform(-12, 0, shape)
    for ev in (ref * rng.uniform(0.9, 1.1, shape), 10.0 ** rng.uniform(-12, 0, shape),
               ref * (1 + 0.02 * np.sign(rng.standard_normal(shape)))):
        want, got = _both(ref, ev, (0.1, 0.12, 0.1), 0.02, 0.05, 0.0, 10, local)
        log(f"gamma decades local={local}: {want} {got}")
        assert want == got


def test_counts_equal_beside_infinities_and_nan():
    """An evaluated map with infinite and NaN voxels: a cell that touches one
    passes nothing beyond what the definition passes."""
    rng = np.random.default_rng(4)
    ref = rng.uniform(0.3, 1.0, (12, 11, 10))
    ev = ref * (1 + 0.05 * rng.standard_normal(ref.shape))
    k = rng.choice(ref.size, 60, replace=False)
    ev.ravel()[k[:20]] = np.inf
    ev.ravel()[k[20:40]] = -np.inf
    ev.ravel()[k[40:]] = np.nan
    for local in (True, False):
        want, got = _both(ref, ev, (0.1, 0.1, 0.1), 0.02, 0.06, 0.01, 10, local)
        log(f"gamma inf/nan local={local}: {want} {got}")
        assert want == got


@pytest.mark.parametrize("n", [1, 7, 8, 31, 32, 33, 2047, 2048, 2049, 70001])
def test_counts_equal_at_list_sizes(n):
    """Every voxel of a line fails at the zero offset: list lengths around a
    wave's 8 voxels, a workgroup's 32 and the first pass's tile."""
    rng = np.random.default_rng(n)
    ref = rng.uniform(0.5, 1.0, (1, 1, n))
    ev = ref * (1 + 0.05 * np.sign(rng.standard_normal(n)))
    want, got = _both(ref, ev, (0.1, 0.1, 0.1), 0.02, 0.05, 0.01, 10, True)
    log(f"gamma list n={n}: {want} {got}")
    assert want == got
