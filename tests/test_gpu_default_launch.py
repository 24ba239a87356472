"""The launch the library chooses when none is given (workgroups, jump
batches, tally tile) against a plain explicit one, over the beams and phantoms
it distinguishes: tally and ledger are equal, whatever it chose."""

from dataclasses import replace

import numpy as np
import pytest

import workloads
from gpu_common import log
from workloads import configs

pytestmark = pytest.mark.gpu

PLAIN = {"block": 256, "grid": 64, "refill": 8, "jump_batch": 8}


def _compare(phantom, params, spots, seed=3):
    import torch
    from paper_2511_03115_amd import sde
    sde.init_materials(phantom.materials, params,
                       workloads.nuclear_for_phantom(phantom, params.lattice()))
    ph = sde.DevicePhantom.from_host(phantom)
    got = []
    for launch in (None, PLAIN):
        dose = torch.zeros(phantom.material_id.shape, dtype=torch.float64, device="cuda")
        tally = torch.zeros(phantom.material_id.shape, dtype=torch.int64, device="cuda")
        r = sde.transport(spots, ph, seed, dose_out=dose, tally_out=tally, launch=launch)
        got.append((tally.cpu().numpy(), r.ledger, dose.cpu().numpy()))
    n = sum(s.n_histories for s in spots)
    log(f"default launch {phantom.shape} spots={len(spots)} n={n}: {got[0][1].tolist()}")
    assert int(got[0][1][6]) == n
    for a, b in zip(*got):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("n", [1, 100, 30_000, 65_536, 65_537, 200_000, 262_145, 1_200_000])
def test_history_counts(n):
    wl = configs.water100_small(n)
    _compare(wl.phantom, wl.params,
             [replace(wl.spots[0], E_MeV=70.0, sigmaE_rel=0.01, sigma_xy_cm=0.3)])


@pytest.mark.parametrize("shape", [(1, 1, 30), (5, 40, 60), (6, 6, 60), (11, 13, 7), (64, 9, 90)])
def test_phantom_sizes(shape):
    ph = workloads.water_box(*shape, 0.1)
    _compare(ph, configs.PhysicsParams(),
             workloads.single_spot(80.0, 5000, sigmaE_rel=0.01, sigma_xy_cm=0.2))


@pytest.mark.parametrize("x,y", [(0.0, 0.0), (1.9, -1.9), (-2.0, 2.0), (2.5, 0.0), (40.0, 0.0),
                                 (-1e30, 1e30)])
def test_beams_off_the_axis(x, y):
    """At the edges, outside (every history escapes) and far outside."""
    wl = configs.slab(100.0, n=1, size=40, depth=80)
    _compare(wl.phantom, wl.params,
             workloads.single_spot(100.0, 20_000, sigmaE_rel=0.01, sigma_xy_cm=0.3, x_cm=x,
                                   y_cm=y))


@pytest.mark.parametrize("half", [0.0, 0.5, 1.0, 2.0])
def test_spots_within_and_beyond_the_tile_rule(half):
    """Footprints on both sides of 4 cm, spots without histories or weight
    among them."""
    wl = configs.insert(120.0, n=1, size=60, depth=120)
    spots = [replace(wl.spots[0], E_MeV=80.0 + 5 * k, x_cm=half * ((k % 3) - 1),
                     y_cm=half * (k // 3 - 1), weight=float(k != 4),
                     n_histories=0 if k == 7 else 3000) for k in range(9)]
    _compare(wl.phantom, wl.params, spots)


@pytest.mark.parametrize("flags", [63, 127 | 128, 127 | 256, 1 | 4 | 32])
def test_other_instances(flags):
    wl = configs.ct_like(100.0, n=1, size=40, depth=100)
    _compare(wl.phantom, replace(wl.params, flags=flags),
             workloads.single_spot(100.0, 4000, sigmaE_rel=0.01, sigma_xy_cm=0.3))
