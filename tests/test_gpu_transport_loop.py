"""The transport's work distribution and step loop at their edges: history
counts around a wave, a workgroup and the first ranges; launches with few and
many waves, small and large claims; step limits around the number of steps a
wave takes between two looks at its waiting lanes; and the instances with and
without per-history records.  The tally and ledger do not depend on any of it."""

from dataclasses import replace

import numpy as np
import pytest

import workloads
from gpu_common import log
from workloads import configs

pytestmark = pytest.mark.gpu

METHOD, GEODESIC = 127, 63


def _setup(flags=METHOD, max_steps=None, size=24):
    from paper_2511_03115_amd import sde
    wl = configs.insert(70.0, n=1, size=size, depth=60)
    params = replace(wl.params, flags=flags, **({"max_steps": max_steps} if max_steps else {}))
    sde.init_materials(wl.phantom.materials, params,
                       workloads.nuclear_for_phantom(wl.phantom, params.lattice()))
    return wl, sde.DevicePhantom.from_host(wl.phantom)


def _run(spots, ph, launch, seed=5, records=False):
    import torch
    from paper_2511_03115_amd import sde
    plan = sde.Plan(spots, ph, seed, launch=launch)
    rec = None
    if records:
        rec = torch.zeros((plan.n_histories, 12), dtype=torch.float32, device="cuda")
        plan.set_records(rec)
    plan.execute(None)
    tally = torch.zeros(ph.material_id.shape, dtype=torch.int64, device="cuda")
    ledger, scale = plan.results(tally)
    plan.close()
    return tally.cpu().numpy(), ledger, scale, None if rec is None else rec.cpu().numpy()


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 511, 513, 4097, 70001])
def test_every_history_runs_once_in_any_launch(n):
    wl, ph = _setup()
    spots = [replace(wl.spots[0], n_histories=n, weight=float(n))]
    ref = None
    for launch in ({"block": 64, "grid": 1}, {"block": 1024, "grid": 3, "refill": 64},
                   {"block": 512, "grid": 512, "refill": 1, "claim_chunk": 1000},
                   {"block": 256, "grid": 256, "jump_batch": 1},
                   {"block": 1024, "grid": 256, "tile_nx": 6, "tile_ny": 6, "tile_nz": 50,
                    "tile_x0": 9, "tile_y0": 9}):
        if n > 5000 and launch["grid"] == 1:
            continue   # one wave would take a second
        tally, ledger, _, _ = _run(spots, ph, launch)
        log(f"loop n={n} launch={launch}: {ledger.tolist()}")
        assert int(ledger[6]) == n
        assert int(tally.sum()) == int(ledger[0])
        if ref is None:
            ref = (tally, ledger)
        assert np.array_equal(tally, ref[0]) and np.array_equal(ledger, ref[1])


@pytest.mark.parametrize("n_per_spot", [1, 7, 300])
def test_spots_with_and_without_histories(n_per_spot):
    wl, ph = _setup()
    sp = wl.spots[0]
    spots = [replace(sp, E_MeV=60.0 + k, x_cm=0.05 * k, weight=1.0,
                     n_histories=n_per_spot if k % 3 else 0) for k in range(20)]
    a = _run(spots, ph, {"block": 64, "grid": 5})
    b = _run(spots, ph, {"block": 1024, "grid": 256})
    assert int(a[1][6]) == sum(s.n_histories for s in spots)
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])


@pytest.mark.parametrize("max_steps", [1, 2, 5, 6, 7, 11, 12, 13, 60])
def test_step_limit_is_exact(max_steps):
    wl, ph = _setup(max_steps=max_steps)
    spots = [replace(wl.spots[0], n_histories=3000, weight=3000.0)]
    tally, ledger, _, rec = _run(spots, ph, None, records=True)
    steps, end = rec[:, 1], rec[:, 3]
    log(f"limit {max_steps}: steps up to {steps.max()}, {np.sum(end == 4)} at the limit")
    assert steps.max() <= max_steps and np.all(steps[end == 4] == max_steps)
    assert int(ledger[5]) == int(steps.sum())
    assert int(tally.sum()) == int(ledger[0])


@pytest.mark.parametrize("flags", [METHOD, GEODESIC])
def test_records_do_not_change_the_tally(flags):
    wl, ph = _setup(flags)
    spots = [replace(wl.spots[0], n_histories=20000, weight=20000.0)]
    a = _run(spots, ph, None)
    b = _run(spots, ph, None, records=True)
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
    assert np.all(b[3][:, 3] > 0) and int(b[3][:, 1].sum()) == int(a[1][5])
    assert int(b[3][:, 2].sum()) == int(a[1][7])
