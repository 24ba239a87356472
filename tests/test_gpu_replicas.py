"""Tally replicas are left zero by the conversion and only the first is
cleared by a plan's next execution: every number of them (those with an
instance of their own, odd ones, one, the most), executed again and again by
launches and by graph replays, in turn, gives the same dose and ledger."""

from dataclasses import replace

import numpy as np
import pytest

import workloads
from gpu_common import log
from workloads import configs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_rep", [1, 2, 3, 4, 8, 11, 16])
def test_executions_with_replicas(n_rep):
    import torch
    from paper_2511_03115_amd import sde
    wl = configs.insert(120.0, n=1, size=37, depth=101)
    sde.init_materials(wl.phantom.materials, wl.params,
                       workloads.nuclear_for_phantom(wl.phantom, wl.params.lattice()))
    ph = sde.DevicePhantom.from_host(wl.phantom)
    spots = [replace(wl.spots[0], E_MeV=80.0 + 9 * k, x_cm=0.4 * (k - 2), n_histories=4000)
             for k in range(5)]
    base = None
    for use in (None, n_rep):
        launch = {"block": 256, "grid": 256, "tally_replicas": use or 1}
        plan = sde.Plan(spots, ph, 11, launch=launch)
        for graph in (False, True, False, True, True, False, False):
            dose = torch.full(wl.phantom.material_id.shape, -1.0, dtype=torch.float64,
                              device="cuda")
            plan.execute(dose, use_graph=graph)
            torch.cuda.synchronize()
            got = dose.cpu().numpy(), plan.results()[0]
            base = base or got
            assert np.array_equal(base[0], got[0]) and np.array_equal(base[1], got[1])
        plan.close()
    log(f"replicas {n_rep}: {base[1].tolist()}")
    assert base[0].max() > 0 and int(base[1][6]) == 20_000


@pytest.mark.parametrize("n", [1000, 263_000])
def test_default_replicas_over_the_rule(n):
    """Two and eight by default: the tally of one."""
    import torch
    from paper_2511_03115_amd import sde
    wl = configs.slab(80.0, n=n, size=33, depth=61)
    sde.init_materials(wl.phantom.materials, wl.params,
                       workloads.nuclear_for_phantom(wl.phantom, wl.params.lattice()))
    ph = sde.DevicePhantom.from_host(wl.phantom)
    got = []
    for launch in (None, {"tally_replicas": 1}):
        tally = torch.zeros(wl.phantom.material_id.shape, dtype=torch.int64, device="cuda")
        sde.transport(wl.spots, ph, 5, tally_out=tally, launch=launch)
        got.append(tally.cpu().numpy())
    log(f"default replicas n={n}")
    assert got[0].any() and np.array_equal(*got)
