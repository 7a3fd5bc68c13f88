"""Gathers that keep a cell's nodes in registers: electrons that stay in one cell
for the whole run, cross one every few steps or several in a step, on the
smallest grids, over the clamped edges of the grid and with negative longitudes
that wrap, against the oracle (round-off of about 1e-16 per step over 300 steps;
bar 1e-10), in every form of the push that keeps cells."""
import math
from dataclasses import replace

import numpy as np
import pytest

from gpu_helpers import compare, run_gpu, run_oracle, say, stored
from synthetic import AU, SphericalGrid, fields, workloads

pytestmark = pytest.mark.gpu

# grid, time step (s): cells of 1.9 AU, 0.5 AU and 0.0075 AU against up to 0.5 c dt
CASES = [((2, 2, 2), 4.0), ((5, 4, 3), 4.0), ((7, 6, 5), 20.0), ((255, 33, 66), 1.0), ((255, 33, 66), 20.0)]
# tail_threshold: one lane per electron, the same in the tail, four lanes
FORMS = {"lane": 0, "latency": 600, "quad": 1 << 20}


@pytest.mark.parametrize("full", [False, True])
@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("store", ["f32", "f64"])
@pytest.mark.parametrize("shape,dt", CASES)
def test_resident_cells_match_the_oracle(shape, dt, store, form, full):
    grid = SphericalGrid(*shape, 0.1 * AU, 2.0 * AU)
    f = stored(fields.parker(grid), store)
    x = stored(fields.parker_extra(grid), store) if full else None
    ens = replace(workloads.config_small(n=300).ensembles[0], lat0=math.radians(10.0), dlat=math.radians(8.0),
                  dlon=0.2, mu_lo=-1.0, r0=0.5 * AU, dr0=0.2 * AU, lambda_par=0.2 * AU, r_out=1.99 * AU, r_in=0.11 * AU)
    wl = workloads.Workload(f"cells-{shape}", grid, None, [ens], dt, 300)
    say(f"cells: grid {shape}, dt {dt}, {store} field, {form} form, full equations: {full}")
    st, _ = run_gpu(wl, f, store_dtype=store, chunk=20, tail_threshold=FORMS[form], extra=x)
    p, _, _, _ = run_oracle(wl, f, extra=x)
    compare(st, p, ens.m, 1e-10, f"{shape} {store} {form}")
    assert np.any(st["ph"] < 0.0)
