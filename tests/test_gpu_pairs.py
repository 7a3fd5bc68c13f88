"""Two lanes per electron: the form taken by a set of an eighth to a quarter of the
tail threshold (and, on FP64 fields, further up), against one lane per electron, bit
by bit, on grids whose cells hold an electron for the whole run or a step, with an
odd number of electrons, collisions, exits and rebirths."""
import math
from dataclasses import replace

import numpy as np
import pytest

from gpu_helpers import run_gpu, same_state, say, stored
from synthetic import AU, SphericalGrid, fields, workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rebirth", [False, True])
@pytest.mark.parametrize("precision", ["f64", "f32_acc64", "f32_kahan"])
@pytest.mark.parametrize("store", ["f32", "f64"])
@pytest.mark.parametrize("shape,dt,n", [((5, 4, 3), 4.0, 301), ((255, 33, 66), 1.0, 333), ((255, 33, 66), 20.0, 449)])
def test_two_lanes_give_the_bits_of_one(shape, dt, n, store, precision, rebirth):
    grid = SphericalGrid(*shape, 0.1 * AU, 2.0 * AU)
    f = stored(fields.parker(grid), store)
    ens = replace(workloads.config_small(n=n).ensembles[0], lat0=math.radians(10.0), dlat=math.radians(8.0),
                  dlon=0.2, mu_lo=-1.0, r0=0.5 * AU, dr0=0.2 * AU, lambda_par=0.02 * AU, r_out=1.0 * AU, r_in=0.11 * AU)
    if rebirth:
        ens = replace(ens, rebirth_steps=400, r_out=0.6 * AU)
    wl = workloads.Workload(f"pairs-{shape}", grid, None, [ens], dt, 300)
    say(f"pairs: grid {shape}, dt {dt}, {store} field, {precision}, rebirth {rebirth}")
    kw = dict(store_dtype=store, chunk=20, precision=precision, log_depth=8)
    one, log1 = run_gpu(wl, f, tail_threshold=0, **kw)
    two, log2 = run_gpu(wl, f, tail_threshold=2000, **kw)
    same_state(one, two)
    assert np.array_equal(log1, log2)
    assert np.any(one["k"] > 0)
