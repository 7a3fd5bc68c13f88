"""The moments kernel's wavefront sums at the edges of wavefronts, workgroups and
bin counts, on sets in radial order (a wavefront in one or two bins) and shuffled
(many bins), on tame and untame fields, against the oracle's moments of the same
state: counts equal, each fixed-point sum within one unit per particle (a floor
of a product in another rounding order)."""
import numpy as np
import pytest

import oracle as O
import paper_2403_06706_amd as gcp
from gpu_helpers import field_of, oracle_to_state, run_oracle, say, small, stored
from test_gpu_moments import SPEC, _check

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def state():
    wl = small(n=3000, hours=1.0)
    f = stored(field_of(wl), "f32")
    p, _, _, _ = run_oracle(wl, f, n_steps=1500, dt=1.0)
    return wl, f, p


@pytest.mark.parametrize("n,n_rbins,tame,store", [(1, 38, True, "f32"), (63, 1, True, "f64"), (64, 2, True, "f32"),
                                                  (65, 500, True, "f32"), (511, 38, False, "f32"),
                                                  (513, 1000, True, "f64"), (1500, 3, False, "f64"),
                                                  (3000, 0, True, "f32"), (3000, 38, True, "f32")])
@pytest.mark.parametrize("order", ["radial", "shuffled"])
def test_sums_at_the_edges(state, n, n_rbins, tame, store, order):
    wl, f, p = state
    idx = np.argsort(p["r"], kind="stable") if order == "radial" else np.random.default_rng(n).permutation(len(p))
    sub = p[idx[:n]].copy()
    if not tame:
        f = f.copy()
        f[-1, -1, 0, 7] = 4e30              # one remote node: every gather is tested again
    spec = O.MomentSpec(**dict(SPEC, n_rbins=n_rbins))
    of = O.Field(wl.grid, f)
    want = O.moments(of, O.make_ens_table(wl.ensembles), sub, spec)
    say(f"moments of {n} particles, {n_rbins} bins, tame {tame}, {store}, {order}")
    ctx = gcp.Context(device=0)
    ctx.load_field(wl.grid, f, store)
    ctx.inject(wl.ensembles[0])
    ctx.set_state(oracle_to_state(sub, wl.ensembles[0].m))
    got = ctx.moments(spec).cpu().numpy()
    ctx.close()
    _check(got, want, spec)
