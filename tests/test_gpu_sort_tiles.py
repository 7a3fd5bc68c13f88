"""The cell sort at the edges of its forms: one workgroup up to a tile of 4,096
slots (one to four items per lane), several tiles with look-back past it, a look-back
longer than the words it keeps in flight, and an old live prefix shorter than the
slots.  Whole numbers: the order is checked exactly, and the state bit by bit
against a run that never reorders."""
import pytest

import oracle as O
import paper_2403_06706_amd as gcp
from gpu_helpers import field_of, same_state, small
from synthetic import AU
from test_gpu_order import check_binning

SPEC = O.MomentSpec(n_rbins=4, r_lo=0.1 * AU, r_hi=2.0 * AU)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [300, 1024, 1025, 4095, 4097, 8192, 12289, 50000])
def test_sort_order_and_moved_particles(n):
    wl = small(n=n, hours=0.5)
    f = field_of(wl)
    out = []
    for order in ("bin", "none"):
        ctx = gcp.Context(device=0, order=order, chunk_steps=64, tail_threshold=0)
        ctx.load_field(wl.grid, f, "f64")
        ctx.inject(wl.ensembles[0])
        if order == "bin":
            check_binning(ctx, wl, 0, wl.dt, 1280, f"n {n}")
        else:
            ctx.advance(wl.dt, 1280)
            ctx.advance(wl.dt, 1)
        ctx.advance(wl.dt, 100)
        counts = ctx.moments(SPEC)[:6].cpu().tolist()      # per status, collisions, steps: sums over all slots
        out.append((gcp.state_to_numpy(ctx.get_state()), counts))
        ctx.close()
    same_state(out[0][0], out[1][0])
    assert out[0][1] == out[1][1] and sum(out[0][1][:4]) == n and out[0][1][0] < n
