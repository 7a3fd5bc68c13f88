"""Export of the state in injection order, whose gathers are shared out by array below
786,432 particles and over the particles above: after reorders, every array against the
same run without any reorder, bit by bit, at workgroup edges and on both sides."""
import pytest

import paper_2403_06706_amd as gcp
from gpu_helpers import field_of, same_state, small

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 1023, 1025, 5000, 786432, 786433])
def test_exported_state_is_in_injection_order(n):
    wl = small(n=n, hours=0.1)
    f = field_of(wl)
    out = []
    for order in ("bin", "none"):
        ctx = gcp.Context(device=0, order=order, chunk_steps=16, tail_threshold=0)
        ctx.load_field(wl.grid, f, "f64")
        ctx.inject(wl.ensembles[0])
        ctx.advance(wl.dt, 48)
        out.append(gcp.state_to_numpy(ctx.get_state()))
        ctx.close()
    same_state(out[0], out[1])
