"""The network with 16, 32, 48 or 64 particles per wavefront and four or eight
wavefronts per workgroup: the values of a point and the trajectory of an electron
do not depend on how many others are evaluated with it, so every batch gives the
bits of the same points within the largest batch (whose own values are checked
against the oracle elsewhere)."""
import numpy as np
import pytest

from gpu_helpers import say
from synthetic import workloads
from synthetic.mlp_setup import init_params, make_spec

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def net():
    wl = workloads.config_small(n=40000)
    f = wl.build_field(wl.grid)
    spec = make_spec(wl.grid, f, seed=1)
    return wl, f, spec, init_params(seed=4)


def _context(net, **kw):
    import paper_2403_06706_amd as gcp
    wl, f, spec, params = net
    ctx = gcp.Context(device=0, **kw)
    ctx.load_field(wl.grid, f, "f64")
    ctx.mlp_set(spec.freq, spec.r_ref, spec.scale, spec.power, params)
    return ctx


def test_evaluation_of_any_batch(net):
    import torch
    wl = net[0]
    ctx = _context(net)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    x = torch.rand((3, 600001), dtype=torch.float64, device="cuda", generator=gen)
    g = wl.grid
    x = torch.stack([g.r_min + (0.05 + 0.9 * x[0]) * (g.r_max - g.r_min), 0.5 + 2.1 * x[1], 6.2 * x[2]]).contiguous()
    ref = ctx.mlp_eval(x)
    assert torch.isfinite(ref).all()
    for n in (1, 15, 16, 17, 64, 65, 1000, 16384, 16385, 32768, 32769, 65537, 98305, 131073, 140000, 524289):
        say(f"evaluation of {n} points")
        got = ctx.mlp_eval(x[:, 1:1 + n].contiguous())
        assert torch.equal(got, ref[1:1 + n]), n
    ctx.close()


@pytest.mark.parametrize("n", [1, 17, 500, 16385, 33000])
def test_push_of_any_set(net, n):
    import paper_2403_06706_amd as gcp
    wl = net[0]

    def run(count):
        ctx = _context(net, field_source="mlp")
        ctx.inject(wl.ensembles[0], n=count)
        ctx.advance(1.0, 6)
        st = gcp.state_to_numpy(ctx.get_state())
        ctx.close()
        return st

    say(f"network push of {n} electrons")
    part, whole = run(n), run(40000)
    for k in part:
        if k not in ("cr", "cth", "cph", "cu", "ct"):
            assert np.array_equal(part[k], whole[k][:n]), k
