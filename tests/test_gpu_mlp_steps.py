"""The training step at the edges of its blocks of 32 pairs and of its splits: one
pair, a block less, exactly and one more than full, the fewest blocks that are
split, more blocks than workgroups, and a smaller step after a larger one in the
same workspace, against the oracle's reverse mode.  The bar per gradient tensor
is that of the BF16 products (three times the arithmetic model's error at 256
pairs, as for the other gradient tests) widened by sqrt(256 / pairs) below that
size, where fewer rounding errors average out."""
import math

import numpy as np
import pytest

import oracle as O  # noqa: F401
from gpu_helpers import say
from oracle import mlp_oracle
from synthetic import workloads
from synthetic.mlp_setup import init_params, make_spec

pytestmark = pytest.mark.gpu
WC, BETA = np.array([1.0, 0.5, 2.0, 1.0, 0.25, 1.0]), 10.0


@pytest.fixture(scope="module")
def net():
    import paper_2403_06706_amd as gcp
    wl = workloads.config_small(n=16)
    f = wl.build_field(wl.grid)
    spec = make_spec(wl.grid, f, seed=1)
    params = {k: np.asarray(v, dtype=np.float32).astype(np.float64) for k, v in init_params(seed=4).items()}
    ctx = gcp.Context(device=0)
    ctx.load_field(wl.grid, f, "f64")
    ctx.mlp_set(spec.freq, spec.r_ref, spec.scale, spec.power, params)
    yield wl, spec, params, ctx
    ctx.close()


@pytest.mark.parametrize("n", [1, 31, 32, 33, 191, 193, 16500, 64])
def test_gradient_at_block_edges(net, n):
    import torch
    wl, spec, params, ctx = net
    rng = np.random.default_rng(n)
    g = wl.grid
    x = np.stack([rng.uniform(0.3, 1.8, n) * 1.495978707e11, rng.uniform(0.6, math.pi - 0.6, n),
                  rng.uniform(0, 2 * math.pi, n)])
    d = np.array([0.1 * (g.r_max - g.r_min) / (g.nr - 1), 0.1 * math.pi / g.nth, 0.2 * math.pi / g.nph])
    y = x + d[:, None] * rng.normal(size=x.shape)
    pts = torch.tensor(np.concatenate([x, y], axis=1), device="cuda").contiguous()
    tgt = ctx.field_sample(pts)[:, :6].contiguous()
    say(f"training gradient of {n} pairs")
    loss = ctx.mlp_train_step(pts, tgt, wc=WC, beta_pair=BETA, apply=False)
    got = ctx.mlp_grads()
    t = tgt.cpu().numpy()
    want_l, want = mlp_oracle.loss_and_grad(spec, params, x.T, t[:n], y.T, t[n:], WC, BETA)
    widen = max(1.0, math.sqrt(256 / n))
    assert abs(loss - want_l) <= 2e-3 * widen * want_l
    for k in want:
        err = np.linalg.norm(got[k] - want[k]) / np.linalg.norm(want[k])
        assert err <= 2e-2 * widen, f"{k}: {err:.3e}"
