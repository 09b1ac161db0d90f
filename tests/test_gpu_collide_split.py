"""The compact strategy's collide kernel with a network sampler takes 16, 32 or
64 accepted pairs per wave, by their number against the grid's 2048 waves
(at most 32768, 65536, more).  Each split against the fused strategy, which
takes its pairs from queues: the same particles bit for bit, and the same
counts."""
import numpy as np
import pytest

from paper_2206_02937_amd import plasma

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2206_02937_amd import compton

    c = compton.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("precision", ["mlp_f32", "mlp_bf16", "mlp_fp8"])
@pytest.mark.parametrize("side, dt_factor, lo, hi", [(64, 0.4, 1000, 32768), (64, 0.8, 32769, 65536),
                                                    (64, 2.0, 65537, 1 << 20)])
def test_split_matches_fused(ctx, precision, side, dt_factor, lo, hi):
    import os

    import torch

    import paper_2206_02937_amd
    from paper_2206_02937_amd import compton

    weights = os.path.join(os.path.dirname(paper_2206_02937_amd.__file__), "weights", "sampler_2x64x4.csnet")
    net = compton.MLP.load(ctx, weights)
    if precision != "mlp_f32":
        cx, cu = plasma.sampler_inputs(4096, seed=7, x_min=1e-8, x_max=1e3)
        net.quantize(precision, torch.from_numpy(cx.astype(np.float32)).cuda(),
                     torch.from_numpy(cu.astype(np.float32)).cuda())
    p = plasma.grid(seed=6, nx=side, ny=side, per_cell=256)
    out = {}
    for strategy in ("compact", "fused"):
        ctx.set_strategy(strategy)
        e, g, oe, og = compton.to_device(p)
        stats = ctx.stats_buffer()
        ctx.step(e, g, oe, og, dt_factor * p.dt, p.density_norm, p.seed, 3, sampler=precision, mlp=net, stats=stats)
        out[strategy] = (e, g, compton.decode_stats(stats))
    ctx.set_strategy("fused")
    net.close()
    (e0, g0, s0), (e1, g1, s1) = out["compact"], out["fused"]
    assert lo <= s0["n_collided"] <= hi
    for k in "xyzw":
        assert torch.equal(e0[k], e1[k]) and torch.equal(g0[k], g1[k]), k
    for k in ("n_pairs", "n_collided", "n_clipped", "n_invalid", "n_fallback"):
        assert s0[k] == s1[k], k
    assert s0["energy_before"] == pytest.approx(s1["energy_before"], rel=1e-12)
    assert s0["energy_after"] == pytest.approx(s1["energy_after"], rel=1e-12)
