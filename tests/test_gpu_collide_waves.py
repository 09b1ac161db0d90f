"""The collide kernel's pairs per wave with a network sampler -- 16, 32 or 64,
by the accepted pairs against the waves of its grid, which are four per
workgroup and at most 512 workgroups with the FP32 network, 768 with BF16 or
FP8 -- for each precision at counts inside each of its own ranges, against the
fused strategy: the same particles bit for bit, and the same counts."""
import os

import numpy as np
import pytest

import paper_2206_02937_amd
from paper_2206_02937_amd import plasma

pytestmark = pytest.mark.gpu

WEIGHTS = os.path.join(os.path.dirname(paper_2206_02937_amd.__file__), "weights", "sampler_2x64x4.csnet")
BLOCKS = {"mlp_f32": 512, "mlp_bf16": 768, "mlp_fp8": 768}
# fractions of the range of each split that the counts are to lie in
SPLITS = {16: (0.0, 16), 32: (16, 32), 64: (32, 64)}


@pytest.mark.parametrize("precision", sorted(BLOCKS))
@pytest.mark.parametrize("per_wave", sorted(SPLITS))
def test_each_split(precision, per_wave):
    import torch

    from paper_2206_02937_amd import compton

    ctx = compton.Context(0)
    net = compton.MLP.load(ctx, WEIGHTS)
    if precision != "mlp_f32":
        cx, cu = plasma.sampler_inputs(4096, seed=7, x_min=1e-8, x_max=1e3)
        net.quantize(precision, torch.from_numpy(cx.astype(np.float32)).cuda(),
                     torch.from_numpy(cu.astype(np.float32)).cuda())
    p = plasma.grid(seed=6, nx=64, ny=64, per_cell=256)  # 2^20 pairs, a collision in 20 at p.dt
    waves = 4 * BLOCKS[precision]
    lo, hi = (waves * f for f in SPLITS[per_wave])
    dt = p.dt * 0.5 * (lo + hi) / (0.05 * p.n_pairs)
    out = {}
    for strategy in ("compact", "fused"):
        ctx.set_strategy(strategy)
        e, g, oe, og = compton.to_device(p)
        stats = ctx.stats_buffer()
        ctx.step(e, g, oe, og, dt, p.density_norm, p.seed, 3, sampler=precision, mlp=net, stats=stats)
        out[strategy] = (e, g, compton.decode_stats(stats))
    (e0, g0, s0), (e1, g1, s1) = out["compact"], out["fused"]
    assert lo < s0["n_collided"] <= hi
    for k in "xyzw":
        assert torch.equal(e0[k], e1[k]) and torch.equal(g0[k], g1[k]), k
    for k in ("n_pairs", "n_collided", "n_clipped", "n_invalid", "n_fallback"):
        assert s0[k] == s1[k], k
    net.close()
    ctx.close()
