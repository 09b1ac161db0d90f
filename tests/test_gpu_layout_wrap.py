"""Offsets that are no valid layout and whose counts leave 32 bits: the step
reports the layout, changes no particle and leaves its scratch fit for the next
step (the scan's cell map is filled inside its bounds whatever the counts add up
to)."""
import numpy as np
import pytest

from paper_2206_02937_amd import plasma

pytestmark = pytest.mark.gpu


def _offsets(kind, off):
    bad = off.copy()
    if kind == "one huge cell":
        bad[1] = 3 * 10 ** 9
    elif kind == "two huge cells":
        bad[1], bad[2] = 16 * 10 ** 8, 32 * 10 ** 8
    elif kind == "beyond the particles":
        bad[1:-1] = off[-1] * np.arange(1, off.size - 1)
    else:
        bad[-2] = 2 ** 31 - 1
    return bad


@pytest.mark.parametrize("strategy", ["fused", "compact", "noalloc"])
@pytest.mark.parametrize("kind", ["one huge cell", "two huge cells", "beyond the particles", "last but one"])
def test_counts_beyond_32_bits(strategy, kind):
    import torch

    from paper_2206_02937_amd import compton

    p = plasma.grid(seed=5, nx=6, ny=5, per_cell=70)
    ctx, fresh = compton.Context(0), compton.Context(0)
    for c in (ctx, fresh):
        c.set_strategy("compact" if strategy == "compact" else "fused")
    step = [c.step_noalloc if strategy == "noalloc" else c.step for c in (ctx, fresh)]
    e, g, oe, og = compton.to_device(p)
    stats = ctx.stats_buffer()
    bad = torch.from_numpy(_offsets(kind, p.off_e)).cuda()
    for _ in range(2):
        step[0](e, g, bad, bad, p.dt, p.density_norm, p.seed, 0, stats=stats)
    torch.cuda.synchronize()
    st = compton.decode_stats(stats)
    assert st["layout_error"] == 1 and st["n_pairs"] == 0 and st["n_collided"] == 0
    for k in "xyzw":
        assert np.array_equal(e[k].cpu().numpy(), p.e[k]) and np.array_equal(g[k].cpu().numpy(), p.g[k])
    step[0](e, g, oe, og, p.dt, p.density_norm, p.seed, 1, stats=stats)
    e1, g1, _, _ = compton.to_device(p)
    stats1 = fresh.stats_buffer()
    step[1](e1, g1, oe, og, p.dt, p.density_norm, p.seed, 1, stats=stats1)
    torch.cuda.synchronize()
    assert torch.equal(stats, stats1) and compton.decode_stats(stats)["n_collided"] > 0
    for k in "xyzw":
        assert torch.equal(e[k], e1[k]) and torch.equal(g[k], g1[k])
    ctx.close()
    fresh.close()
