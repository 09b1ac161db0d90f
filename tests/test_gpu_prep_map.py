"""The scan's map from pairs to cells at the limits of its three ways of writing
a cell's entries (by its lane one by one, four at a time, by the whole wave): the
fused and the compact step on such cells against the multi-kernel baseline, which
has no map, bit for bit."""
import numpy as np
import pytest

from paper_2206_02937_amd import plasma

pytestmark = pytest.mark.gpu

# entries per cell (of 64 pairs for the compact strategy, of 256 for the fused)
PATTERNS = {
    "one by one": [8, 0, 1, 8, 7],
    "four at a time": [9] * 7 + [10, 11, 12, 13, 31, 32],
    "four long ones": [33, 8, 40, 9, 100, 3, 64],
    "five long ones": [33, 8, 40, 9, 100, 3, 64, 65],
    "many long ones": [33] * 20 + [200] + [34] * 50,
    "one": [257],
}


@pytest.mark.parametrize("unit", [64, 256])
@pytest.mark.parametrize("name", sorted(PATTERNS))
def test_cells_of_many_entries(name, unit):
    import torch

    from paper_2206_02937_amd import compton

    rng = np.random.default_rng(11)
    entries = np.array(PATTERNS[name])
    if unit == 256:
        entries = entries[: 30]
    n = entries * unit - np.where(entries > 0, rng.integers(0, 64, entries.size), 0)
    p = plasma.grid(seed=4, nx=1, ny=1, per_cell=int(n.sum()))
    off = torch.from_numpy(np.concatenate([[0], np.cumsum(n)]).astype(np.int64)).cuda()
    got = {}
    for strategy in ("multi_kernel", "fused", "compact"):
        ctx = compton.Context(0)
        ctx.set_strategy(strategy)
        e, g, _, _ = compton.to_device(p)
        stats = ctx.stats_buffer()
        ctx.step(e, g, off, off, p.dt, p.density_norm, p.seed, 3, stats=stats)
        torch.cuda.synchronize()
        st = compton.decode_stats(stats)
        assert st["layout_error"] == 0 and st["n_pairs"] == int(n.sum()) and st["n_collided"] > 0
        got[strategy] = [d[k] for d in (e, g) for k in "xyzw"]
        ctx.close()
    for strategy in ("fused", "compact"):
        assert all(torch.equal(a, b) for a, b in zip(got["multi_kernel"], got[strategy])), strategy
