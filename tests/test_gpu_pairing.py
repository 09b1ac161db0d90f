"""The pair kernels' pairing, which depends on how many cells a wave of 64
consecutive pairs spans (one, two, up to 64, more) and on how many points its
cycle-walk can leave the range at, against the per-cell strategy, which pairs
every lane by itself: the same particles bit for bit and the same counts.
And a wave that holds one unusable or extreme pair: the other pairs' results
do not change."""
import numpy as np
import pytest

from paper_2206_02937_amd import plasma

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2206_02937_amd import compton

    c = compton.Context(0)
    yield c
    c.set_strategy("fused")
    c.close()


def _plasma(ne, ng, dtype, seed=8):
    """Cells with ne[c] electrons and ng[c] photons; dt for P of order 0.1 in
    a cell of 256."""
    rng = np.random.default_rng(seed)
    off_e = np.concatenate([[0], np.cumsum(ne)]).astype(np.int64)
    off_g = np.concatenate([[0], np.cumsum(ng)]).astype(np.int64)
    e = plasma._electrons_from_pmag(rng, plasma.maxwell_juttner_momentum(rng, int(off_e[-1]), 0.5), dtype)
    g = plasma._photons_from_energy(rng, plasma.log_uniform(rng, int(off_g[-1]), 1e-4, 1e1), dtype)
    return plasma.Plasma("cells", e, g, off_e, off_g, 0.1, 1.0 / 256, seed, {})


def _cells(kind):
    rng = np.random.default_rng(3)
    if kind == "one":  # M a power of two; odd M, few points out; many points out (generic walk)
        return [4096, 4095, 2049, 20000], [4096, 4095, 2049, 20000]
    if kind == "two":  # waves across two cells: points out of both, at most 64 and more
        return [250] * 40 + [129] * 40 + [1000, 33, 1000, 65], [250] * 40 + [129] * 40 + [1000, 33, 1000, 65]
    if kind == "unequal":
        n = rng.integers(0, 300, 200)
        return n, rng.integers(0, 300, 200)
    if kind == "small":  # 64 and 65 cells in a chunk, more than 64 in a wave (empty cells)
        n = np.concatenate([np.full(64, 4), np.full(65, 4), rng.integers(0, 2, 1000), rng.integers(0, 4, 1000)])
        return n, n
    if kind == "runs":  # long runs of the cell map between small cells, and an empty end
        n = np.array([1, 0, 5000, 3, 2, 513, 0, 12000, 64, 0, 0])
        return n, n
    return [1], [1]  # "single"


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("kind", ["single", "one", "two", "unequal", "small", "runs"])
def test_pairing_matches_per_cell(ctx, kind, dtype):
    import torch

    from paper_2206_02937_amd import compton

    p = _plasma(*_cells(kind), dtype)
    out = []
    for strategy, chunks, ppl, wide in (("per_cell", 0, 0, 0), ("fused", 0, 0, 0), ("fused", 3, 0, 1),
                                        ("compact", 0, 1, 0), ("compact", 3, 2, 1), ("compact", 32, 4, 0)):
        ctx.set_strategy(strategy)
        ctx.set_chunks_per_block(chunks)
        ctx.set_pairs_per_lane(ppl)
        ctx.set_wide_index(wide)
        e, g, oe, og = compton.to_device(p)
        stats = ctx.stats_buffer()
        ctx.step(e, g, oe, og, p.dt, p.density_norm, p.seed, 3, stats=stats)
        out.append((e, g, compton.decode_stats(stats)))
    for setter in (ctx.set_chunks_per_block, ctx.set_pairs_per_lane, ctx.set_wide_index):
        setter(0)
    e0, g0, s0 = out[0]
    assert s0["n_pairs"] == int(np.minimum(np.diff(p.off_e), np.diff(p.off_g)).sum())
    for e, g, s in out[1:]:
        for k in "xyzw":
            assert torch.equal(e0[k], e[k]) and torch.equal(g0[k], g[k]), k
        for k in ("n_pairs", "n_collided", "n_clipped", "n_invalid"):
            assert s0[k] == s[k], k
        assert s0["sum_prob"] == pytest.approx(s["sum_prob"], rel=1e-12)
        assert s0["energy_before"] == pytest.approx(s["energy_before"], rel=1e-12)
        assert s0["energy_after"] == pytest.approx(s["energy_after"], rel=1e-12)


@pytest.mark.parametrize("strategy", ["fused", "compact", "per_cell"])
@pytest.mark.parametrize("species, comp, value, invalid", [
    ("e", "x", np.nan, 1), ("e", "w", -1.0, 1), ("g", "w", np.inf, 1), ("g", "z", -np.inf, 1), ("e", "w", -0.0, 0),
    ("g", "xyz", 0.0, 0), ("g", "xyz", 1e-170, 0), ("e", "y", 1e160, 0), ("g", "xyz", 5e-324, 0)])
def test_one_odd_pair_leaves_the_others(ctx, strategy, species, comp, value, invalid):
    import torch

    from paper_2206_02937_amd import compton

    ctx.set_strategy(strategy)
    n, i = 192, 77
    res = []
    for odd in (False, True):
        p = _plasma([n], [n], np.float64)
        for c in comp if odd else "":
            (p.e if species == "e" else p.g)[c][i] = value
        e, g, oe, og = compton.to_device(p)
        stats = ctx.stats_buffer()
        ctx.step(e, g, oe, og, 20 * p.dt, p.density_norm, p.seed, 3, stats=stats)
        res.append((e, g, compton.decode_stats(stats)))
    (e0, g0, s0), (e1, g1, s1) = res
    assert s0["n_invalid"] == 0 and s1["n_invalid"] == invalid
    assert s0["n_collided"] > 20
    # at most the odd particle and its partner differ
    for d0, d1 in ((e0, e1), (g0, g1)):
        diff = sum((d0[k].view(torch.int64) != d1[k].view(torch.int64)).int() for k in "xyzw") > 0
        assert int(diff.sum()) <= 1
