"""No-time-counter step on the GPU (cs_ntc_step) against the FP64 oracle of
the same method, element by element: the grid workload in FP32 and FP64
storage over several steps, unequal species and weights with empty cells,
long chains of candidates that share a particle (resolved by the per-cell
serial pass), invalid particles, empty inputs, a bad layout, and the full
128x128 grid.

Per-event metric and tolerances as for the pairing step (1e-12 for FP64
storage, 1e-5 for FP32, relative to gamma resp. eps).  A cell with a
candidate whose acceptance is decided within rounding (|u - P/P_max| below
1e-12 P/P_max: both sides decide in FP64) is left out of the per-particle comparison and
counted; every other particle must match, untouched ones bitwise."""
import numpy as np
import pytest

from paper_2206_02937_amd import plasma

pytestmark = pytest.mark.gpu

TOL = {np.float64: 1e-12, np.float32: 1e-5}
AMB = 1e-12


@pytest.fixture(scope="module")
def ctx():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2206_02937_amd import compton

    c = compton.Context(0)
    yield c
    c.close()


def _copy(d):
    return {k: v.copy() for k, v in d.items()}


def _stats(buf):
    s = buf.cpu().numpy()
    d = s.view(np.float64)
    return {"n_pairs": int(s[0]), "n_collided": int(s[1]), "n_clipped": int(s[2]), "n_invalid": int(s[3]),
            "layout_error": int(s[5]), "sum_prob": float(d[8]), "energy_before": float(d[9]),
            "energy_after": float(d[10])}


def _gpu_steps(ctx, p, steps):
    import torch

    from paper_2206_02937_amd import compton

    e, g, oe, og = compton.to_device(p)
    out = []
    for s in steps:
        buf = ctx.stats_buffer()
        ctx.ntc_step(e, g, oe, og, p.dt, p.density_norm, p.seed, s, stats=buf)
        torch.cuda.synchronize()
        out.append((compton.to_host(e), compton.to_host(g), _stats(buf)))
    return out


def _compare(p, before_e, before_g, gpu, ref, diag, dtype):
    """Per-event errors outside ambiguous cells; returns the number of
    ambiguous cells."""
    tol = TOL[np.dtype(dtype).type]
    ge, gg, gst = gpu
    re, rg, rst = ref
    # the decision is taken in FP64 on both sides, whatever the storage
    amb = np.abs(diag["u"] - diag["ratio"]) <= AMB * np.maximum(diag["ratio"], 1e-300)
    amb &= diag["ratio"] >= 0
    bad_cells = np.unique(diag["cell"][amb])
    ne, ng = re["x"].size, rg["x"].size
    mask_e = np.ones(ne, dtype=bool)
    mask_g = np.ones(ng, dtype=bool)
    for c in bad_cells:
        mask_e[p.off_e[c]:p.off_e[c + 1]] = False
        mask_g[p.off_g[c]:p.off_g[c + 1]] = False
    P = lambda d: np.stack([d["x"], d["y"], d["z"]], axis=1).astype(np.float64)
    pr, kr = P(re), P(rg)
    gam = np.sqrt(1 + np.sum(pr * pr, axis=1))
    eps = np.maximum(np.sqrt(np.sum(kr * kr, axis=1)), 1e-300)
    # particles holding a non-finite value never collide: compared exactly
    fin_e, fin_g = np.all(np.isfinite(pr), axis=1), np.all(np.isfinite(kr), axis=1)
    assert np.array_equal(P(ge)[~fin_e], pr[~fin_e], equal_nan=True)
    assert np.array_equal(P(gg)[~fin_g], kr[~fin_g], equal_nan=True)
    mask_e &= fin_e
    mask_g &= fin_g
    err_e = np.linalg.norm(P(ge) - pr, axis=1) / np.where(fin_e, gam, 1.0)
    err_g = np.linalg.norm(P(gg) - kr, axis=1) / np.where(fin_g, eps, 1.0)
    assert np.max(err_e[mask_e], initial=0) <= tol, np.max(err_e[mask_e])
    assert np.max(err_g[mask_g], initial=0) <= tol, np.max(err_g[mask_g])
    # particles the oracle left untouched are bitwise unchanged on the GPU
    for k in "xyz":
        same_e = re[k] == before_e[k]
        same_g = rg[k] == before_g[k]
        assert np.array_equal(ge[k][same_e & mask_e], before_e[k][same_e & mask_e])
        assert np.array_equal(gg[k][same_g & mask_g], before_g[k][same_g & mask_g])
    for k in "w":
        assert np.array_equal(ge[k], before_e[k], equal_nan=True)
        assert np.array_equal(gg[k], before_g[k], equal_nan=True)
    if bad_cells.size == 0:
        for k in ("n_pairs", "n_collided", "n_clipped", "n_invalid"):
            assert gst[k] == rst[k], (k, gst, rst)
    else:
        assert gst["n_pairs"] == rst["n_pairs"]
    assert gst["sum_prob"] == pytest.approx(rst["sum_prob"], rel=1e-9, abs=1e-12)
    return bad_cells.size


def _chain_compare(ctx, orc, p, steps):
    """Each step from the oracle's state of the previous step (so a rare
    ambiguous decision does not spread)."""
    dtype = p.e["x"].dtype
    e, g = _copy(p.e), _copy(p.g)
    n_amb = 0
    res = []
    for s in steps:
        q = plasma.Plasma(p.name, _copy(e), _copy(g), p.off_e, p.off_g, p.dt, p.density_norm, p.seed)
        gres = _gpu_steps(ctx, q, [s])[0]
        be, bg = _copy(e), _copy(g)
        st, diag = orc.ntc_step(e, g, p.off_e, p.off_g, p.dt, p.density_norm, p.seed, s, diagnostics=True)
        n_amb += _compare(p, be, bg, gres, (e, g, st), diag, dtype)
        res.append((st, gres[2], diag))
    assert n_amb <= 2
    return res


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_grid_matches_oracle(ctx, orc, dtype):
    p = plasma.grid(seed=5, nx=8, ny=8, per_cell=256, dtype=dtype)
    res = _chain_compare(ctx, orc, p, [0, 1, 2])
    st, gst, _ = res[0]
    assert st["n_collided"] > 100 and st["n_pairs"] < 64 * 256 / 4
    assert gst["energy_after"] == pytest.approx(gst["energy_before"], rel=1e-12)


def test_unequal_species_weights_and_empty_cells(ctx, orc):
    rng = np.random.default_rng(9)
    counts_e = np.array([5, 0, 17, 300, 3, 1, 0, 40, 513])
    counts_g = np.array([9, 4, 17, 10, 3, 0, 0, 600, 2])
    ne, ng = int(counts_e.sum()), int(counts_g.sum())
    pm = plasma.maxwell_juttner_momentum(rng, ne, 0.5)
    ux, uy, uz = plasma.isotropic(rng, ne)
    eps = plasma.log_uniform(rng, ng, 1e-3, 1.0)
    vx, vy, vz = plasma.isotropic(rng, ng)
    e = {"x": pm * ux, "y": pm * uy, "z": pm * uz, "w": rng.uniform(0.5, 2.0, ne)}
    g = {"x": eps * vx, "y": eps * vy, "z": eps * vz, "w": rng.uniform(0.5, 2.0, ng)}
    off_e = np.concatenate([[0], np.cumsum(counts_e)]).astype(np.int64)
    off_g = np.concatenate([[0], np.cumsum(counts_g)]).astype(np.int64)
    p = plasma.Plasma("unequal", e, g, off_e, off_g, 0.2, 0.05, 11)
    res = _chain_compare(ctx, orc, p, [0, 1])
    st, _, diag = res[0]
    assert st["n_collided"] > 0
    # cells without one of the species draw no candidates
    both = (counts_e > 0) & (counts_g > 0)
    per_cell = np.bincount(diag["cell"], minlength=counts_e.size)
    assert np.all(per_cell[~both] == 0) and per_cell[3] > 50 and per_cell[7] > 50


def test_long_chains_use_the_serial_pass(ctx, orc):
    """Cells of one electron and many photons (and the reverse) with a large
    bound: every candidate of such a cell shares its lone particle, so the
    chains are far longer than the parallel rounds and the per-cell serial
    pass resolves them."""
    rng = np.random.default_rng(12)
    counts_e = np.array([1, 64, 1, 30, 200])
    counts_g = np.array([64, 1, 1, 30, 3])
    ne, ng = int(counts_e.sum()), int(counts_g.sum())
    pm = rng.uniform(0, 2, ne)
    ux, uy, uz = plasma.isotropic(rng, ne)
    eps = plasma.log_uniform(rng, ng, 0.05, 2.0)
    vx, vy, vz = plasma.isotropic(rng, ng)
    e = {"x": pm * ux, "y": pm * uy, "z": pm * uz, "w": np.ones(ne)}
    g = {"x": eps * vx, "y": eps * vy, "z": eps * vz, "w": np.ones(ng)}
    off_e = np.concatenate([[0], np.cumsum(counts_e)]).astype(np.int64)
    off_g = np.concatenate([[0], np.cumsum(counts_g)]).astype(np.int64)
    p = plasma.Plasma("chains", e, g, off_e, off_g, 1.0, 1.0, 3)
    res = _chain_compare(ctx, orc, p, [0, 1])
    st, _, diag = res[0]
    coll_per_cell = np.bincount(diag["cell"][diag["u"] < diag["ratio"]], minlength=5)
    assert coll_per_cell[0] > 8 and coll_per_cell[1] > 8, coll_per_cell


def test_invalid_particles(ctx, orc):
    p = plasma.grid(seed=4, nx=3, ny=3, per_cell=256, dtype=np.float64)
    p.e["w"][5] = np.nan
    p.e["x"][300] = np.inf
    p.g["w"][7] = -1.0
    p.g["y"][600] = np.nan
    res = _chain_compare(ctx, orc, p, [0])
    st, gst, _ = res[0]
    assert st["n_invalid"] > 0 and gst["n_invalid"] == st["n_invalid"]


def test_empty_and_degenerate(ctx):
    import torch

    from paper_2206_02937_amd import compton

    # no cells, no particles
    p = plasma.Plasma("empty", {k: np.zeros(0) for k in "xyzw"}, {k: np.zeros(0) for k in "xyzw"},
                      np.zeros(1, dtype=np.int64), np.zeros(1, dtype=np.int64), 0.1, 1.0, 1)
    (_, _, st), = _gpu_steps(ctx, p, [0])
    assert st["n_pairs"] == 0 and st["n_collided"] == 0 and st["layout_error"] == 0
    # cells without photons, and density 0: no candidates, nothing changes
    q = plasma.grid(seed=2, nx=2, ny=2, per_cell=64, dtype=np.float64)
    q0 = plasma.Plasma("d0", _copy(q.e), _copy(q.g), q.off_e, q.off_g, q.dt, 0.0, q.seed)
    (e1, g1, st), = _gpu_steps(ctx, q0, [0])
    assert st["n_pairs"] == 0 and all(np.array_equal(e1[k], q.e[k]) for k in "xyzw")
    # a bad layout: CS_ERR_LAYOUT, nothing touched, stats flagged
    e, g, oe, og = compton.to_device(q)
    bad = oe.clone()
    bad[2] = bad[1] - 1
    buf = ctx.stats_buffer()
    with pytest.raises(RuntimeError):
        ctx.ntc_step(e, g, bad, og, q.dt, q.density_norm, q.seed, 0, stats=buf)
    torch.cuda.synchronize()
    assert _stats(buf)["layout_error"] == 1
    assert all(np.array_equal(compton.to_host(e)[k], q.e[k]) for k in "xyzw")


def test_deterministic(ctx):
    p = plasma.grid(seed=6, nx=8, ny=8, per_cell=256, dtype=np.float32)
    a = _gpu_steps(ctx, p, [0, 1])
    b = _gpu_steps(ctx, p, [0, 1])
    for (ea, ga, sa), (eb, gb, sb) in zip(a, b):
        assert all(np.array_equal(ea[k], eb[k]) and np.array_equal(ga[k], gb[k]) for k in "xyzw")
        assert sa == sb


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_full_grid_matches_oracle(ctx, orc, dtype):
    """The 128x128-cell grid (2^22 electrons and photons), one step."""
    p = plasma.grid(seed=0, nx=128, ny=128, per_cell=256, dtype=dtype)
    res = _chain_compare(ctx, orc, p, [0])
    st, gst, _ = res[0]
    assert st["n_pairs"] > 100000 and st["n_collided"] > 10000


def test_uneven_cells_match_oracle(ctx, orc):
    """Poisson cell counts with a dense bump (64 x 64 cells): the bump's cells
    draw hundreds of candidates each, so they take the tagged rounds rather
    than the in-wave path of small cells."""
    p = plasma.uneven(seed=1, side=64)
    res = _chain_compare(ctx, orc, p, [0, 1])
    st, gst, diag = res[0]
    per_cell = np.bincount(diag["cell"], minlength=p.n_cells)
    assert per_cell.max() > 64 and st["n_collided"] > 1000, (per_cell.max(), st)


def test_graph_replays_equal_eager_steps(ctx):
    """cs_ntc_graph_create: replays of the captured step (step index from
    the graph's device word, advanced by each replay) leave the particles and
    the stats record bitwise equal to eager cs_ntc_step calls with the same
    step indices, with eager work and synchronisations between the replays;
    a graph sized below the step's candidate count changes nothing and flags
    the overflow."""
    import torch

    from paper_2206_02937_amd import compton

    p = plasma.grid(seed=3, nx=128, ny=128, per_cell=256, dtype=np.float32)
    steps = [5, 6, 7]
    eager = []
    e, g, oe, og = compton.to_device(p)
    for s in steps:
        buf = ctx.stats_buffer()
        ctx.ntc_step(e, g, oe, og, p.dt, p.density_norm, p.seed, s, stats=buf)
        torch.cuda.synchronize()
        eager.append((compton.to_host(e), compton.to_host(g), compton.decode_stats(buf)))
    n_cand = max(st["n_pairs"] for _, _, st in eager)
    assert n_cand > 100000
    e, g, oe, og = compton.to_device(p)
    stats = ctx.stats_buffer()
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        gr = ctx.ntc_graph(e, g, oe, og, p.dt, p.density_norm, p.seed, n_cand + n_cand // 2, stats=stats)
        try:
            gr.set_step(steps[0])
            for k, (ee, ge, se) in enumerate(eager):
                gr.launch()
                stream.synchronize()
                st = compton.decode_stats(stats)
                print(f"  replay {k}: {st['n_pairs']} candidates, {st['n_collided']} collisions", flush=True)
                assert st == se, (st, se)
                he, hg = compton.to_host(e), compton.to_host(g)
                for key in "xyzw":
                    assert np.array_equal(he[key], ee[key]) and np.array_equal(hg[key], ge[key]), (k, key)
                torch.zeros(1 << 20, device="cuda").sum().item()  # unrelated eager work between replays
        finally:
            gr.close()
        # too small a capacity: the replay changes nothing, stats flag it
        before_e, before_g = compton.to_host(e), compton.to_host(g)
        small = ctx.ntc_graph(e, g, oe, og, p.dt, p.density_norm, p.seed, 1000, stats=stats)
        try:
            small.set_step(steps[0])
            small.launch()
            stream.synchronize()
        finally:
            small.close()
    st = compton.decode_stats(stats)
    assert st["overflow"] == 1 and st["n_pairs"] > 1000 and st["n_collided"] == 0
    he, hg = compton.to_host(e), compton.to_host(g)
    for key in "xyzw":
        assert np.array_equal(he[key], before_e[key]) and np.array_equal(hg[key], before_g[key])


def test_capacity_grows_between_calls(ctx):
    """A context that stepped a small plasma (small candidate capacity) then
    steps a larger one: the larger step overflows the capacity, changes
    nothing, and is queued again on grown scratch; the result equals a fresh
    context's."""
    import torch

    from paper_2206_02937_amd import compton

    small = plasma.grid(seed=4, nx=2, ny=2, per_cell=32, dtype=np.float32)
    big = plasma.grid(seed=4, nx=32, ny=32, per_cell=256, dtype=np.float32)
    c1 = compton.Context(0)
    c2 = compton.Context(0)
    try:
        _gpu_steps(c1, small, [0])
        a = _gpu_steps(c1, big, [0])
        b = _gpu_steps(c2, big, [0])
    finally:
        c1.close()
        c2.close()
    torch.cuda.synchronize()
    (ea, ga, sa), = a
    (eb, gb, sb), = b
    assert sa == sb and sa["n_pairs"] > 1000
    assert all(np.array_equal(ea[k], eb[k]) and np.array_equal(ga[k], gb[k]) for k in "xyzw")


def _unequal_plasma(dtype):
    rng = np.random.default_rng(21)
    counts_e = np.array([5, 0, 17, 300, 3, 1, 0, 40, 513, 1, 64])
    counts_g = np.array([9, 4, 17, 10, 3, 0, 0, 600, 2, 64, 1])
    ne, ng = int(counts_e.sum()), int(counts_g.sum())
    pm = plasma.maxwell_juttner_momentum(rng, ne, 0.5)
    ux, uy, uz = plasma.isotropic(rng, ne)
    eps = plasma.log_uniform(rng, ng, 1e-3, 1.0)
    vx, vy, vz = plasma.isotropic(rng, ng)
    e = {k: v.astype(dtype) for k, v in {"x": pm * ux, "y": pm * uy, "z": pm * uz,
                                         "w": rng.uniform(0.5, 2.0, ne)}.items()}
    g = {k: v.astype(dtype) for k, v in {"x": eps * vx, "y": eps * vy, "z": eps * vz,
                                         "w": rng.uniform(0.5, 2.0, ng)}.items()}
    off_e = np.concatenate([[0], np.cumsum(counts_e)]).astype(np.int64)
    off_g = np.concatenate([[0], np.cumsum(counts_g)]).astype(np.int64)
    return plasma.Plasma("unequal", e, g, off_e, off_g, 0.5, 0.2, 13)


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_graph_replays_on_uneven_cells_and_chains(ctx, dtype):
    """Graph replays equal eager steps where every path of the step runs:
    empty cells, cells of more than 64 candidates (tagged rounds), cells of a
    lone particle (the serial pass), unequal weights; FP32 and FP64
    storage; the capacity exactly the largest candidate count."""
    import torch

    from paper_2206_02937_amd import compton

    p = _unequal_plasma(dtype)
    steps = [0, 1, 2]
    eager = _gpu_steps(ctx, p, steps)
    n_max = max(st["n_pairs"] for _, _, st in eager)
    assert n_max > 1000
    e, g, oe, og = compton.to_device(p)
    stats = ctx.stats_buffer()
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        gr = ctx.ntc_graph(e, g, oe, og, p.dt, p.density_norm, p.seed, n_max, stats=stats)
        try:
            gr.set_step(steps[0])
            for k, (ee, ge, se) in enumerate(eager):
                gr.launch()
                stream.synchronize()
                st = _stats(stats)
                assert st == se, (k, st, se)
                he, hg = compton.to_host(e), compton.to_host(g)
                for key in "xyzw":
                    assert np.array_equal(he[key], ee[key], equal_nan=True), (k, key)
                    assert np.array_equal(hg[key], ge[key], equal_nan=True), (k, key)
        finally:
            gr.close()


def test_graph_layout_errors(ctx):
    """A graph over offsets that are not a valid layout changes nothing and
    flags its stats record on every replay; creation refuses particles
    without cells and a capacity outside [1, 2^31 - 2]."""
    import torch

    from paper_2206_02937_amd import compton

    q = plasma.grid(seed=2, nx=2, ny=2, per_cell=64, dtype=np.float64)
    e, g, oe, og = compton.to_device(q)
    bad = oe.clone()
    bad[2] = bad[1] - 1
    stats = ctx.stats_buffer()
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        gr = ctx.ntc_graph(e, g, bad, og, q.dt, q.density_norm, q.seed, 4096, stats=stats)
        try:
            for _ in range(2):
                gr.launch()
                stream.synchronize()
                st = _stats(stats)
                assert st["layout_error"] == 1 and st["n_pairs"] == 0
        finally:
            gr.close()
        assert all(np.array_equal(compton.to_host(e)[k], q.e[k]) for k in "xyzw")
        for cap in (0, 1 << 31):
            with pytest.raises(RuntimeError):
                ctx.ntc_graph(e, g, oe, og, q.dt, q.density_norm, q.seed, cap, stats=stats)
        no_cells = torch.zeros(1, dtype=torch.int64, device="cuda")
        with pytest.raises(RuntimeError):
            ctx.ntc_graph(e, g, no_cells, no_cells, q.dt, q.density_norm, q.seed, 16, stats=stats)


def test_too_many_candidates(ctx):
    """A cell whose expected candidate count N_e N_g P_max reaches 2^31 - 1
    (2^16 x 2^16 particles, P_max = 2): the call fails with
    CS_ERR_UNSUPPORTED before any candidate is drawn, no particle changes,
    and the stats record is flagged (overflow = 1, n_pairs = 2^31 - 1)."""
    import torch

    from paper_2206_02937_amd import compton

    rng = np.random.default_rng(31)
    n = 1 << 16
    ux, uy, uz = plasma.isotropic(rng, n)
    vx, vy, vz = plasma.isotropic(rng, n)
    e = {"x": (2 * ux).astype(np.float32), "y": (2 * uy).astype(np.float32), "z": (2 * uz).astype(np.float32),
         "w": np.ones(n, np.float32)}
    g = {"x": (0.1 * vx).astype(np.float32), "y": (0.1 * vy).astype(np.float32),
         "z": (0.1 * vz).astype(np.float32), "w": np.ones(n, np.float32)}
    off = np.array([0, n], dtype=np.int64)
    p = plasma.Plasma("too_many", e, g, off, off.copy(), 1.0, 1.0, 3)
    de, dg, oe, og = compton.to_device(p)
    buf = ctx.stats_buffer()
    with pytest.raises(RuntimeError) as info:
        ctx.ntc_step(de, dg, oe, og, p.dt, p.density_norm, p.seed, 0, stats=buf)
    assert "candidates" in str(info.value)
    torch.cuda.synchronize()
    st = compton.decode_stats(buf)
    assert st["overflow"] == 1 and st["n_pairs"] == (1 << 31) - 1 and st["n_collided"] == 0
    assert all(np.array_equal(compton.to_host(de)[k], e[k]) for k in "xyzw")
    assert all(np.array_equal(compton.to_host(dg)[k], g[k]) for k in "xyzw")


def _cells_plasma(counts_e, counts_g, f, seed, heavy=1.0):
    """Cells of the given counts with N_e N_g f candidates on average; with
    heavy > 1 the first electron of each cell carries that weight, so that
    the other pairs are accepted with 1 / heavy of the probability (chains of
    many candidates, few collisions)."""
    rng = np.random.default_rng(seed)
    counts_e, counts_g = np.asarray(counts_e), np.asarray(counts_g)
    ne, ng = int(counts_e.sum()), int(counts_g.sum())
    pm = rng.uniform(0, 2, ne)
    ux, uy, uz = plasma.isotropic(rng, ne)
    eps = plasma.log_uniform(rng, ng, 0.05, 2.0)
    vx, vy, vz = plasma.isotropic(rng, ng)
    off_e = np.concatenate([[0], np.cumsum(counts_e)]).astype(np.int64)
    off_g = np.concatenate([[0], np.cumsum(counts_g)]).astype(np.int64)
    w = np.ones(ne)
    w[off_e[:-1][counts_e > 0]] = heavy
    e = {"x": pm * ux, "y": pm * uy, "z": pm * uz, "w": w}
    g = {"x": eps * vx, "y": eps * vy, "z": eps * vz, "w": np.ones(ng)}
    return plasma.Plasma("cells", e, g, off_e, off_g, 0.5, f / heavy, seed)


@pytest.mark.parametrize("kind", ["limit", "chains", "sparse", "mixed", "dense", "pieces"])
def test_cells_at_the_limits_of_the_window(ctx, orc, kind):
    """Cells that fill a window exactly and by one too many, chains as long as
    both, single cells among thousands of empty ones, cells of 0 .. 200
    candidates side by side, cells with several windows of candidates left
    after the parallel rounds, and counts around a piece and a workgroup of
    the scan.  Tolerance: the module's for FP64 storage."""
    rng = np.random.default_rng(17)
    if kind == "limit":
        p = _cells_plasma([16, 257, 15, 16, 2], [16, 1, 17, 16, 3], 1.0, 21, heavy=16.0)
        want = [256, 257, 255, 256, 6]
    elif kind == "chains":
        p = _cells_plasma([1, 256, 1, 300], [256, 1, 257, 1], 1.0, 22, heavy=32.0)
        want = [256, 256, 257, 300]
        p.e["w"][:] = np.where(p.e["w"] > 1, 1.0, p.e["w"])  # unit weights, and one heavy photon in each cell
        p.g["w"][p.off_g[:-1]] = 32.0
    elif kind == "sparse":
        n = np.zeros(5000, dtype=int)
        n[[0, 1023, 1024, 2500, 4999]] = [4, 5, 6, 1, 3]
        p, want = _cells_plasma(n, n, 1.0, 23), n * n
    elif kind == "mixed":
        p = _cells_plasma(rng.integers(0, 30, 3000), rng.integers(0, 30, 3000), 0.25, 24, heavy=4.0)
        want = None
    elif kind == "dense":
        p, want = _cells_plasma([40] * 30, [40] * 30, 0.5, 25, heavy=16.0), [800] * 30
    else:
        n = np.tile([1, 2, 3], 700)[:2049]
        p, want = _cells_plasma(n, n, 1.0, 26), n * n
    (st, gst, diag), = _chain_compare(ctx, orc, p, [0])
    per_cell = np.bincount(diag["cell"], minlength=p.off_e.size - 1)
    if want is not None:
        assert np.array_equal(per_cell, want)
    else:
        assert per_cell.max() > 150 and (per_cell == 0).any()
    assert st["n_collided"] > 0
