"""Which way the no-time-counter step takes a cell: one wave up to 64 candidates,
the kernels of the large cells beyond 256, queued before or after the counts are
known, and between the two by the cells that there are; and the largest weight of
cells far longer than the average.  Against the FP64 oracle element by element,
with the metric and tolerances of the no-time-counter tests."""
import numpy as np
import pytest

from paper_2206_02937_amd import plasma
from tests.test_gpu_ntc import _cells_plasma, _chain_compare, _gpu_steps, ctx  # noqa: F401

pytestmark = pytest.mark.gpu


def _products(want):
    """(N_e, N_g) with the given products, neither larger than need be (1 and 0
    for 0)."""
    ne = np.array([max(d for d in range(1, max(2, int(w ** 0.5) + 1)) if w % d == 0) for w in want])
    return ne, np.asarray(want) // ne


@pytest.mark.parametrize("n_cells, n_mid, most", [(7, 2, 100), (8, 2, 128), (8, 2, 129), (700, 0, 0), (700, 639, 128),
                                                 (700, 639, 129), (700, 639, 256), (700, 640, 256),
                                                 (700, 3, 257), (639, 3, 257), (639, 0, 300), (90, 40, 129),
                                                 (3000, 700, 257)])
def test_cells_at_the_limits(ctx, orc, n_cells, n_mid, most):  # noqa: F811
    """Cells of 64 candidates and of one more, and n_mid cells in all between
    there and 256, the densest cell with `most` (unit probability bound: N_e N_g
    candidates): the ways that the middle cells go by their number, by the
    densest among them, by a denser one, and with few cells."""
    rng = np.random.default_rng(n_cells + n_mid + most)
    want = rng.integers(1, 12, n_cells)
    cells = rng.permutation(n_cells)
    want[cells[:n_mid]] = rng.integers(65, min(most, 128) + 1, n_mid) if n_mid else 0
    if n_mid:
        want[cells[0]] = 65
    if most > 64:
        want[cells[1 if most <= 256 else n_mid]] = most
    want[cells[-1]] = 64
    want[cells[-3:-1]] = 0  # (cells without one of the species)
    ne, ng = _products(want)
    p = _cells_plasma(ne, ng, 1.0, 31 + n_cells, heavy=4.0)
    for st, gst, diag in _chain_compare(ctx, orc, p, [0, 1]):
        per_cell = np.bincount(diag["cell"], minlength=n_cells)
        assert np.array_equal(per_cell, want) and np.sum((per_cell > 64) & (per_cell <= 256)) == n_mid
        assert st["n_collided"] > 0


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("n_cells, where", [(197, 0), (197, 77), (197, 196), (196, 195), (199, 198), (198, 196)])
def test_largest_weight_of_long_cells(ctx, orc, dtype, n_cells, where):  # noqa: F811
    """Cells of 2 and one of 511 to 3000 (16 lanes share out a cell, the whole
    wave a long one, also in the last wave, which has fewer cells): its one heavy
    particle, anywhere in it, sets its bound."""
    for n_long, heavy_at, species in ((511, 510, "e"), (512, 0, "g"), (3000, 2999, "e"), (2950, 1234, "g")):
        n = np.full(n_cells, 2)
        n[where] = n_long
        p = _cells_plasma(n, n, 0.002, 5)
        w = p.e["w"] if species == "e" else p.g["w"]
        w[p.off_e[where] + heavy_at] = 8.0
        for d in (p.e, p.g):
            for k in d:
                d[k] = d[k].astype(dtype)
        assert n.sum() <= 32 * n_cells
        (st, gst, diag), = _chain_compare(ctx, orc, p, [3])
        want = 0.002 * 8.0 * n_long ** 2
        assert abs(np.sum(diag["cell"] == where) - want) <= 1.0


def test_large_cells_come_and_go():
    """A context that meets steps with large cells, without, with more
    candidates than it has room for, and with an invalid layout in between:
    each as on a context of its own."""
    import torch

    from paper_2206_02937_amd import compton

    small = _cells_plasma([3] * 20, [4] * 20, 0.9, 41, heavy=4.0)
    dense = _cells_plasma([30] * 12, [20] * 12, 0.9, 42, heavy=4.0)
    denser = _cells_plasma([90] * 40, [80] * 40, 0.9, 43, heavy=4.0)
    shared = compton.Context(0)
    try:
        for p in (dense, small, small, denser, dense, "bad", dense, small):
            if p == "bad":
                e, g, oe, og = compton.to_device(dense)
                with pytest.raises(RuntimeError):
                    shared.ntc_step(e, g, oe.flip(0).contiguous(), og, 1.0, 1.0, 1, 0)
                torch.cuda.synchronize()
                assert all(np.array_equal(compton.to_host(e)[k], dense.e[k]) for k in "xyzw")
                continue
            own = compton.Context(0)
            try:
                (ea, ga, sa), = _gpu_steps(shared, p, [2])
                (eb, gb, sb), = _gpu_steps(own, p, [2])
            finally:
                own.close()
            assert sa == sb and sa["n_collided"] > 0
            assert all(np.array_equal(ea[k], eb[k]) and np.array_equal(ga[k], gb[k]) for k in "xyzw")
    finally:
        shared.close()
