"""Which way the no-time-counter step takes a cell: one wave up to a number of
candidates that falls with the cell count, the kernels of the large cells
beyond, queued before or after the counts are known; and the largest weight of
cells far longer than the average.  Against the FP64 oracle element by element,
with the metric and tolerances of the no-time-counter tests."""
import numpy as np
import pytest

from paper_2206_02937_amd import plasma
from tests.test_gpu_ntc import _cells_plasma, _chain_compare, _gpu_steps, ctx  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_cells, local", [(7, 64), (8, 128), (639, 128), (640, 192), (1279, 192), (1280, 256)])
def test_cells_at_the_limit(ctx, orc, n_cells, local):  # noqa: F811
    """Cells of exactly the limit, one candidate fewer and one more (unit
    probability bound: N_e N_g candidates), and small ones around them."""
    ne, ng = np.full(n_cells, 2), np.full(n_cells, 3)
    at = [0, n_cells // 2, n_cells - 1]
    ne[at[0]], ng[at[0]] = 8, local // 8
    ne[at[1]], ng[at[1]] = 1, local - 1
    ne[at[2]], ng[at[2]] = 1, local + 1
    p = _cells_plasma(ne, ng, 1.0, 31 + n_cells, heavy=4.0)
    for st, gst, diag in _chain_compare(ctx, orc, p, [0, 1]):
        assert np.array_equal(np.bincount(diag["cell"], minlength=n_cells), ne * ng)
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
