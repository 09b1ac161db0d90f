"""The plain sampler at the ends of its inputs: at infinite x the photon goes
backwards without energy (the limit of eps'/eps = 1 / (1 + x (1 - mu))), and a NaN
stays one, in either storage type and whichever samples stand beside."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_infinite_and_nan_x(dtype):
    import torch

    from paper_2206_02937_amd import compton

    ctx = compton.Context(0)
    rng = np.random.default_rng(9)
    x = np.exp(rng.uniform(np.log(1e-8), np.log(1e3), 1000)).astype(dtype)
    u = rng.random(1000).astype(dtype)
    base = [t.cpu().numpy() for t in ctx.sample_plain(torch.from_numpy(x).cuda(), torch.from_numpy(u).cuda())]
    inf, nan = np.arange(3, 1000, 100), np.arange(64, 1000, 100)
    x[inf], x[nan] = np.inf, np.nan
    x[5] = np.finfo(dtype).max if dtype == np.float32 else 1e100
    u[5] = 0.5
    mu, r = [t.cpu().numpy() for t in ctx.sample_plain(torch.from_numpy(x).cuda(), torch.from_numpy(u).cuda())]
    ctx.close()
    assert np.all(r[inf] == 0.0) and np.all(mu[inf] == -1.0)
    assert np.all(np.isnan(r[nan]))
    assert 0.0 < r[5] < 1e-3 and mu[5] == 1.0
    same = np.setdiff1d(np.arange(1000), np.concatenate([inf, nan, [5]]))
    assert np.array_equal(mu[same], base[0][same]) and np.array_equal(r[same], base[1][same])
