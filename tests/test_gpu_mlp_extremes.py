"""FP32 inference with activations far outside those of a trained network:
infinite, huge and NaN pre-activations give what SiLU(z) = z / (1 + e^-z) in
FP32 gives (z above, 0 below, NaN for NaN), and the samples beside such a one
keep their bits."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

H = 64


@pytest.fixture(scope="module")
def ctx():
    from paper_2206_02937_amd import compton

    c = compton.Context(0)
    yield c
    c.close()


def _chain(z, b2):
    """A network of one neuron per layer: SiLU(z), plus b2, then as it is
    (weights of 1); outputs that and its half.  Every sum has one term that is
    not zero, so it is exact."""
    p = np.zeros(12802, np.float32)
    p[128] = z
    p[192], p[192 + 4096] = 1.0, b2
    p[4352] = p[8512] = 1.0
    p[12672], p[12672 + H] = 1.0, 0.5
    return p


def _all_ones(w1u, b1):
    """z = w1u (2u - 1) + b1 in every neuron, every other weight 1 / 64."""
    p = np.full(12802, 1.0 / H, np.float32)
    p[0:2 * H:2], p[1:2 * H:2], p[2 * H:3 * H] = 0.0, w1u, b1
    for b in (4288, 8448, 12608):
        p[b:b + H] = 0.0
    p[-2:] = 0.0
    return p


def _forward(ctx, params, x, u):
    import torch

    from paper_2206_02937_amd import compton

    net = compton.MLP(ctx, params)
    y = net.forward(torch.from_numpy(x).cuda(), torch.from_numpy(u).cuda(), "mlp_f32").cpu().numpy()
    mu = net.sample(torch.from_numpy(x).cuda(), torch.from_numpy(u).cuda(), "mlp_f32")[0].cpu().numpy()
    net.close()
    return y, mu


@pytest.mark.parametrize("z, want", [(-3e38, 0.0), (-1e30, 0.0), (-1e20, 0.0), (-200.0, 0.0), (-89.0, 0.0),
                                     (-88.5, 0.0), (-87.2, 0.0), (87.5, 87.5), (88.5, 88.5), (200.0, 200.0),
                                     (1e30, 1e30), (2e35, 2e35)])
def test_large_pre_activations(ctx, z, want):
    """z in the first layer, plus 128 in the second, which the layers after
    it leave as it is."""
    y, _ = _forward(ctx, _chain(z, 128.0), np.full(200, 0.5, np.float32), np.full(200, 0.5, np.float32))
    want = np.float32(want) + np.float32(128.0)
    assert np.all(y[:, 0] == want) and np.all(y[:, 1] == want / 2)


def test_infinite_and_nan_pre_activations(ctx):
    x, u = np.full(70, 0.5, np.float32), np.full(70, 0.9375, np.float32)
    y, mu = _forward(ctx, _all_ones(3e38, 3e38), x, u)  # z = 3e38 (1 + 0.875): infinite
    assert np.all(np.isposinf(y)) and np.all(mu == 1.0)
    y, _ = _forward(ctx, _all_ones(0.0, np.nan), x, u)
    assert np.all(np.isnan(y))


@pytest.mark.parametrize("which", [0, 17, 40, 63, 64])
def test_neighbours_keep_their_bits(ctx, which):
    """One sample of a wave with an infinite pre-activation."""
    rng = np.random.default_rng(3)
    p = np.concatenate([rng.uniform(-0.3, 0.3, 12802)]).astype(np.float32)
    p[1:2 * H:2] = 2e38  # weights of 2u - 1: z is infinite at u = 2, 0 times them at u = 1/2
    x = np.exp(rng.uniform(np.log(1e-4), np.log(1e2), 130)).astype(np.float32)
    u = np.full(130, 0.5, np.float32)
    base, _ = _forward(ctx, p, x, u)
    assert np.all(np.isfinite(base))
    u[which] = 2.0
    y, _ = _forward(ctx, p, x, u)
    keep = np.arange(130) != which
    assert np.array_equal(y[keep].view(np.uint32), base[keep].view(np.uint32))
