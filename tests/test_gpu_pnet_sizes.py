"""The probability network's forward at the sizes where it changes between its two
ways of reading the parameters: every pair's output has the bits that a small
batch gives it, and nothing is written past the last."""
import numpy as np
import pytest

from oracle import pnet_oracle as N

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 257, 3 << 17, (3 << 17) + 1, 1 << 19, 1 << 20, (1 << 20) + 1])
@pytest.mark.parametrize("shift", [0, 1])
def test_forward_bits_do_not_depend_on_the_batch(n, shift):
    import torch

    from paper_2206_02937_amd import compton

    ctx = compton.Context(0)
    rng = np.random.default_rng(7)
    params = torch.from_numpy(N.glorot_uniform(rng).astype(np.float32)).cuda()
    gen = torch.Generator(device="cuda").manual_seed(n)
    flat = torch.randn(9 * n + shift, generator=gen, device="cuda")
    x = flat[shift:].view(n, 9)  # (rows of 36 bytes: no more than 4-byte aligned)
    y = torch.full((n + 64,), -1.0, device="cuda")
    ctx.pnet_forward(params, x, y[:n])
    ref = torch.cat([ctx.pnet_forward(params, x[a:a + (1 << 17)]) for a in range(0, n, 1 << 17)])
    torch.cuda.synchronize()
    assert torch.equal(y[:n], ref) and bool((y[n:] == -1.0).all())
    want = N.forward(params.cpu().numpy().astype(np.float64), x[-1000:].cpu().numpy().astype(np.float64))
    assert np.max(np.abs(y[:n][-1000:].cpu().numpy() - want)) <= 1e-5
    ctx.close()
