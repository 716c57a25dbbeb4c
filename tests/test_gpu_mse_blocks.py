"""fsim_mse over its block counts: one per 256 values up to 128 blocks, then one
per 9216 values up to 1536.  Whole numbers and a mean over a power of two, whose
float32 sums are exact in any order."""

import ctypes

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SHARE = 256 * 36


@pytest.mark.parametrize("n", [1, 255, 32767, 32769, 128 * SHARE - 1, 129 * SHARE + 1,
                               1536 * SHARE - 1, 1537 * SHARE + 5])
def test_loss_and_gradient_are_exact(n):
    from paper_2510_24968_amd import guess
    g = torch.Generator().manual_seed(n % 1000)
    Y = torch.randint(-1, 2, (n,), generator=g).float().cuda()
    T = torch.randint(-1, 2, (n,), generator=g).float().cuda()
    # a quarter of the values, so that the sum stays below 2^24
    M = (torch.randint(0, 4, (n,), generator=g) == 0).float().cuda()
    dY, loss = torch.full_like(Y, float("nan")), torch.zeros(1, device="cuda")
    inv = 2.0 ** -20
    assert guess._lib().fsim_mse(n, *(guess._p(t) for t in (Y, T, M)), ctypes.c_float(inv),
                                 guess._p(dY), guess._p(loss), guess._stream()) == 0
    d = M * (Y - T)
    total = int((d.double() ** 2).sum().item())
    assert total < 2 ** 24
    assert loss.item() == total * inv
    assert torch.equal(dY, 2.0 * d * inv)
