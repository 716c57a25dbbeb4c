"""fsim_bias_grad and fsim_bias_grad_ws sum every column in a fixed order, so
equal inputs give equal bits: around the 256 row lanes, the blocks of 16 and 32
columns, the runs of 1024 rows and the 2048 rows from which runs are used."""

import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

ONE_PASS, SPLIT = 2048, 1024


def _lane_sums(x):
    """float32: partial sums of rows r, r + 256, ..., then a tree of the 256."""
    s = np.zeros((256, x.shape[1]), np.float32)
    for i in range(0, len(x), 256):
        s[:min(256, len(x) - i)] += x[i:i + 256]
    o = 128
    while o:
        s[:o] += s[o:2 * o]
        o //= 2
    return s[0]


def _in_runs(x):
    return _lane_sums(np.stack([_lane_sums(x[i:i + SPLIT]) for i in range(0, len(x), SPLIT)]))


def _ptr(t):
    return ctypes.c_void_p(t.data_ptr() if t is not None else None)


@pytest.mark.parametrize("n", [1, 255, 257, 1023, 1025, 2047, 2048, 2049, 8192, 33000])
def test_order_of_the_sums(n):
    from paper_2510_24968_amd import guess
    L, s = guess._lib(), ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    for m in (1, 15, 17, 31, 33, 36, 256):
        x = torch.randn(n, m, generator=torch.Generator().manual_seed(n + m))
        d, h = x.cuda(), x.numpy()
        ws = torch.full((-(-n // SPLIT), m), float("nan"), device="cuda")
        for w, ref in ((None, _lane_sums(h)), (ws, _in_runs(h) if n > ONE_PASS else _lane_sums(h))):
            for _ in range(3):
                db = torch.full((m,), float("nan"), device="cuda")
                assert L.fsim_bias_grad_ws(n, m, _ptr(d), _ptr(db), _ptr(w), s) == 0
                assert np.array_equal(db.cpu().numpy(), ref), (n, m, w is None)
        db = torch.full((m,), float("nan"), device="cuda")
        assert L.fsim_bias_grad(n, m, _ptr(d), _ptr(db), s) == 0
        assert np.array_equal(db.cpu().numpy(), _lane_sums(h)), (n, m)


@pytest.mark.parametrize("n", [513, 5000, 20001])
def test_every_row_counts_once(n):
    """Whole numbers, whose float32 sums are exact in any order."""
    from paper_2510_24968_amd import guess
    L, s = guess._lib(), ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    x = torch.randint(-8, 9, (n, 33), generator=torch.Generator().manual_seed(n))
    d, db = x.float().cuda(), torch.empty(33, device="cuda")
    ws = torch.empty(-(-n // SPLIT), 33, device="cuda")
    for w in (None, ws):
        assert L.fsim_bias_grad_ws(n, 33, _ptr(d), _ptr(db), _ptr(w), s) == 0
        assert torch.equal(db.cpu().long(), x.sum(0))


def test_bias_gradients_repeat():
    """The last layer's, whose input repeats bit for bit, and all of them from
    their own inputs: a training batch gives the same bias gradients again."""
    from paper_2510_24968_amd import guess
    net = guess.GuessNet(seed=1)
    g = torch.Generator().manual_seed(2)
    n = 20000
    X = net.to_bf16(torch.randn(n, 64, generator=g).cuda())
    T = torch.randn(n, 36, generator=g).cuda()
    M = (torch.rand(n, 36, generator=g) < 0.6).float().cuda()
    first = net.gradients(X, T, M)[2]
    for _ in range(3):
        assert all(torch.equal(a, b) for a, b in zip(first, net.gradients(X, T, M)[2]))
