"""fsim_gemm_bf16 where its 16-byte loads may not be used: operands that start
or step off a vector boundary, and sizes around its 64-wide tiles and stages;
fsim_bias_grad around its 512-row splits and 32-column blocks.

Against float64 results of the same values: K 2^-23 (|A| |B|), the rounding of
K float32 additions, and likewise n 2^-23 sum |dY| for the column sums."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _bits(x):
    return x.to(torch.bfloat16).view(torch.int16)


@pytest.mark.parametrize("off,pad", [(0, 0), (1, 0), (4, 3), (8, 8)])
@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
def test_offsets_and_pitches(off, pad, ta, tb):
    from paper_2510_24968_amd import guess
    g = torch.Generator().manual_seed(off + 10 * pad + 100 * ta + 200 * tb)
    for M, N, K, ks in [(1, 1, 1, 1), (63, 65, 64, 1), (64, 64, 63, 1), (65, 36, 129, 1),
                        (130, 72, 200, 3), (8, 200, 1000, 16)]:
        ra, ca = (K, M) if ta else (M, K)
        rb, cb = (N, K) if tb else (K, N)
        A = _bits(torch.randn(off + ra * (ca + pad) + 8, generator=g)).cuda()
        B = _bits(torch.randn(off + rb * (cb + pad) + 8, generator=g)).cuda()
        C = torch.zeros(M, N, dtype=torch.float32, device="cuda")
        guess.GuessNet.gemm(M, N, K, A[off:], ca + pad, ta, B[off:], cb + pad, tb, C=C, ksplit=ks)
        view = lambda t, r, c: t[off:off + r * (c + pad)].view(torch.bfloat16).view(r, c + pad)[
            :, :c].double().cpu()
        a, b = view(A, ra, ca), view(B, rb, cb)
        a, b = (a.T if ta else a), (b.T if tb else b)
        ref = (a @ b).numpy()
        bound = K * 2.0 ** -23 * (a.abs() @ b.abs()).numpy() + 1e-30
        err = np.abs(C.double().cpu().numpy() - ref)
        assert np.all(err <= bound), (M, N, K, ks, float((err / bound).max()))


@pytest.mark.parametrize("n", [1, 127, 128, 511, 512, 513, 5000])
def test_column_sums(n):
    import ctypes
    from paper_2510_24968_amd import guess
    for m in (1, 31, 33, 256):
        g = torch.Generator().manual_seed(n + m)
        dY = torch.randn(n, m, generator=g)
        db = torch.full((m,), float("nan"), dtype=torch.float32, device="cuda")
        d = dY.cuda()
        ptr = lambda t: ctypes.c_void_p(t.data_ptr())
        s = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
        assert guess._lib().fsim_bias_grad(n, m, ptr(d), ptr(db), s) == 0
        err = (db.double().cpu() - dY.double().sum(0)).abs()
        assert torch.all(err <= n * 2.0 ** -23 * dY.double().abs().sum(0) + 1e-30), (n, m)
