"""fsim_gemm_bf16 where its 16-byte loads may not be used: operands that start
or step off a vector boundary, and sizes around its 64-wide tiles and stages.

Against a float64 product of the same BF16 values: K 2^-23 (|A| |B|), the
rounding of K float32 additions."""

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
