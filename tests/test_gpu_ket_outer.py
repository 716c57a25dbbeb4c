"""The ket-outer kernel's integrals against the oracle where its tables meet:
Boys arguments on both sides of the grid's end of every order, primitive
pairs whose common factor underflows, d components' norms.

Per contracted integral 1e-12 in FP64, as for the other kernels; FP32 tiles
2e-5 relative to the largest element, their documented accuracy."""

import itertools

import numpy as np
import pytest

import oracle
from helpers import custom_basis

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _check(basis, quartets):
    from paper_2510_24968_amd import fsim
    ctx = fsim.Context(basis)
    ctx.set_all_variants(4, 4)
    B = oracle.Basis(basis)
    ref = [B.eri_block(*q) for q in quartets]
    for prec in ("fp64", "mixed"):
        got = ctx.eri_quartets(quartets, prec)
        worst = max(float(np.max(np.abs(g - r))) for g, r in zip(got, ref))
        scale = max(1.0, max(float(np.max(np.abs(r))) for r in ref))
        print(f"{basis['name']} {prec}: max |dERI| {worst:.2e}", flush=True)
        assert worst < (1e-12 if prec == "fp64" else 2e-5 * scale)
    ctx.close()


@pytest.mark.parametrize("l", [0, 1, 2])
def test_boys_grid_ends(l):
    """Two centres with single primitives of exponent 1 (alpha = 1 for a
    quartet between them): T = R^2 steps through every order's grid end
    (36 to 52 for these classes) in steps of about 0.35."""
    for T in np.concatenate([np.linspace(35.4, 53.0, 50), [2.0, 9.7, 99.9, 100.1, 1e4]]):
        sh = lambda x: [(k, [1.0], [1.0]) for k in range(x + 1)]
        b = custom_basis([([0.0, 0.0, 0.0], 2.0, sh(l)),
                          ([0.6 * np.sqrt(T), 0.0, 0.8 * np.sqrt(T)], 2.0, sh(l))],
                         nelec=2, name=f"T={T:.2f}")
        n = l + 1
        q = [(a, bb, n + c, n + d) for a in range(n) for bb in range(a + 1)
             for c in range(n) for d in range(c + 1)]
        _check(b, [x for x in q if sum(min(v % n, 2) for v in x) <= 5])


def test_underflowing_pairs_and_norms():
    """Tight primitives far apart (their product factor is exactly zero) in
    one contraction with diffuse ones, s, p and d shells."""
    b = custom_basis([
        ([0.0, 0.0, 0.0], 4.0, [(0, [900.0, 0.2], [0.5, 0.5]), (1, [700.0, 0.3], [0.4, 0.6]),
                                (2, [500.0, 0.4], [0.3, 0.7])]),
        ([6.0, -1.0, 2.0], 2.0, [(0, [800.0, 0.15], [0.5, 0.5]), (1, [0.25], [1.0]),
                                 (2, [0.5], [1.0])]),
    ], nelec=6, name="underflow")
    qs = [q for q in itertools.product(range(6), repeat=4) if q[0] != q[1]][::5]
    _check(b, qs)
