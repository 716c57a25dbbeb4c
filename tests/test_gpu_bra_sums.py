"""Bras of the ket-outer kernel whose components come from sums over powers of
A - B: both functions on one centre, along an axis, close and far, and the
molecule off the origin, where P - A loses digits to the coordinates.

Per contracted integral 1e-12 in FP64, as for the other kernels; FP32 tiles
2e-5 relative to the largest element."""

import itertools

import numpy as np
import pytest

import oracle
from helpers import custom_basis

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SHELLS = [(0, [6.0, 0.9, 0.2], [0.2, 0.5, 0.4]), (1, [4.0, 0.7], [0.3, 0.8]),
          (1, [0.25], [1.0])]


@pytest.mark.parametrize("sep", [(0.0, 0.0, 1e-3), (0.0, 1.4, 0.0), (-1.1, 0.3, 0.9),
                                 (3.0, -4.0, 5.0)])
@pytest.mark.parametrize("origin", [0.0, 40.0])
def test_bra_sums(sep, origin):
    from paper_2510_24968_amd import fsim
    at = lambda v: [origin + x for x in v]
    # the close centres carry different shells: no linear dependence
    b = custom_basis([(at((0.0, 0.0, 0.0)), 2.0, SHELLS),
                      (at(sep), 2.0, [(0, [2.5, 0.5], [0.4, 0.6]), (1, [1.7, 0.45], [0.5, 0.6])]),
                      (at((0.5, 2.0, -1.5)), 2.0, [(0, [0.8], [1.0]), (1, [0.6], [1.0])])],
                     nelec=6, name=f"sep {sep} origin {origin}")
    ctx = fsim.Context(b)
    ctx.set_all_variants(4, 4)
    B = oracle.Basis(b)
    # every pair with a p function as the bra, kets over all classes
    pairs = [(i, j) for i, j in itertools.product(range(7), repeat=2) if i >= j]
    qs = [p + k for p in pairs if p[0] in (1, 2, 4, 6) or p[1] in (1, 2, 4, 6) for k in pairs[::3]]
    ref = [B.eri_block(*q) for q in qs]
    for prec in ("fp64", "mixed"):
        got = ctx.eri_quartets(qs, prec)
        worst = max(float(np.max(np.abs(g - r))) for g, r in zip(got, ref))
        scale = max(1.0, max(float(np.max(np.abs(r))) for r in ref))
        print(f"{b['name']} {prec}: max |dERI| {worst:.2e}", flush=True)
        assert worst < (1e-12 if prec == "fp64" else 2e-5 * scale)
    ctx.close()
