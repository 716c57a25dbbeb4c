"""Segment launches of few tiles, which share each tile out over chunks, ket
primitives, bra primitives and blocks: from one quartet to past the number of
tiles where sharing ends, with 1 to 8 primitives per shell, in every lane
variant, against the oracle.

J and K within 1e-11 in FP64 (as the other parity tests); all-FP32 builds
within 1e-6 of their largest element (each integral to 2e-5 of its size, and
they add up incoherently)."""

import numpy as np
import pytest

import oracle
import synth
from helpers import custom_basis, spd_molecule

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _contracted(k, lmax):
    """Two atoms with shells of k primitives each."""
    ex = [0.2 * 2.1 ** i for i in range(k)]
    co = [0.3 + 0.1 * i for i in range(k)]
    sh = [(l, [e * (1.0 + 0.1 * l) for e in ex], co) for l in range(lmax + 1)]
    return custom_basis([([0.0, 0.0, 0.0], 3.0, sh), ([1.1, -0.7, 1.9], 3.0, sh)], nelec=6,
                        name=f"{k} primitives, l <= {lmax}")


MOLECULES = {
    "one_function": lambda: custom_basis([([0.0, 0.0, 0.0], 2.0, [(0, [1.0], [1.0])])], nelec=2),
    "h2": lambda: synth.h_chain(2, 1.4),
    "h32": lambda: synth.h_chain(32, 1.4),
    "spd": spd_molecule,
    "one_primitive": lambda: _contracted(1, 2),
    "two_primitives": lambda: _contracted(2, 2),
    "eight_primitives": lambda: _contracted(8, 2),
    "water1": lambda: synth.water_cluster(1, 5),
    "water5": lambda: synth.water_cluster(5, 5),
}


@pytest.mark.parametrize("name", sorted(MOLECULES))
def test_shared_tiles_match_oracle(name):
    from paper_2510_24968_amd import fsim
    b = MOLECULES[name]()
    B = oracle.Basis(b)
    tau = 1e-12
    a = np.random.default_rng(7).standard_normal((B.nbf, B.nbf))
    D = 0.5 * (a + a.T)
    Jo, Ko = B.fock_jk(D, tau=tau)
    Dd = torch.tensor(D, device="cuda")
    for tau32, prec in ((0.0, "fp64"), (1e3, "mixed")):
        ctx = fsim.Context(b, tau=tau, tau_fp32=tau32)
        ctx.schwarz_screen()
        scale = 1e-11 if prec == "fp64" else None
        for variant in (None, 0, 1, 2, 4, 5):
            if variant is not None:
                ctx.set_all_variants(variant, 8)
            r = ctx.fock_build(Dd, prec, want_jk=True)
            dJ = np.max(np.abs(r["J"].cpu().numpy() - Jo))
            dK = np.max(np.abs(r["K"].cpu().numpy() - Ko))
            print(f"{name} {prec} variant {variant}: |dJ| {dJ:.2e} |dK| {dK:.2e}", flush=True)
            assert dJ < (scale or 1e-6 * np.max(np.abs(Jo))), (name, prec, variant)
            assert dK < (scale or 1e-6 * np.max(np.abs(Ko))), (name, prec, variant)
        ctx.close()
