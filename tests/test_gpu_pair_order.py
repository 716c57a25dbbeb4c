"""The pair-ordered density and J' half-sums of the Fock build against the
oracle: elements of dropped shell pairs, one and several molecules, private
and shared accumulators, and the pairs of a partly filled last tile.

J and K elements sum at most a few 1e4 integrals of order one here, each
within 1e-12 of the oracle's in FP64 at worst and a few ulp typically:
1e-11 absolute, as in the other parity tests."""

import numpy as np
import pytest

import oracle
import synth
from helpers import spd_molecule

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = 1e-11


def _apart(basis, shift):
    """Two copies of a molecule shift bohr apart along x: at a loose
    threshold every pair between them is dropped."""
    n, ns = len(basis["Z"]), len(basis["shell_l"])
    b = dict(basis)
    b["xyz"] = np.concatenate([basis["xyz"], basis["xyz"] + [shift, 0.0, 0.0]])
    b["Z"] = np.tile(basis["Z"], 2)
    b["shell_atom"] = np.concatenate([basis["shell_atom"], basis["shell_atom"] + n]).astype(np.int32)
    for k in ("shell_l", "shell_nprim", "shell_prim0"):
        b[k] = np.tile(basis[k], 2)
    b["nelec"] = 2 * basis["nelec"]
    assert len(b["shell_l"]) == 2 * ns
    return b


def _density(n, seed):
    a = np.random.default_rng(seed).standard_normal((n, n))
    return 0.5 * (a + a.T)


@pytest.mark.parametrize("private", [True, False])
def test_dropped_pairs_and_private_copies(private):
    from paper_2510_24968_amd import fsim
    b = _apart(spd_molecule(), 60.0)
    B = oracle.Basis(b)
    tau = 1e-9
    D = _density(B.nbf, 3)
    Jo, Ko = B.fock_jk(D, tau=tau)
    ctx = fsim.Context(b, tau=tau)
    ctx.set_xcd_private(private)
    _, st = ctx.schwarz_screen()
    assert st["pairs_kept"] < st["shell_pairs"]
    Dd = torch.tensor(D, device="cuda")
    h = B.nbf // 2
    for _ in range(2):
        r = ctx.fock_build(Dd, want_jk=True)
        J, K = r["J"].cpu().numpy(), r["K"].cpu().numpy()
        assert np.max(np.abs(J - Jo)) < TOL and np.max(np.abs(K - Ko)) < TOL
        assert np.all(J[:h, h:] == 0.0) and np.all(J[h:, :h] == 0.0)
    F = torch.empty_like(Dd)
    Jn, Kn = torch.empty_like(Dd), torch.empty_like(Dd)
    ctx.fock_build_noalloc(Dd, F, Jn, Kn)
    assert np.max(np.abs(Jn.cpu().numpy() - Jo)) < TOL
    assert np.max(np.abs(Kn.cpu().numpy() - Ko)) < TOL
    # a second screen with every pair kept replaces the maps
    ctx.schwarz_screen(0.0)
    Jo, Ko = B.fock_jk(D)
    r = ctx.fock_build(Dd, want_jk=True)
    assert np.max(np.abs(r["J"].cpu().numpy() - Jo)) < TOL
    assert np.max(np.abs(r["K"].cpu().numpy() - Ko)) < TOL
    ctx.close()


def test_batch_of_unequal_molecules():
    from paper_2510_24968_amd import fsim
    mols = [spd_molecule(), synth.water_cluster(1, 3), synth.ch_molecule(4_000_005),
            _apart(spd_molecule(), 60.0)]
    tau = 1e-9
    bt = fsim.Batch(mols, tau=tau)
    bt.schwarz_screen()
    Bs = [oracle.Basis(b) for b in mols]
    Ds = [_density(B.nbf, 10 + k) for k, B in enumerate(Bs)]
    r = bt.fock_build(bt.pack([torch.tensor(d, device="cuda") for d in Ds]), want_jk=True)
    for B, D, J, K in zip(Bs, Ds, bt.unpack(r["J"]), bt.unpack(r["K"])):
        Jo, Ko = B.fock_jk(D, tau=tau)
        assert np.max(np.abs(J.cpu().numpy() - Jo)) < TOL
        assert np.max(np.abs(K.cpu().numpy() - Ko)) < TOL
    bt.close()
