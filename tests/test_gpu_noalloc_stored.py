"""fsim_fock_build_noalloc on a context with stored integrals: the store holds
FP64 blocks in the tile order of the unsplit quartet lists, so a request for
mixed precision digests those too."""

import numpy as np
import pytest

import synth
from helpers import spd_molecule

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("which,tau,tau_fp32", [("spd", 0.0, 1e-2), ("water3", 1e-10, 1e-5)])
def test_noalloc_mixed_digests_the_store(which, tau, tau_fp32):
    """J, K, F and E equal the direct FP64 build's up to the order of the
    FP64 sums (1e-11, as for the stored build itself)."""
    from paper_2510_24968_amd import fsim
    b = spd_molecule() if which == "spd" else synth.water_cluster(3, 2)
    print(f"[gpu] noalloc over a store, {which}", flush=True)
    ctx = fsim.Context(b, tau=tau, tau_fp32=tau_fp32)
    ctx.schwarz_screen()
    A = np.random.default_rng(3).standard_normal((ctx.nbf, ctx.nbf))
    D = torch.tensor(0.5 * (A + A.T), dtype=torch.float64, device="cuda")
    ref = ctx.fock_build(D, "fp64", want_jk=True)
    assert ctx.store_eris() > 0
    for prec in ("fp64", "mixed"):
        F, J, K = (torch.full_like(D, float("nan")) for _ in range(3))
        E = ctx.fock_build_noalloc(D, F, J, K, prec)
        for name, x in (("J", J), ("K", K), ("F", F)):
            err = (x - ref[name]).abs().max().item()
            print(f"  {prec} |d{name}| {err:.2e}", flush=True)
            assert err < 1e-11, (prec, name)
        assert abs(E - ref["E_elec"]) < 1e-9
    ctx.close()
