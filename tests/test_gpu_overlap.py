"""The class launches of a build overlap on side streams of its context, forked
from the caller's stream and joined to it again: on streams of the caller's, on
two contexts at once, under capture, and from the first build of a context on,
whichever entry point makes it."""

import ctypes

import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = 1e-11   # FP64 sums in another order


def _density(n, seed):
    A = np.random.default_rng(seed).standard_normal((n, n))
    return torch.tensor(0.5 * (A + A.T), dtype=torch.float64, device="cuda")


def _context(n, seed, **kw):
    from paper_2510_24968_amd import fsim
    ctx = fsim.Context(synth.water_cluster(n, seed), tau=1e-10, **kw)
    ctx.schwarz_screen()
    return ctx


def test_first_build_without_allocation_overlaps_in_a_callers_graph():
    """The first build of a context, captured by its caller: the launches are
    branches of the graph (a chain has one edge less than nodes), and every
    replay gives F of the density it finds."""
    from paper_2510_24968_amd import fsim
    L = fsim.lib()
    ctx = _context(3, 2)
    D, F = _density(ctx.nbf, 1), torch.zeros(ctx.nbf, ctx.nbf, dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    st = torch.cuda.Stream()
    handle = ctypes.c_void_p(st.cuda_stream)
    graph, gexec = ctypes.c_void_p(), ctypes.c_void_p()
    nodes, edges = ctypes.c_size_t(), ctypes.c_size_t()
    with torch.cuda.stream(st):
        assert L.hipStreamBeginCapture(handle, 1) == 0          # thread-local
        ctx.fock_build_noalloc(D, F, energy=False)
        assert L.hipStreamEndCapture(handle, ctypes.byref(graph)) == 0
    assert L.hipGraphGetNodes(graph, None, ctypes.byref(nodes)) == 0
    assert L.hipGraphGetEdges(graph, None, None, ctypes.byref(edges)) == 0
    print(f"[gpu] captured build: {nodes.value} nodes, {edges.value} edges", flush=True)
    assert edges.value > nodes.value - 1
    assert L.hipGraphInstantiate(ctypes.byref(gexec), graph, None, None, ctypes.c_size_t(0)) == 0
    for seed in (2, 3, 4):
        D.copy_(_density(ctx.nbf, seed))
        F.fill_(float("nan"))
        torch.cuda.synchronize()
        assert L.hipGraphLaunch(gexec, handle) == 0
        torch.cuda.synchronize()
        ref = ctx.fock_build(D)["F"]                            # eager work between the replays
        torch.cuda.synchronize()
        assert (F - ref).abs().max().item() < TOL
    assert L.hipGraphExecDestroy(gexec) == 0 and L.hipGraphDestroy(graph) == 0
    ctx.close()


def test_two_contexts_on_two_streams():
    """Builds of two contexts enqueued in turn on two streams, outputs
    overwritten by the next round without a wait in between."""
    ctxs = [_context(3, 2), _context(4, 5, tau_fp32=1e-5)]
    Ds = [[_density(c.nbf, 10 * k + r) for r in range(3)] for k, c in enumerate(ctxs)]
    refs = [[c.fock_build(d, want_jk=True) for d in ds] for c, ds in zip(ctxs, Ds)]
    streams = [torch.cuda.Stream() for _ in ctxs]
    outs = [[None] * 3 for _ in ctxs]
    torch.cuda.synchronize()
    for r in range(3):
        for k, c in enumerate(ctxs):
            with torch.cuda.stream(streams[k]):
                # a density made, used and freed on this stream
                d = Ds[k][r] * 1.0
                outs[k][r] = c.fock_build(d, want_jk=True, energy=False)
                del d
    torch.cuda.synchronize()
    for k in range(2):
        for r in range(3):
            for x in ("F", "J", "K"):
                err = (outs[k][r][x] - refs[k][r][x]).abs().max().item()
                assert err < TOL, (k, r, x, err)
    for c in ctxs:
        c.close()
