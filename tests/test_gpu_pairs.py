"""Pairs of q-points: P0^{-q}(beta - tau) = P0^q(tau)^T, so a range of
q-points that holds both q and -q contracts one of them and transposes.
Ranges that split pairs, self-inverse q, the Hermitian mode and node chunks,
at matrix sizes around the 32 x 32 tiles of the transposing kernel, against
the oracle and against one call per q (which cannot pair q != -q)."""
import numpy as np
import pytest

from paper_2206_07660_amd import inputs as inp
from oracle import grids as og
from oracle import gw as ogw

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# sums of at most Nk nao^2 = 96 products in fp64, both sides: 96 eps of the
# largest entry, with a margin of 10
REL = 96 * 2.3e-16 * 10


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to("cuda")


def make(mesh, nao, naux, ntau):
    wl = inp.small_workload(name="pairs", mesh=mesh, nao=nao, naux=naux, ntau=ntau, beta=10.0, seed=53,
                            n_target=float(nao))
    g = og.Grids(wl.beta, wl.ntau)
    H0, S, V = inp.make_H0(wl), inp.make_S(wl), inp.make_V(wl)
    return wl, g, H0, S, V


@pytest.mark.parametrize("mesh,nao,naux,ntau,chunk", [
    ((3, 1, 2), 4, 1, 2, 2),       # one-entry matrices, the fewest nodes
    ((3, 1, 2), 4, 31, 8, 3),      # node chunks that do not divide the half range
    ((2, 2, 1), 3, 32, 6, 6),      # every q = -q
    ((5, 1, 1), 4, 33, 8, 5),      # only q = 0 is its own inverse
])
@pytest.mark.parametrize("herm", [False, True])
def test_polarization_pairs(mesh, nao, naux, ntau, chunk, herm):
    from paper_2206_07660_amd import gw
    wl, g, H0, S, V = make(mesh, nao, naux, ntau)
    rng = np.random.default_rng(5)
    G = inp.random_hermitian_tau(rng, ntau, wl.nk, nao, 0.3)
    if not herm:
        G = G + inp.circular_gaussian(rng, G.shape, 0.1)
    ref = ogw.polarization(V, G, wl.mesh, wl.ns)
    tol = REL * np.abs(ref).max()
    ctx = gw.Context(wl.mesh, nao, naux, ntau, wl.beta, ns=wl.ns, tau_chunk=chunk)
    try:
        gw.gw_set_hermitian(ctx, herm)
        dV, dG = dev(V), dev(G)
        for q0, nq in ((0, wl.nk), (1, wl.nk - 1), (0, wl.nk - 1), (wl.nk - 1, 1)):
            P = torch.full((nq, ntau, naux, naux), float("nan"), dtype=torch.complex128, device="cuda")
            gw.gw_polarization(ctx, dV, dG, q0, nq, P)
            one = torch.full((1, ntau, naux, naux), float("nan"), dtype=torch.complex128, device="cuda")
            for q in range(q0, q0 + nq):
                gw.gw_polarization(ctx, dV, dG, q, 1, one)
                assert np.abs(P[q - q0].cpu().numpy() - ref[q]).max() < tol
                assert (P[q - q0] - one[0]).abs().max().item() < tol
    finally:
        ctx.close()
