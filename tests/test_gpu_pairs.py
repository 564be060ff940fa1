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


@pytest.mark.parametrize("mesh,nao,naux,ntau,chunk", [
    ((3, 1, 2), 4, 31, 8, 3),
    ((2, 2, 1), 3, 32, 6, 6),
    ((5, 1, 1), 4, 33, 8, 5),
    ((1, 1, 1), 5, 7, 2, 1),
])
def test_self_energy_pairs(mesh, nao, naux, ntau, chunk):
    """gw_sigma and gw_sigma_jvp of a Hermitian G: the pair {q, -q} from the
    long contraction of q, against the oracle and against the general mode."""
    from paper_2206_07660_amd import gw
    wl, g, H0, S, V = make(mesh, nao, naux, ntau)
    G = ogw.g0_tau(H0, S, 0.03, wl.beta, g.tau)
    r_inf, r_tau, _ = ogw.sigma_evaluation(V, G, g, wl.mesh, wl.ns)
    # the tolerance of every fp64 comparison with the oracle
    tol = 1e-10
    rng = np.random.default_rng(6)
    dG = dev(inp.random_hermitian_tau(rng, ntau, wl.nk, nao, 0.2))
    ctx = gw.Context(wl.mesh, nao, naux, ntau, wl.beta, ns=wl.ns, tau_chunk=chunk)
    z = dict(dtype=torch.complex128, device="cuda")
    nan = lambda shape: torch.full(shape, float("nan"), **z)
    try:
        dV, dG0 = dev(V), dev(G)
        got = {}
        for herm in (False, True):
            gw.gw_set_hermitian(ctx, herm, two_slot=herm)
            pt, pw, p0 = nan((wl.nk, ntau, naux, naux)), nan((wl.nk, ctx.nw_b, naux, naux)), nan((wl.nk, ctx.nw_b, naux, naux))
            si, st = nan(ctx.k_shape()), nan(ctx.g_shape())
            phi = gw.gw_sigma(ctx, dV, dG0, si, st, P_tau=pt, P0_iw=p0, Pt_iw=pw, want_phi=True)
            si2, st2 = nan(ctx.k_shape()), nan(ctx.g_shape())
            phi2 = gw.gw_sigma(ctx, dV, dG0, si2, st2, want_phi=True)
            for a, b in ((si, st), (si2, st2)):
                assert np.abs(a.cpu().numpy() - r_inf).max() < tol
                assert np.abs(b.cpu().numpy() - r_tau).max() < tol
            assert abs(phi - phi2) < tol
            j = [nan(ctx.k_shape()), nan(ctx.g_shape())]
            gw.gw_sigma_jvp(ctx, dV, dG0, pt, pw, dG, *j)
            jq = [nan(ctx.k_shape()), nan(ctx.g_shape())]
            gw.gw_sigma_jvp(ctx, dV, dG0, None, None, dG, *jq)
            got[herm] = (phi, j, jq)
        assert abs(got[True][0] - got[False][0]) < tol
        for a, b in zip(got[True][1] + got[True][2], got[False][1] + got[False][1]):
            assert (a - b).abs().max().item() < tol
    finally:
        ctx.close()


def test_sigma_per_q_of_a_general_G():
    """q by q without the Hermitian mode: P0^{-q} is still the transpose of P0^q."""
    from paper_2206_07660_amd import gw
    wl, g, H0, S, V = make((3, 1, 2), 3, 17, 6)
    rng = np.random.default_rng(7)
    G = inp.circular_gaussian(rng, (6, wl.nk, 3, 3), 0.2)
    r_inf, r_tau, _ = ogw.sigma_evaluation(V, G, g, wl.mesh, wl.ns)
    ctx = gw.Context(wl.mesh, 3, 17, 6, wl.beta, ns=wl.ns, tau_chunk=4)
    try:
        si = torch.empty(ctx.k_shape(), dtype=torch.complex128, device="cuda")
        st = torch.empty(ctx.g_shape(), dtype=torch.complex128, device="cuda")
        gw.gw_sigma(ctx, dev(V), dev(G), si, st)
        assert np.abs(si.cpu().numpy() - r_inf).max() < 1e-10
        assert np.abs(st.cpu().numpy() - r_tau).max() < 1e-10
    finally:
        ctx.close()
