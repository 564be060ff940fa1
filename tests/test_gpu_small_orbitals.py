"""Products L V R of one to four orbitals (a thread per row of the product)
and of five (matrix instructions), around the widths of their workgroups:
polarization, written and accumulated, and the self-energy adjoint, which takes
L^H, against the oracle and the general adjoint identity."""
import numpy as np
import pytest

from paper_2206_07660_amd import inputs as inp
from oracle import gw as ogw

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

EPS = 2.3e-16


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to("cuda")


@pytest.mark.parametrize("nao,naux,mesh,chunk", [
    (1, 1, (1, 1, 1), 2), (1, 64, (2, 1, 1), 3), (1, 257, (3, 1, 1), 4), (2, 31, (2, 1, 1), 4), (2, 33, (1, 1, 1), 1),
    (2, 129, (2, 1, 1), 3), (3, 21, (2, 1, 1), 4), (3, 22, (3, 1, 1), 2), (3, 86, (1, 1, 1), 4), (4, 16, (2, 1, 1), 3),
    (4, 17, (1, 1, 1), 4), (4, 65, (3, 1, 1), 4), (5, 13, (2, 1, 1), 4),
])
def test_products(nao, naux, mesh, chunk):
    from paper_2206_07660_amd import gw
    ntau = 4
    wl = inp.small_workload(name="few", mesh=mesh, nao=nao, naux=naux, ntau=ntau, beta=5.0, seed=41, n_target=0.5)
    V = inp.make_V(wl)
    rng = np.random.default_rng(19)
    cg = lambda *s: inp.circular_gaussian(rng, s, 0.3)
    Ga, Gb, Sb = (cg(ntau, wl.nk, nao, nao) for _ in range(3))
    Pt, Pd = cg(wl.nk, ntau, naux, naux), cg(wl.nk, ntau, naux, naux)
    pol = lambda v, g: ogw.polarization(v, g, mesh, wl.ns)
    # K nao^2 products per entry, each within a few eps of the moduli's
    tol = 4 * wl.nk * nao ** 4 * EPS * np.abs(pol(np.abs(V) + 0j, np.abs(Ga) + np.abs(Gb) + 0j)).max() + 1e-300
    ref = pol(V, Ga)
    two = pol(V, Ga + Gb) - ref - pol(V, Gb)
    ctx = gw.Context(mesh, nao, naux, ntau, 5.0, ns=wl.ns, tau_chunk=chunk)
    z = dict(dtype=torch.complex128, device="cuda")
    try:
        dV, da, db, dS, dP = dev(V), dev(Ga), dev(Gb), dev(Sb), dev(Pt)
        P = torch.full(ref.shape, float("nan"), **z)
        gw.gw_polarization(ctx, dV, da, 0, wl.nk, P)
        assert np.abs(P.cpu().numpy() - ref).max() < tol
        gw.gw_polarization2(ctx, dV, da, db, 0, wl.nk, P)
        gw.gw_polarization2(ctx, dV, db, da, 0, wl.nk, P, accumulate=True)
        assert np.abs(P.cpu().numpy() - two).max() < 4 * tol
        # <Sbar, SE[dP, G]> = <Pbar, dP>
        gb, Pb = torch.zeros(ctx.g_shape(), **z), torch.full(ref.shape, float("nan"), **z)
        gw.gw_self_energy_vjp(ctx, dV, da, dP, dS, 0, wl.nk, gb, Pb)
        se = ogw.self_energy(V, Ga, Pd, mesh)
        lhs, rhs = np.vdot(Sb, se), np.vdot(Pb.cpu().numpy(), Pd)
        bound = np.abs(Sb).sum() * 4 * wl.nk * naux * nao ** 2 * EPS * \
            np.abs(ogw.self_energy(np.abs(V) + 0j, np.abs(Ga) + 0j, np.abs(Pd) + 0j, mesh)).max()
        assert abs(lhs - rhs) < bound + 1e-300
    finally:
        ctx.close()
