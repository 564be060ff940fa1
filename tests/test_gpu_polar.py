"""The block-wise long contraction of the polarization against the oracle:
matrix sizes around its 16-wide blocks, workgroup shapes (1, 2, 4 and 8
waves), parts and superblocks; K sums that are not multiples of 4 or 8 and that
straddle k-points; full and Hermitian matrices, written and accumulated."""
import numpy as np
import pytest

from paper_2206_07660_amd import inputs as inp
from oracle import gw as ogw

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

EPS = 2.3e-16


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to("cuda")


@pytest.mark.parametrize("herm", [False, True])
@pytest.mark.parametrize("naux,nao,mesh,chunk", [
    (16, 2, (3, 1, 1), 4), (17, 3, (3, 1, 1), 3), (33, 2, (1, 1, 1), 1), (48, 3, (2, 1, 1), 4), (49, 4, (2, 1, 1), 3),
    (65, 5, (1, 1, 1), 4), (96, 2, (2, 1, 1), 4), (97, 4, (1, 1, 1), 4), (113, 3, (2, 1, 1), 4), (150, 6, (2, 1, 1), 4),
    (256, 4, (1, 1, 1), 4), (257, 3, (2, 1, 1), 4), (300, 5, (1, 1, 1), 2),
])
def test_blocks(naux, nao, mesh, chunk, herm):
    from paper_2206_07660_amd import gw
    ntau = 4
    wl = inp.small_workload(name="polar", mesh=mesh, nao=nao, naux=naux, ntau=ntau, beta=5.0, seed=37, n_target=1.0)
    V = inp.make_V(wl)
    rng = np.random.default_rng(13)
    Ga, Gb = (inp.random_hermitian_tau(rng, ntau, wl.nk, nao, 0.3) if herm else
              inp.circular_gaussian(rng, (ntau, wl.nk, nao, nao), 0.3) for _ in range(2))
    # K nao^2 products per entry, each within a few eps of the moduli's
    tol = 4 * wl.nk * nao ** 4 * EPS * np.abs(ogw.polarization(np.abs(V) + 0j, np.abs(Ga) + np.abs(Gb) + 0j, mesh,
                                                               wl.ns)).max()
    ref = ogw.polarization(V, Ga, mesh, wl.ns)
    # bilinear in the two slots: P[a + b] - P[a] - P[b] = P[a, b] + P[b, a]
    two = ogw.polarization(V, Ga + Gb, mesh, wl.ns) - ref - ogw.polarization(V, Gb, mesh, wl.ns)
    ctx = gw.Context(mesh, nao, naux, ntau, 5.0, ns=wl.ns, tau_chunk=chunk)
    try:
        gw.gw_set_hermitian(ctx, herm, two_slot=herm)
        dV, da, db = dev(V), dev(Ga), dev(Gb)
        P = torch.full(ref.shape, float("nan"), dtype=torch.complex128, device="cuda")
        gw.gw_polarization(ctx, dV, da, 0, wl.nk, P)
        assert np.abs(P.cpu().numpy() - ref).max() < tol
        P.fill_(float("nan"))
        gw.gw_polarization2(ctx, dV, da, db, 0, wl.nk, P)
        gw.gw_polarization2(ctx, dV, db, da, 0, wl.nk, P, accumulate=True)
        assert np.abs(P.cpu().numpy() - two).max() < 4 * tol
    finally:
        ctx.close()
