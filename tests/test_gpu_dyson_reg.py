"""The register-resident Dyson inversion at matrix sizes around its lane
layouts, with pivots that force row interchanges, against numpy; the
electron-count search against a plain bisection of the same counts, also where
the count is flat in mu."""
import numpy as np
import pytest

from oracle import grids as og
from oracle import gw as ogw

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to("cuda")


def system(nao, nk, seed, gap):
    rng = np.random.default_rng(seed)
    z = rng.normal(size=(nk, nao, nao)) + 1j * rng.normal(size=(nk, nao, nao))
    U = np.linalg.qr(z)[0]
    e = rng.uniform(-1.0, 1.0, (nk, nao))
    if gap:
        e = np.where(np.arange(nao) < (nao + 1) // 2, -3.0 + 0.2 * e, 3.0 + 0.2 * e)
    H0 = (U * e[:, None, :]) @ U.conj().transpose(0, 2, 1)
    B = 0.1 * (rng.normal(size=(nk, nao, nao)) + 1j * rng.normal(size=(nk, nao, nao)))
    S = np.eye(nao) + 0.2 / nao * (B + B.conj().transpose(0, 2, 1))
    return H0, S


@pytest.mark.parametrize("nao", [1, 2, 7, 8, 9, 12, 13, 16, 17, 20, 21, 26, 27, 32, 33])
def test_inverse(nao):
    from paper_2206_07660_amd import gw
    nk, ntau, beta = 3, 8, 8.0
    H0, S = system(nao, nk, nao, False)
    # a zero leading entry in every matrix but the frequency's: rows must move
    S[:, 0, 0] = 0.0
    H0[:, 0, 0] = 0.0
    ctx = gw.Context((nk, 1, 1), nao, 4, ntau, beta)
    try:
        G = torch.empty(ctx.giw_shape(), dtype=torch.complex128, device="cuda")
        w = (2 * ctx.grids["nF"] + 1) * np.pi / beta
        M = (1j * w[:, None, None, None] + 0.3) * S - H0
        if nao == 1:
            M = M + 1.0
            H0 = H0 - 1.0
        gw.gw_dyson_G(ctx, dev(H0), dev(S), None, None, 0.3, G)
        g = G.cpu().numpy()
        # residual of a pivoted elimination: n^2 eps of |M| |G|
        bound = 8 * nao ** 2 * 2.3e-16 * (np.abs(M) @ np.abs(g)).max()
        assert np.abs(M @ g - np.eye(nao)).max() < bound
    finally:
        ctx.close()


@pytest.mark.parametrize("nao,nk,ntau,gap", [(6, 4, 20, False), (26, 2, 40, False), (17, 3, 30, False), (5, 2, 20, True)])
def test_search_is_the_bisection(nao, nk, ntau, gap):
    from paper_2206_07660_amd import gw
    beta = float(ntau)
    H0, S = system(nao, nk, 3 * nao, gap)
    g = og.Grids(beta, ntau)
    target = float(nao) if not gap else 2.0 * ((nao + 1) // 2)
    zero, zero_w = np.zeros_like(H0), np.zeros((len(g.nF),) + H0.shape, complex)
    ctx = gw.Context((nk, 1, 1), nao, 4, ntau, beta)
    try:
        dH, dS = dev(H0), dev(S)
        G = torch.empty(ctx.giw_shape(), dtype=torch.complex128, device="cuda")
        for mu0 in (0.0, 0.7, -2.5):
            mu, n = gw.gw_find_mu(ctx, dH, dS, None, None, target, mu0, G_iw=G)
            ref = ogw.find_mu(H0, S, zero, zero_w, target, g, 2, mu0=mu0)[0]
            assert abs(n - target) < 1e-9
            if gap:
                # flat count: the midpoints' rounding decides, any mu of the gap will do
                assert -2.8 < mu < 2.8
            else:
                # the two counts differ by rounding, over a slope of at least one per Ha
                assert abs(mu - ref) < 1e-10
    finally:
        ctx.close()
