"""gw_find_mu against the oracle's bisection in every form the search takes:
matrices inverted a wave each or (nao > 32) a workgroup each, and many, a few or
one value of mu per launch; metals and gaps."""
import numpy as np
import pytest

from oracle import grids as og
from oracle import gw as ogw

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to("cuda")


# values of mu per launch, of a tree and of a way ahead: 15 / 15, 7 / 15, 3 / 15, 1 / 15 and 1 / 1
@pytest.mark.parametrize("nao,nk,ntau", [(5, 3, 20), (8, 25, 40), (12, 30, 40), (20, 30, 40), (26, 30, 40), (33, 2, 12),
                                         (60, 1, 12)])
@pytest.mark.parametrize("gap", [False, True])
def test_forms(nao, nk, ntau, gap):
    from paper_2206_07660_amd import gw
    beta = 0.8 * ntau
    rng = np.random.default_rng([nao, nk])
    U = np.linalg.qr(rng.normal(size=(nk, nao, nao)) + 1j * rng.normal(size=(nk, nao, nao)))[0]
    e = rng.uniform(-1.0, 1.0, (nk, nao))
    occ = (nao + 1) // 2
    if gap:
        e = np.where(np.arange(nao) < occ, -0.6 + 0.3 * e, 0.6 + 0.3 * e)
    H0 = (U * e[:, None, :]) @ U.conj().transpose(0, 2, 1)
    S = np.tile(np.eye(nao, dtype=complex), (nk, 1, 1))
    # a fraction of a level above the gap's filling, so that the root is where the count rises
    target = 2.0 * occ + (0.02 if gap else 0.0) - (nao % 2 if not gap else 0)
    g = og.Grids(beta, ntau)
    zero_w = np.zeros((len(g.nF),) + H0.shape, complex)
    ref, _, n_ref = ogw.find_mu(H0, S, np.zeros_like(H0), zero_w, target, g, 2, mu0=0.1)
    ctx = gw.Context((nk, 1, 1), nao, 4, ntau, beta)
    try:
        G = torch.empty(ctx.giw_shape(), dtype=torch.complex128, device="cuda")
        mu, n = gw.gw_find_mu(ctx, dev(H0), dev(S), None, None, target, 0.1, G_iw=G)
        # both counts are within some 1e-12 of each other (sums of nw nk nao terms of order one times
        # their weights); the count rises by more than 0.1 per Ha at the root
        assert abs(n - target) < 1e-10
        assert abs(n_ref - target) < 1e-10
        assert abs(mu - ref) < 1e-9
        # the same from another start: the bracket differs, the root does not
        mu2, _ = gw.gw_find_mu(ctx, dev(H0), dev(S), None, None, target, -0.4, G_iw=G)
        assert abs(mu2 - mu) < 1e-9
    finally:
        ctx.close()


# 48, 960, 4320 and 17280 matrices of order 8: 15 / 15, 7 / 15, 3 / 15 and 1 / 1 values of mu per launch
@pytest.mark.parametrize("mesh", [(2, 1, 1), (40, 1, 1), (12, 15, 1), (24, 30, 1)])
@pytest.mark.parametrize("seed,mu0", [(8, 0.0), (32, 0.1), (39, 0.0)])
def test_count_that_falls(mesh, seed, mu0):
    """24 nodes at beta 1000: in the gap the count of the sparse grids is not
    monotonic in mu, and which of its roots is the answer depends on the
    midpoints that the bisection visits."""
    from paper_2206_07660_amd import gw
    beta, ntau, nao = 1000.0, 24, 8
    rng = np.random.default_rng([seed, 2])
    e = np.where(np.arange(nao) < 4, -0.6, 0.6) + 0.3 * rng.uniform(-1, 1, (2, nao))
    g = og.Grids(beta, ntau)
    r = np.asarray(g.w) @ g.TFp

    def excess(mu):
        return -np.real(r * (1.0 / (1j * g.wF[:, None, None] + mu - e)).sum((1, 2))).sum() - 8.0

    lo, hi = mu0 - 1.0, mu0 + 1.0
    assert excess(lo) < 0 < excess(hi)
    while hi - lo > 1e-13:
        mid = 0.5 * (lo + hi)
        x = excess(mid)
        # the decisions are clear of the counts' rounding, some 1e-12
        assert hi - lo < 1e-7 or abs(x) > 1e-8
        lo, hi = (mid, hi) if x < 0 else (lo, mid)
    ctx = gw.Context(mesh, nao, 4, ntau, beta)
    try:
        H0 = np.zeros((ctx.nk, nao, nao), complex)
        H0[:, np.arange(nao), np.arange(nao)] = np.tile(e, (ctx.nk // 2, 1))
        S = np.tile(np.eye(nao, dtype=complex), (ctx.nk, 1, 1))
        mu, _ = gw.gw_find_mu(ctx, dev(H0), dev(S), None, None, 8.0, mu0)
        # the count rises by more than 10 per Ha at the root
        assert abs(mu - 0.5 * (lo + hi)) < 1e-8
    finally:
        ctx.close()


@pytest.mark.parametrize("pole,needed", [(0.0, True), (0.5, True), (0.75, False), (-0.75, False)])
def test_zero_pivot(pole, needed):
    """A matrix that is singular at one value of mu: an error where the
    bisection asks for that count, and none where it is only looked at ahead."""
    from paper_2206_07660_amd import gw
    beta, ntau, nao, at = 20.0, 20, 3, 10
    g = og.Grids(beta, ntau)
    r = np.asarray(g.w) @ g.TFp
    ctx = gw.Context((1, 1, 1), nao, 4, ntau, beta)
    try:
        # diag(i w + mu - 0.4, i w + mu + 0.3, i w + mu - pole), the last one mu - pole at one frequency
        w = (2.0 * ctx.grids["nF"] + 1.0) * np.pi / beta
        sig = np.zeros((len(w), 1, nao, nao), complex)
        sig[at, 0, 2, 2] = 1j * w[at]
        e = np.array([0.4, -0.3, pole])
        x = 1j * w[:, None] - e - sig[:, 0, np.arange(3), np.arange(3)]
        lo, hi, asked = -1.0, 1.0, False
        while hi - lo > 1e-13 and not asked:
            mid = 0.5 * (lo + hi)
            asked = mid == pole
            if not asked:
                lo, hi = (mid, hi) if -2.0 * np.real(r[:, None] / (x + mid)).sum() < 2.5 else (lo, mid)
        assert asked == needed
        a = (dev(np.diag(e).astype(complex)[None]), dev(np.eye(nao, dtype=complex)[None]), None, dev(sig), 2.5, 0.0)
        if needed:
            with pytest.raises(gw.GwError) as err:
                gw.gw_find_mu(ctx, *a)
            assert err.value.status == gw.GW_ERR_SINGULAR
        else:
            # the count rises by seven per Ha there
            assert abs(gw.gw_find_mu(ctx, *a)[0] - 0.5 * (lo + hi)) < 1e-10
    finally:
        ctx.close()
