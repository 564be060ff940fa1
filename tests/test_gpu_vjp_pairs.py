"""gw_sigma_vjp with one polarization adjoint per {q, -q}: against the adjoint
identity <s, J dG> = <J^H s, dG> with the forward derivative, and the Hermitian
mode and the q-by-q mode against the general stored one; meshes with and
without self-inverse q, node chunks that do not divide the half range."""
import numpy as np
import pytest

from paper_2206_07660_amd import inputs as inp
from oracle import grids as og
from oracle import gw as ogw

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to("cuda")


@pytest.mark.parametrize("mesh,nao,naux,ntau,chunk", [((3, 1, 2), 4, 31, 8, 3), ((2, 2, 1), 3, 33, 6, 6),
                                                      ((5, 1, 1), 1, 7, 4, 4), ((1, 1, 1), 5, 17, 2, 1)])
def test_adjoint(mesh, nao, naux, ntau, chunk):
    from paper_2206_07660_amd import gw
    wl = inp.small_workload(name="vjp", mesh=mesh, nao=nao, naux=naux, ntau=ntau, beta=10.0, seed=61, n_target=0.5)
    g = og.Grids(wl.beta, ntau)
    H0, S, V = inp.make_H0(wl), inp.make_S(wl), inp.make_V(wl)
    rng = np.random.default_rng(17)
    dV, dG0 = dev(V), dev(ogw.g0_tau(H0, S, 0.03, wl.beta, g.tau))
    cg = lambda *shape: dev(inp.circular_gaussian(rng, shape, 1.0))
    dG, sb, tb = cg(ntau, wl.nk, nao, nao), cg(wl.nk, nao, nao), cg(ntau, wl.nk, nao, nao)
    z = dict(dtype=torch.complex128, device="cuda")
    nan = lambda shape: torch.full(shape, float("nan"), **z)
    ctx = gw.Context(mesh, nao, naux, ntau, wl.beta, ns=wl.ns, tau_chunk=chunk)
    try:
        gw.gw_set_hermitian(ctx, False)
        pt, pw = nan((wl.nk, ntau, naux, naux)), nan((wl.nk, ctx.nw_b, naux, naux))
        si, st = nan(ctx.k_shape()), nan(ctx.g_shape())
        gw.gw_sigma(ctx, dV, dG0, si, st, P_tau=pt, P0_iw=torch.empty_like(pw), Pt_iw=pw)
        out = {}
        for herm in (False, True):
            for stored in (True, False):
                gw.gw_set_hermitian(ctx, herm)
                gb = nan(ctx.g_shape())
                gw.gw_sigma_vjp(ctx, dV, dG0, pt if stored else None, pw if stored else None, sb, tb, gb)
                out[herm, stored] = gb
        gw.gw_set_hermitian(ctx, False)
        gw.gw_sigma_jvp(ctx, dV, dG0, pt, pw, dG, si, st)
        ip = lambda a, b: complex((a.conj() * b).sum().item())
        lhs, rhs = ip(sb, si) + ip(tb, st), ip(out[False, True], dG)
        # sums of ntau nk nao^2 products of size one times the fp64 comparison bound
        assert abs(lhs - rhs) < 1e-10 * ntau * wl.nk * nao * nao * max(1.0, out[False, True].abs().max().item())
        for k, v in out.items():
            assert (v - out[False, True]).abs().max().item() < 1e-10 * max(1.0, v.abs().max().item()), k
    finally:
        ctx.close()
