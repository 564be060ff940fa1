"""gw_sigma_vjp with a given P~ of a G that is not Hermitian: GW_HERM_FORWARD
speaks of the G that a polarization is formed from, and none is formed there."""
import numpy as np
import pytest

from paper_2206_07660_amd import inputs as inp
from oracle import grids as og

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to("cuda")


@pytest.mark.parametrize("mesh,nao,naux,ntau,chunk", [((3, 1, 2), 4, 17, 8, 3), ((2, 1, 1), 3, 33, 6, 6)])
def test_given_polarization(mesh, nao, naux, ntau, chunk):
    from paper_2206_07660_amd import gw
    wl = inp.small_workload(name="vjpg", mesh=mesh, nao=nao, naux=naux, ntau=ntau, beta=10.0, seed=71, n_target=0.5)
    rng = np.random.default_rng(23)
    cg = lambda *shape: dev(inp.circular_gaussian(rng, shape, 0.3))
    dV, G = dev(inp.make_V(wl)), cg(ntau, wl.nk, nao, nao)
    dG, sb, tb = cg(ntau, wl.nk, nao, nao), cg(wl.nk, nao, nao), cg(ntau, wl.nk, nao, nao)
    z = dict(dtype=torch.complex128, device="cuda")
    ctx = gw.Context(mesh, nao, naux, ntau, wl.beta, ns=wl.ns, tau_chunk=chunk)
    try:
        gw.gw_set_hermitian(ctx, False)
        pt, pw = torch.empty((wl.nk, ntau, naux, naux), **z), torch.empty((wl.nk, ctx.nw_b, naux, naux), **z)
        si, st = torch.empty(ctx.k_shape(), **z), torch.empty(ctx.g_shape(), **z)
        gw.gw_sigma(ctx, dV, G, si, st, P_tau=pt, P0_iw=torch.empty_like(pw), Pt_iw=pw)
        gw.gw_sigma_jvp(ctx, dV, G, pt, pw, dG, si, st)
        ip = lambda a, b: complex((a.conj() * b).sum().item())
        lhs = ip(sb, si) + ip(tb, st)
        for herm in (False, True):
            gw.gw_set_hermitian(ctx, herm)
            gb = torch.empty(ctx.g_shape(), **z)
            gw.gw_sigma_vjp(ctx, dV, G, pt, pw, sb, tb, gb)
            # <s, J dG> = <J^H s, dG>: sums of ntau nk nao^2 products, to the fp64 comparison bound
            scale = (gb.abs() * dG.abs()).sum().item()
            assert abs(lhs - ip(gb, dG)) < 1e-10 * max(1.0, scale), herm
    finally:
        ctx.close()
