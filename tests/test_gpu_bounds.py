"""With GW_DEBUG_BOUNDS=1 every triple product and polarization contraction of
the fp64 calls, and every GEMM beside them, is proven on the host to stay inside
its operands: ranges of q, stored and q-by-q evaluations, node chunks that do
not divide the nodes, pairs and self-inverse q, the exchange and the adjoints."""
import numpy as np
import pytest

from paper_2206_07660_amd import inputs as inp
from oracle import grids as og
from oracle import gw as ogw

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to("cuda")


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("mesh,nao,naux,ntau,chunk", [((3, 1, 2), 4, 31, 8, 3), ((2, 2, 1), 1, 5, 6, 4),
                                                      ((1, 1, 1), 5, 2, 2, 1), ((5, 1, 1), 17, 3, 4, 4)])
def test_every_call(mesh, nao, naux, ntau, chunk, precision, monkeypatch):
    from paper_2206_07660_amd import gw
    monkeypatch.setenv("GW_DEBUG_BOUNDS", "1")
    wl = inp.small_workload(name="bounds", mesh=mesh, nao=nao, naux=naux, ntau=ntau, beta=10.0, seed=83, n_target=0.5)
    g = og.Grids(wl.beta, ntau)
    ctx = gw.Context(mesh, nao, naux, ntau, wl.beta, ns=wl.ns, tau_chunk=chunk, max_nq=1, precision=precision)
    z = dict(dtype=torch.complex128, device="cuda")
    new = lambda *s: torch.zeros(s, **z)
    try:
        dV = dev(inp.make_V(wl)).to(ctx.v_dtype)
        G = dev(ogw.g0_tau(inp.make_H0(wl), inp.make_S(wl), 0.03, wl.beta, g.tau))
        nk = wl.nk
        pt, pw, p0 = new(nk, ntau, naux, naux), new(nk, ctx.nw_b, naux, naux), new(nk, ctx.nw_b, naux, naux)
        si, st, gb = new(*ctx.k_shape()), new(*ctx.g_shape()), new(*ctx.g_shape())
        for herm in (False, True):
            gw.gw_set_hermitian(ctx, herm, two_slot=herm)
            for q0, nq in ((0, nk), (nk - 1, 1)):
                gw.gw_polarization(ctx, dV, G, q0, nq, pt[:nq])
                gw.gw_polarization_noalloc(ctx, dV, G, q0, nq, pt[:nq])
                gw.gw_polarization2(ctx, dV, G, G, q0, nq, pt[:nq], accumulate=True)
                gw.gw_self_energy(ctx, dV, G, pt[:nq], q0, nq, st)
                gw.gw_self_energy_vjp(ctx, dV, G, pt[:nq], st, q0, nq, gb, torch.empty_like(pt[:nq]))
                gw.gw_polarization_vjp(ctx, dV, G, pt[:nq], q0, nq, gb)
            gw.gw_hf(ctx, dV, G, None, si)
            gw.gw_hf_vjp(ctx, dV, si, gb)
            gw.gw_sigma(ctx, dV, G, si, st)
            gw.gw_sigma(ctx, dV, G, si, st, want_phi=True)
            gw.gw_sigma(ctx, dV, G, si, st, P_tau=pt, P0_iw=p0, Pt_iw=pw)
            for a in ((pt, pw), (None, None)):
                gw.gw_sigma_jvp(ctx, dV, G, *a, G, si, st)
                gw.gw_sigma_vjp(ctx, dV, G, *a, si, st, gb)
        assert torch.isfinite(torch.view_as_real(gb)).all()
    finally:
        ctx.close()
