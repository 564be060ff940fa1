"""gw_sigma with a Hermitian G solves at Omega >= 0 for one q of each pair and
fills the rest: all its stored arrays against the general mode, at matrix sizes
around the filling kernel's 32 x 32 tiles, with and without a workspace that
splits the solves, and with frequency sets whose zero is and is not a member."""
import numpy as np
import pytest

from paper_2206_07660_amd import inputs as inp
from oracle import grids as og
from oracle import gw as ogw

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to("cuda")


@pytest.mark.parametrize("mesh,nao,naux,ntau", [((3, 1, 2), 4, 31, 8), ((2, 2, 1), 3, 32, 6), ((5, 1, 1), 4, 33, 8),
                                                 ((1, 1, 1), 5, 1, 2)])
def test_stored_arrays(mesh, nao, naux, ntau):
    from paper_2206_07660_amd import gw
    wl = inp.small_workload(name="half", mesh=mesh, nao=nao, naux=naux, ntau=ntau, beta=10.0, seed=59,
                            n_target=float(nao))
    g = og.Grids(wl.beta, wl.ntau)
    H0, S, V = inp.make_H0(wl), inp.make_S(wl), inp.make_V(wl)
    dV, dG = dev(V), dev(ogw.g0_tau(H0, S, 0.03, wl.beta, g.tau))
    z = dict(dtype=torch.complex128, device="cuda")
    nan = lambda shape: torch.full(shape, float("nan"), **z)
    got = {}
    for herm in (False, True):
        ctx = gw.Context(mesh, nao, naux, ntau, wl.beta, ns=wl.ns)
        try:
            gw.gw_set_hermitian(ctx, herm)
            out = [nan((wl.nk, ntau, naux, naux))] + [nan((wl.nk, ctx.nw_b, naux, naux)) for _ in range(2)]
            si, st = nan(ctx.k_shape()), nan(ctx.g_shape())
            gw.gw_sigma(ctx, dV, dG, si, st, P_tau=out[0], P0_iw=out[1], Pt_iw=out[2])
            got[herm] = out + [si, st]
        finally:
            ctx.close()
    for a, b in zip(got[True], got[False]):
        # the tables keep their symmetries to 1e-11 of their largest entry
        assert torch.isfinite(torch.view_as_real(a)).all()
        assert (a - b).abs().max().item() < 1e-10 * max(1.0, b.abs().max().item())
