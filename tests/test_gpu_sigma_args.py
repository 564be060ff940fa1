"""gw_sigma refuses one array for P0(i Omega) and P~(i Omega), with and without
the Hermitian mode, and writes nothing."""
import numpy as np
import pytest

from paper_2206_07660_amd import inputs as inp

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("herm", [False, True])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_one_array_for_both(herm, precision):
    from paper_2206_07660_amd import gw
    mesh, nao, naux, ntau = (2, 1, 1), 2, 5, 4
    wl = inp.small_workload(name="args", mesh=mesh, nao=nao, naux=naux, ntau=ntau, beta=10.0, seed=89, n_target=0.5)
    ctx = gw.Context(mesh, nao, naux, ntau, wl.beta, ns=wl.ns, precision=precision)
    z = dict(dtype=torch.complex128, device="cuda")
    try:
        gw.gw_set_hermitian(ctx, herm)
        V = torch.from_numpy(np.ascontiguousarray(inp.make_V(wl))).to("cuda").to(ctx.v_dtype)
        G = torch.zeros(ctx.g_shape(), **z)
        seven = lambda *s: torch.full(s, 7.0, **z)
        si, st = seven(*ctx.k_shape()), seven(*ctx.g_shape())
        pt, pw = seven(wl.nk, ntau, naux, naux), seven(wl.nk, ctx.nw_b, naux, naux)
        with pytest.raises(gw.GwError) as e:
            gw.gw_sigma(ctx, V, G, si, st, P_tau=pt, P0_iw=pw, Pt_iw=pw)
        assert e.value.status == gw.GW_ERR_ARG
        torch.cuda.synchronize()
        assert all(bool((x == 7.0).all()) for x in (si, st, pt, pw))
    finally:
        ctx.close()
