"""The blocked solve of (I - P0) P~ = P0 at matrix orders around its panels of
32 columns, its 256- and 512-row panel kernels and the general panel beyond
them, for matrices that need no, some and many row interchanges."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 31, 32, 33, 63, 64, 65, 97, 255, 256, 257, 289, 512, 513, 545])
@pytest.mark.parametrize("kind", ["screening", "random", "reversed"])
def test_solve(n, kind):
    from paper_2206_07660_amd import gw
    rng = np.random.default_rng([n, len(kind)])
    ntau = 2
    ctx = gw.Context((1, 1, 1), 2, n, ntau, 10.0)
    try:
        z = rng.normal(size=(ctx.nw_b, n, n)) + 1j * rng.normal(size=(ctx.nw_b, n, n))
        if kind == "screening":
            P0 = -(z @ z.conj().transpose(0, 2, 1)) / n
        elif kind == "random":
            P0 = z / np.sqrt(n) + 3.0 * np.eye(n)[rng.permutation(n)]
        else:
            # I - P0 is large on the antidiagonal: every pivot is at the far end
            P0 = np.eye(n) - 4.0 * np.eye(n)[::-1] + 0.05 * z / np.sqrt(n)
        A = np.eye(n) - P0
        X = torch.empty((1,) + P0.shape, dtype=torch.complex128, device="cuda")
        gw.gw_screened_W(ctx, torch.from_numpy(P0[None].copy()).cuda(), X)
        x = X.cpu().numpy()[0]
        # residual of a pivoted elimination: a few n eps of |A| |X| per entry,
        # ten times that for its growth
        bound = 40 * n * 2.3e-16 * (np.abs(A) @ np.abs(x) + np.abs(P0)).max()
        assert np.abs(A @ x - P0).max() < bound
    finally:
        ctx.close()


def test_zero_pivot_is_reported():
    from paper_2206_07660_amd import gw
    n = 40
    ctx = gw.Context((1, 1, 1), 2, n, 2, 10.0)
    try:
        P0 = torch.zeros((1, ctx.nw_b, n, n), dtype=torch.complex128, device="cuda")
        P0[0, 1, 35, 35] = 1.0                  # a zero column of I - P0
        with pytest.raises(gw.GwError):
            gw.gw_screened_W(ctx, P0, torch.empty_like(P0))
        P0.zero_()
        X = torch.empty_like(P0)
        gw.gw_screened_W(ctx, P0, X)
        assert X.abs().max().item() == 0.0
    finally:
        ctx.close()
