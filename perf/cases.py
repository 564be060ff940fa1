"""Workloads of the GW path whose speed matters, as a program that uses the
package runs them: inputs, one pass, the work of a pass, and 64-bit results.

A case is a plain dict.  `kind` names the call:

  one_shot   GWPath.start + GWPath.step: G0 at the chemical potential of the
             electron count, then one damped scGW iteration
  sigma      one Sigma[G] + Pi evaluation (GWPath.sigma with every P~ kept, or
             gw_sigma q by q when `stored` is false)
  pol, se    gw_polarization / gw_self_energy on a range of q-points, the unit
             that a program sharded over q calls
  screened   gw_screened_W on nq q-points
  mu         gw_find_mu: Dyson equation inside the electron-count search
  hf         gw_hf
  jvp, vjp   gw_sigma_jvp / gw_sigma_vjp, a Newton-Krylov product and a
             gradient, with P~ kept from the forward call

Sizes: n1 x n2 x n3 k-points, nao orbitals, naux auxiliary functions, ntau
Chebyshev nodes, inverse temperature beta.  `metal` takes the bands of H0 from
one interval (-1, 1) Ha, otherwise 4 occupied ones in (-1, -0.2) and the rest
in (0.1, 3).
"""
import math

import numpy as np
import torch

from paper_2206_07660_amd import gw
from paper_2206_07660_amd.scgw import GWPath

NS = 2
C128 = torch.complex128


def _case(name, kind, mesh, nao, naux, ntau, beta, precision="fp64", metal=False, hermitian=True,
          stored=True, q0=0, nq=1):
    return {"name": name, "kind": kind, "n1": mesh[0], "n2": mesh[1], "n3": mesh[2], "nao": nao, "naux": naux,
            "ntau": ntau, "beta": float(beta), "precision": precision, "metal": metal, "hermitian": hermitian,
            "stored": stored, "q0": q0, "nq": nq}


def listed():
    return [
        # the smallest whole calculation (smoke and oracle size): every launch and
        # every wait of a short scGW step, two mu searches among them
        _case("one_shot_222_nao6", "one_shot", (2, 2, 2), 6, 24, 24, 50, metal=True),
        # a small odd system: nao^2 and naux odd, mixed even and odd mesh, no
        # Hermitian shortcut, nothing kept per q
        _case("sigma_312_nao7_perq", "sigma", (3, 1, 2), 7, 61, 30, 30, hermitian=False, stored=False),
        # the ordinary evaluation of a solver's inner loop
        _case("sigma_333_nao16", "sigma", (3, 3, 3), 16, 150, 60, 100),
        # the Si-like basis on a 3x3x3 mesh: the largest whole evaluation here
        _case("sigma_333_nao26", "sigma", (3, 3, 3), 26, 250, 100, 100),
        # the same inner loop in mixed precision, split-bf16 and fp32
        _case("sigma_333_nao16_bf16x3", "sigma", (3, 3, 3), 16, 150, 60, 100, precision="bf16x3"),
        _case("sigma_333_nao16_fp32", "sigma", (3, 3, 3), 16, 150, 60, 100, precision="fp32"),
        # one q-point of the Si-like 4x4x4 workload: what one owner of q does
        _case("pol_444_nao26_q", "pol", (4, 4, 4), 26, 250, 100, 100, q0=1),
        _case("se_444_nao26_q", "se", (4, 4, 4), 26, 250, 100, 100, q0=1),
        # the frequency-space solves of four q-points of that workload
        _case("screened_naux250_4q", "screened", (4, 4, 4), 26, 250, 100, 100, nq=4),
        # chemical potential and Dyson equation of the 4x4x4 workload's sizes
        _case("mu_444_nao26", "mu", (4, 4, 4), 26, 250, 100, 100, metal=True),
        # Newton-Krylov product (Hermitian direction) and gradient
        _case("jvp_333_nao16", "jvp", (3, 3, 3), 16, 150, 60, 100),
        _case("vjp_333_nao16", "vjp", (3, 3, 3), 16, 150, 60, 100),
    ]


# ------------------------------------------------------------------ draws ---
_MESHES = [(1, 1, 1), (2, 1, 1), (2, 2, 1), (3, 1, 2), (2, 2, 2), (3, 2, 2), (1, 5, 3), (4, 2, 2), (3, 3, 2),
           (3, 3, 3), (4, 3, 3), (4, 4, 4)]
_KINDS = ["one_shot", "sigma", "sigma", "sigma", "pol", "se", "screened", "mu", "hf", "jvp", "vjp"]


def _nk(c):
    return c["n1"] * c["n2"] * c["n3"]


def _chain_flops(c, nq):
    """Contractions of the polarization and of the self-energy for nq q-points."""
    nk, nao, naux, nt = _nk(c), c["nao"], c["naux"], c["ntau"]
    per = nq * nk * nt * 8.0 * (naux * naux * nao * nao + 2.0 * naux * nao ** 3)
    return per, per


def _cost(c):
    nk, n = _nk(c), c["naux"]
    pol, se = _chain_flops(c, nk)
    return {"one_shot": pol + se, "sigma": pol + se, "pol": pol * c["nq"] / nk, "se": se * c["nq"] / nk,
            "screened": (32.0 / 3.0) * n ** 3 * (c["ntau"] + 1) * c["nq"], "mu": 1e9,
            "hf": 16.0 * nk * nk * n * c["nao"] ** 3, "jvp": 3 * pol + 2 * se, "vjp": 3 * pol + 3 * se}[c["kind"]]


def _v_bytes(c):
    nk = _nk(c)
    return nk * nk * c["naux"] * c["nao"] ** 2 * (16 if c["precision"] == "fp64" else 8)


def draw(rng):
    """One more case of the ranges above: meshes of 1 to 64 k-points, nao 4..30,
    naux 2..11 nao, ntau 20..120."""
    cap = _cost(listed()[3])
    while True:
        kind = rng.choice(_KINDS)
        mesh = rng.choice(_MESHES)
        nk = mesh[0] * mesh[1] * mesh[2]
        nao = int(round(math.exp(rng.uniform(math.log(4), math.log(30)))))
        naux = min(300, max(12, int(round(nao * math.exp(rng.uniform(math.log(2.5), math.log(11)))))))
        ntau = 2 * int(round(math.exp(rng.uniform(math.log(10), math.log(60)))))
        beta = round(min(100.0, max(15.0, ntau * rng.uniform(0.8, 1.8))), 1)
        precision = rng.choice(["fp64", "fp64", "fp64", "bf16x3", "fp32", "bf16x6"])
        if kind in ("screened", "mu", "vjp"):
            precision = "fp64"
        q0 = rng.randrange(nk)
        nq = rng.randint(1, min(4, nk - q0))
        c = _case("", kind, mesh, nao, naux, ntau, beta, precision, metal=kind in ("mu", "one_shot") or rng.random() < 0.3,
                  hermitian=rng.random() < 0.75 or kind in ("mu", "one_shot"), stored=rng.random() < 0.7,
                  q0=q0 if kind in ("pol", "se") else 0, nq=nq)
        del c["name"]
        if kind in ("mu", "one_shot") and nk * nao < 48:
            continue                      # too few levels: the count hardly fixes mu
        # whole evaluations keep V and P~ of every q
        small = nk * ntau * naux * naux * 16 <= 4e9 if kind in ("sigma", "one_shot", "jvp", "vjp") else True
        if _cost(c) <= cap and _v_bytes(c) <= 12e9 and small:
            return c


# ----------------------------------------------------------------- inputs ---
def _device():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _gen(seed, stream, device="cpu"):
    return torch.Generator(device=device).manual_seed(int(seed) * 1009 + stream)


def _shifts(c):
    n = (c["n1"], c["n2"], c["n3"])
    p = np.stack(np.meshgrid(*(np.arange(m) for m in n), indexing="ij"), -1).reshape(-1, 3)
    idx = lambda x: (x[..., 0] % n[0] * n[1] + x[..., 1] % n[1]) * n[2] + x[..., 2] % n[2]  # noqa: E731
    return idx(p[:, None] + p[None]), idx(-p)          # plus[q][k] = k + q, neg[q] = -q


def _bands(c, seed):
    """Eigenvalues and eigenvectors of H0(k), the target count and mu inside it."""
    nk, n = _nk(c), c["nao"]
    g = _gen(seed, 1)
    z = torch.randn((nk, n, n), generator=g, dtype=C128)
    U = torch.linalg.qr(z).Q
    u = torch.rand((nk, n), generator=g, dtype=torch.float64)
    if c["metal"]:
        e, target, mu = 2.0 * u - 1.0, float(n), 0.0
    else:
        occ = min(4, max(1, n // 3))
        e = torch.cat([-1.0 + 0.8 * u[:, :occ], 0.1 + 2.9 * u[:, occ:]], 1)
        target, mu = 2.0 * occ, -0.05
    e = e.sort(1).values
    return e, U, target, mu


def _h0(e, U):
    H = (U * e[:, None, :].to(C128)) @ U.conj().transpose(1, 2)
    return 0.5 * (H + H.conj().transpose(1, 2))


def _g0(e, U, mu, tau, beta):
    """G0(tau) = -U e^{-tau xi} / (1 + e^{-beta xi}) U^H at the nodes."""
    t = torch.as_tensor(tau)[:, None, None]
    xi = (e - mu)[None]
    f = -torch.where(xi > 0, torch.exp(-t * xi.clamp(min=0)) / (1 + torch.exp(-beta * xi.clamp(min=0))),
                     torch.exp((beta - t) * xi.clamp(max=0)) / (1 + torch.exp(beta * xi.clamp(max=0))))
    dev = _device()
    f, U = f.to(dev).to(C128), U.to(dev)
    G = (U[None] * f[:, :, None, :]) @ U.conj().transpose(1, 2)[None]
    return 0.5 * (G + G.conj().transpose(2, 3))


def _v(c, seed):
    """V[q][k] = V^{k,k+q}: Gaussian, with V^{k2,k1}(Q) = V^{k1,k2}(Q)^H."""
    dev, nk = _device(), _nk(c)
    plus, neg = _shifts(c)
    dt = C128 if c["precision"] == "fp64" else torch.complex64
    V = torch.empty((nk, nk, c["naux"], c["nao"], c["nao"]), dtype=dt, device=dev)
    g = _gen(seed, 2, dev)
    s = 0.1 * math.sqrt(24.0 / c["naux"])
    adj = lambda x: x.conj().transpose(2, 3)  # noqa: E731
    for q in range(nk):
        p = torch.as_tensor(plus[q], device=dev)
        if q <= neg[q]:
            R = torch.randn(V.shape[1:], generator=g, dtype=dt, device=dev) * s
            if q == neg[q]:
                R = (R + adj(R[p])) / math.sqrt(2.0)
            V[q] = R
        else:                              # V[q][k] = V[-q][k+q]^H
            V[q] = adj(V[neg[q]][p])
    return V


def _hermitian(shape, gen, scale, dev):
    x = torch.randn(shape, generator=gen, dtype=C128, device=dev) * scale
    return 0.5 * (x + x.conj().transpose(-1, -2))


def _p_tilde(c, seed, tau):
    """P~^q(tau) for nq q-points: negative definite, decaying from both ends."""
    dev, n = _device(), c["naux"]
    g = _gen(seed, 3, dev)
    M = torch.randn((c["nq"], n, n // 2 + 1), generator=g, dtype=C128, device=dev) / n
    gap = 0.3 + torch.rand(n // 2 + 1, generator=g, dtype=torch.float64, device=dev)
    t = torch.as_tensor(tau, device=dev)[:, None]
    w = -(torch.exp(-t * gap) + torch.exp(-(c["beta"] - t) * gap))
    P = torch.stack([(M[:, None] * w[None, :, None, :].to(C128))[i] @ M[i].conj().T for i in range(c["nq"])])
    return 0.5 * (P + P.conj().transpose(2, 3))


def _p_bare(c, seed, wB):
    """P0^q(i Omega): -sum_j m_j m_j^H (2 d_j + i c_j Omega) / (d_j^2 + Omega^2)."""
    dev, n = _device(), c["naux"]
    g = _gen(seed, 3, dev)
    M = torch.randn((c["nq"], n, n), generator=g, dtype=C128, device=dev) * (0.5 / math.sqrt(n))
    d = 0.3 + 2.0 * torch.rand(n, generator=g, dtype=torch.float64, device=dev)
    a = 0.4 * torch.rand(n, generator=g, dtype=torch.float64, device=dev) - 0.2
    W = torch.as_tensor(wB, device=dev)[:, None]
    D = torch.complex(-2.0 * d / (d * d + W * W), -a * W / (d * d + W * W))
    return torch.stack([(M[i][None] * D[:, None, :]) @ M[i].conj().T for i in range(c["nq"])])


def _self_energy_poles(c, seed, wF):
    """Sigma_inf and Sigma~(i w) = sum_p B_p / (i w - e_p), B_p >= 0."""
    nk, n = _nk(c), c["nao"]
    g = _gen(seed, 4)
    dev = _device()
    sinf = _hermitian((nk, n, n), g, 0.05, "cpu").to(dev)
    siw = torch.zeros((len(wF), nk, n, n), dtype=C128, device=dev)
    for e in (-1.5, 1.7):
        A = torch.randn((nk, n, n), generator=g, dtype=C128).to(dev) * (0.15 / math.sqrt(n))
        B = A @ A.conj().transpose(1, 2)
        siw += B[None] / torch.as_tensor(1j * wF - e, device=dev)[:, None, None, None]
    return sinf, siw


def _directions(c, seed):
    """A Hermitian direction dG, or the cotangents of (Sigma_inf, Sigma~)."""
    dev, nk, n = _device(), _nk(c), c["nao"]
    g = _gen(seed, 5, dev)
    tau = _hermitian((c["ntau"], nk, n, n), g, 0.1, dev)
    if not c["hermitian"]:
        tau = tau + 0.05 * torch.randn(tau.shape, generator=g, dtype=C128, device=dev)
    return _hermitian((nk, n, n), g, 0.1, dev), tau


def prepare(case, seed):
    c, kind = case, case["kind"]
    nk = _nk(c)
    z = dict(dtype=C128, device="cuda")
    few = kind in ("pol", "se", "screened", "mu", "hf")
    ctx = gw.Context((c["n1"], c["n2"], c["n3"]), c["nao"], c["naux"], c["ntau"], c["beta"], ns=NS,
                     max_nq=c["nq"] if few else None, precision=c["precision"])
    s = {"case": c, "ctx": ctx}
    g = ctx.grids
    e, U, target, mu = _bands(c, seed)
    herm = c["hermitian"]
    if kind in ("one_shot", "sigma", "jvp", "vjp", "pol", "se", "hf"):
        s["V"] = _v(c, seed)
        s["G"] = _g0(e, U, mu, g["tau"], c["beta"])
        gw.gw_set_hermitian(ctx, herm, two_slot=herm and kind == "jvp")
    if kind == "one_shot" or (kind == "sigma" and c["stored"]):
        S = torch.eye(c["nao"], dtype=C128).repeat(nk, 1, 1).cuda()
        s["path"] = GWPath(ctx, s["V"], _h0(e, U).cuda(), S, target, hermitian=herm)
    if kind in ("sigma", "jvp", "vjp", "hf"):
        s["sinf"], s["gamma"] = torch.empty(ctx.k_shape(), **z), torch.empty(ctx.k_shape(), **z)
        s["stau"] = torch.empty(ctx.g_shape(), **z)
    if kind == "pol":
        s["P"] = torch.empty((c["nq"], c["ntau"], c["naux"], c["naux"]), **z)
    if kind == "se":
        s["Pt"] = _p_tilde(c, seed, g["tau"])
        s["stau"] = torch.empty(ctx.g_shape(), **z)
    if kind == "screened":
        s["P0"] = _p_bare(c, seed, 2.0 * np.pi * g["nB"] / c["beta"])
        s["P"] = torch.empty_like(s["P0"])
    if kind == "mu":
        s["H0"], s["S"] = _h0(e, U).cuda(), torch.eye(c["nao"], dtype=C128).repeat(nk, 1, 1).cuda()
        s["target"], s["mu0"] = target, mu + 0.03
        s["sinf"], s["siw"] = _self_energy_poles(c, seed, (2.0 * g["nF"] + 1.0) * np.pi / c["beta"])
        s["Giw"], s["Gtau"] = torch.empty(ctx.giw_shape(), **z), torch.empty(ctx.g_shape(), **z)
    if kind in ("jvp", "vjp"):
        n = c["naux"]
        s["Pt"], s["Pw"] = torch.empty((nk, c["ntau"], n, n), **z), torch.empty((nk, ctx.nw_b, n, n), **z)
        gw.gw_sigma(ctx, s["V"], s["G"], s["sinf"], s["stau"], P_tau=s["Pt"], P0_iw=torch.empty_like(s["Pw"]),
                    Pt_iw=s["Pw"])
        s["dinf"], s["dtau"] = _directions(c, seed)
        s["Gbar"] = torch.empty(ctx.g_shape(), **z)
    return s


def run(s):
    c, ctx, kind = s["case"], s["ctx"], s["case"]["kind"]
    if kind == "one_shot":
        st = s["path"].start(0.0)
        st = s["path"].step(st)
        return {"mu": st.mu, "n_e": st.n_e, "sig_inf": st.sig_inf, "sig_tau": st.sig_tau, "G_tau": st.G_tau}
    if kind == "sigma":
        if c["stored"]:
            p = s["path"]
            sinf, stau = p.sigma(s["G"])
            return {"sig_inf": sinf, "sig_tau": stau, "gamma": p.gamma, "P_tau": p.P0, "P_iw": p.Pw}
        gw.gw_sigma(ctx, s["V"], s["G"], s["sinf"], s["stau"], gamma=s["gamma"])
        return {"sig_inf": s["sinf"], "sig_tau": s["stau"], "gamma": s["gamma"]}
    if kind == "pol":
        gw.gw_polarization(ctx, s["V"], s["G"], c["q0"], c["nq"], s["P"])
        return {"P0": s["P"]}
    if kind == "se":
        s["stau"].zero_()
        gw.gw_self_energy(ctx, s["V"], s["G"], s["Pt"], c["q0"], c["nq"], s["stau"])
        return {"sig_tau": s["stau"]}
    if kind == "screened":
        gw.gw_screened_W(ctx, s["P0"], s["P"])
        return {"P_iw": s["P"]}
    if kind == "mu":
        mu, ne = gw.gw_find_mu(ctx, s["H0"], s["S"], s["sinf"], s["siw"], s["target"], s["mu0"], G_iw=s["Giw"],
                               G_tau=s["Gtau"])
        return {"mu": mu, "n_e": ne, "G_iw": s["Giw"], "G_tau": s["Gtau"]}
    if kind == "hf":
        gw.gw_hf(ctx, s["V"], s["G"], s["gamma"], s["sinf"])
        return {"sig_inf": s["sinf"], "gamma": s["gamma"]}
    if kind == "jvp":
        gw.gw_sigma_jvp(ctx, s["V"], s["G"], s["Pt"], s["Pw"], s["dtau"], s["sinf"], s["stau"])
        return {"d_inf": s["sinf"], "d_tau": s["stau"]}
    gw.gw_sigma_vjp(ctx, s["V"], s["G"], s["Pt"], s["Pw"], s["dinf"], s["dtau"], s["Gbar"])
    return {"G_bar": s["Gbar"]}


def work(case):
    """Inputs read once, outputs written once; the flops of the equations at 8
    per complex multiply-add, without their symmetries."""
    c, kind = case, case["kind"]
    nk, nao, n, nt = _nk(c), c["nao"], c["naux"], c["ntau"]
    k = 16.0 * nk * nao * nao
    G, V = nt * k, float(_v_bytes(c))
    nb = nt + 1
    Pt, Pw = 16.0 * nt * n * n, 16.0 * nb * n * n
    pol, se = _chain_flops(c, 1)
    solve = (32.0 / 3.0) * n ** 3 * nb + 2 * 8.0 * nt * nb * n * n
    hf = 16.0 * nk * nk * n * nao ** 3
    dyson = 8.0 * nt * nk * nao ** 3
    if kind == "mu":
        return {"bytes": 3 * k + 3 * G, "flops": dyson + 8.0 * nt * nt * nk * nao * nao}
    if kind == "screened":
        return {"bytes": 2 * c["nq"] * Pw, "flops": c["nq"] * (32.0 / 3.0) * n ** 3 * nb}
    if kind == "pol":
        return {"bytes": c["nq"] * (V / nk + Pt) + G, "flops": c["nq"] * pol}
    if kind == "se":
        return {"bytes": c["nq"] * (V / nk + Pt) + 2 * G, "flops": c["nq"] * se}
    if kind == "hf":
        return {"bytes": V + G + 2 * k, "flops": hf}
    if kind in ("sigma", "one_shot"):
        return {"bytes": V + 2 * G + 2 * k + (nk * (Pt + 2 * Pw) if c["stored"] else 0.0),
                "flops": nk * (pol + se + solve) + hf + (2 * dyson if kind == "one_shot" else 0.0)}
    flops = nk * (2 * pol + 2 * se + 2 * 8.0 * n ** 3 * nb) + hf
    if kind == "vjp":
        flops = nk * (2 * pol + 2 * se + 2 * 8.0 * n ** 3 * nb) + 2 * hf
    return {"bytes": V + 3 * G + 2 * k + nk * (Pt + Pw), "flops": flops}


# ---------------------------------------------------------- 64-bit results ---
def _transform(nu, beta, nt, x):
    """T[n][i] = int_0^beta L_i(tau) e^{i nu_n tau} d tau, L_i the Lagrange
    polynomials of the nodes: Gauss-Legendre moments of the Chebyshev basis."""
    cheb = np.polynomial.chebyshev.chebvander
    xg, wg = np.polynomial.legendre.leggauss(nt + int(math.ceil(beta * np.abs(nu).max() / 2.0)) + 200)
    E = np.exp(1j * np.outer(nu, beta * (1.0 + xg) / 2.0)) * (wg * beta / 2.0)
    return (E @ cheb(xg, nt - 1)) @ np.linalg.inv(cheb(x, nt - 1))


def _grids(c):
    """Nodes, transforms and density row of a context's default grids: symmetric
    Matsubara pairs among n < 4 ntau by largest remaining transform rows."""
    beta, nt = c["beta"], c["ntau"]
    x = -np.cos((2 * np.arange(nt) + 1) * np.pi / (2 * nt))
    x[nt // 2:] = -x[:nt // 2][::-1]
    tau = beta * (1.0 + x) / 2.0
    tau[nt // 2:] = beta - tau[:nt // 2][::-1]
    cand = np.arange(4 * nt)
    out = {"tau": tau}
    for stat in "FB":
        w = (2 * cand + 1 if stat == "F" else 2 * cand) * np.pi / beta
        T = _transform(np.concatenate([w, -w]), beta, nt, x)      # rows n and their partners
        R = T / np.linalg.norm(T, axis=1)[:, None]
        free, chosen, basis = np.ones(len(cand), bool), [], []
        first = [[0]] if stat == "B" else []
        while len(chosen) < nt // 2 + len(first):
            if len(chosen) < len(first):
                i, rows = 0, [0]
            else:
                res = (np.abs(R) ** 2).sum(1)
                res = np.where(free, res[:len(cand)] + res[len(cand):], -1.0)
                i = int(np.nonzero(res >= res.max() * (1.0 - 1e-9))[0][0])
                rows = [i, i + len(cand)]
            free[i] = False
            chosen.append(i)
            for r in rows:
                v = T[r].copy()
                for _ in range(2):
                    for b in basis:
                        v -= b * np.vdot(b, v)
                v /= np.linalg.norm(v)
                basis.append(v)
                R = R - np.outer(R @ v.conj(), v)
        s = np.array(sorted(chosen[len(first):]))
        n = np.concatenate([-s[::-1] - 1, s]) if stat == "F" else np.concatenate([-s[::-1], [0], s])
        nu = (2 * n + 1 if stat == "F" else 2 * n) * np.pi / beta
        T = _transform(nu, beta, nt, x)
        out["nu" + stat], out["T" + stat], out["T" + stat + "p"] = nu, T, np.linalg.pinv(T)
    out["w"] = np.ones(nt) @ np.linalg.inv(np.polynomial.chebyshev.chebvander(x, nt - 1))
    dev = _device()
    for k in ("TF", "TFp", "TB", "TBp", "w"):
        out[k] = torch.as_tensor(np.asarray(out[k], np.complex128), device=dev)
    return out


def _apply(T, X):
    return (T @ X.reshape(X.shape[0], -1)).reshape((T.shape[0],) + tuple(X.shape[1:]))


def _adj(x):
    return x.conj().transpose(-1, -2)


def _solve(A, B):
    """A^{-1} B for batches whose A has a positive definite Hermitian part, by
    2 x 2 blocks down to sizes that the batched LU takes."""
    n = A.shape[-1]
    if n <= 128:
        return torch.linalg.solve(A, B)
    h = n // 2
    Y = _solve(A[..., :h, :h], torch.cat([A[..., :h, h:], B[..., :h, :]], -1))
    E, F = Y[..., :n - h], Y[..., n - h:]
    low = _solve(A[..., h:, h:] - _mm(A[..., h:, :h], E), B[..., h:, :] - _mm(A[..., h:, :h], F))
    return torch.cat([F - _mm(E, low), low], -2)


def _mm(a, b):
    return torch.matmul(a.resolve_conj().contiguous(), b.resolve_conj().contiguous())


class _Exact:
    """The chain of one evaluation in plain complex128 products, q by q."""

    def __init__(self, c, seed):
        self.c, self.g = c, _grids(c)
        self.nk, self.n, self.nao, self.nt = _nk(c), c["naux"], c["nao"], c["ntau"]
        plus, _ = _shifts(c)
        self.plus = torch.as_tensor(plus, device=_device())
        self.V = _v(c, seed)

    def vq(self, q):
        return self.V[q].to(C128)                                  # [k][Q][i][j]

    def pol(self, Ga, Gb, q):
        """-(ns/Nk) sum_k tr[V(Q) Ga^{k+q}(tau) V(Q')^H Gb^k(beta - tau)]"""
        V, n, m = self.vq(q), self.n, self.nk * self.nao ** 2
        Vh = _adj(V)
        out = []
        for i in range(self.nt):
            X = _mm(V, Ga[i][self.plus[q]][:, None])                       # [k][Q][d][b]
            Z = _mm(Vh, Gb[self.nt - 1 - i][:, None]).transpose(2, 3)      # [k][Q'][d][b]
            out.append(_mm(X.transpose(0, 1).reshape(n, m), Z.transpose(0, 1).reshape(n, m).T))
        return (-NS / self.nk) * torch.stack(out)

    def se(self, G, Pt, q):
        V, n, nk, a = self.vq(q), self.n, self.nk, self.nao
        Vh, Vm = _adj(V), V.transpose(0, 1).reshape(n, -1)
        out = []
        for i in range(self.nt):
            W = _mm(Pt[i], Vm).reshape(n, nk, a, a).transpose(0, 1)        # [kk][Q][b][j]
            L = _mm(Vh, G[i][:, None]).transpose(1, 2).reshape(nk, a, n * a)
            s = _mm(L, W.reshape(nk, n * a, a)) * (-1.0 / nk)
            out.append(torch.zeros_like(s).index_copy(0, self.plus[q], s))
        return torch.stack(out)

    def hf(self, G):
        gamma = -_apply(self.g["w"][None], G)[0]
        V0 = self.vq(0)
        v = (NS / self.nk) * (V0 * gamma.transpose(1, 2)[:, None]).sum((0, 2, 3))
        out = (V0 * v[None, :, None, None]).sum(1)
        for q in range(self.nk):
            V = self.vq(q)
            T = _mm(V, gamma[self.plus[q]][:, None])                       # [k][Q][i][b]
            A = T.transpose(1, 2).reshape(self.nk, self.nao, -1)
            B = V.transpose(1, 2).reshape(self.nk, self.nao, -1)
            out = out - _mm(A, _adj(B)) / self.nk
        return out, gamma

    def solve(self, P0t):
        """P~(i Omega) and P~(tau) of P0(tau)."""
        P0 = _apply(self.g["TB"], P0t)
        Pw = _solve(torch.eye(self.n, dtype=C128, device=P0.device) - P0, P0)
        return Pw, _apply(self.g["TBp"], Pw)

    def sigma(self, G):
        stau, pts, pws = torch.zeros_like(G), [], []
        for q in range(self.nk):
            Pw, Pt = self.solve(self.pol(G, G, q))
            stau += self.se(G, Pt, q)
            pts.append(Pt)
            pws.append(Pw)
        return self.hf(G) + (stau, pts, pws)

    def jvp(self, G, dG):
        out = torch.zeros_like(G)
        one = torch.eye(self.n, dtype=C128, device=G.device)
        for q in range(self.nk):
            Pw, Pt = self.solve(self.pol(G, G, q))
            dP0 = _apply(self.g["TB"], self.pol(dG, G, q) + self.pol(G, dG, q))
            dPt = _apply(self.g["TBp"], _mm(_mm(one + Pw, dP0), one + Pw))
            out += self.se(G, dPt, q) + self.se(dG, Pt, q)
        return self.hf(dG)[0], out

    def vjp(self, G, sbar, tbar):
        G = G.detach().requires_grad_(True)
        total = torch.zeros_like(G)
        inner = lambda a, b: (a.conj() * b).real.sum()  # noqa: E731
        with torch.enable_grad():
            total += torch.autograd.grad(inner(sbar, self.hf(G)[0]), G)[0]
            for q in range(self.nk):
                _, Pt = self.solve(self.pol(G, G, q))
                total += torch.autograd.grad(inner(tbar, self.se(G, Pt, q)), G)[0]
        return total


def _count_solver(c, g, H0, sinf, siw, target, mu0):
    """mu of the electron count by bisection, and G there (S = identity)."""
    nk = _nk(c)
    iw = torch.as_tensor(1j * g["nuF"], device=H0.device)[:, None, None, None]
    one = torch.eye(c["nao"], dtype=C128, device=H0.device)
    base = H0[None] + (0 if sinf is None else sinf[None]) + (0 if siw is None else siw)
    r = g["w"] @ g["TFp"]
    green = lambda mu: torch.linalg.inv((iw + mu) * one - base)  # noqa: E731
    count = lambda G: -(NS / nk) * float((r[:, None] * G.diagonal(dim1=2, dim2=3).sum(2)).real.sum())  # noqa: E731
    lo, hi = mu0 - 1.0, mu0 + 1.0
    while count(green(lo)) > target:
        lo -= 2.0
    while count(green(hi)) < target:
        hi += 2.0
    while hi - lo > 1e-13:
        mid = 0.5 * (lo + hi)
        if mid in (lo, hi):
            break
        lo, hi = (mid, hi) if count(green(mid)) < target else (lo, mid)
    mu = 0.5 * (lo + hi)
    G = green(mu)
    return mu, count(G), G, _apply(g["TFp"], G)


def exact(case, seed):
    c, kind = case, case["kind"]
    dev = _device()
    if _cost(c) > 1.2 * _cost(listed()[3]):
        return None
    with torch.no_grad():
        e, U, target, mu = _bands(c, seed)
        if kind == "screened":
            P0 = _p_bare(c, seed, _grids(c)["nuB"])
            one = torch.eye(c["naux"], dtype=C128, device=dev)
            return {"P_iw": torch.stack([_solve(one - p, p) for p in P0])}
        if kind == "mu":
            g = _grids(c)
            sinf, siw = _self_energy_poles(c, seed, g["nuF"])
            m, ne, Giw, Gtau = _count_solver(c, g, _h0(e, U).to(dev), sinf, siw, target, mu + 0.03)
            return {"mu": m, "n_e": ne, "G_iw": Giw, "G_tau": Gtau}
        x = _Exact(c, seed)
        if kind == "one_shot":
            H0 = _h0(e, U).to(dev)
            m0, _, _, G = _count_solver(c, x.g, H0, None, None, target, 0.0)
            sinf, _, stau, _, _ = x.sigma(G)
            sinf, stau = 0.5 * sinf, 0.5 * stau
            m, ne, _, Gtau = _count_solver(c, x.g, H0, sinf, _apply(x.g["TF"], stau), target, m0)
            return {"mu": m, "n_e": ne, "sig_inf": sinf, "sig_tau": stau, "G_tau": Gtau}
        G = _g0(e, U, mu, x.g["tau"], c["beta"])
        if kind == "sigma":
            sinf, gamma, stau, pts, pws = x.sigma(G)
            out = {"sig_inf": sinf, "sig_tau": stau, "gamma": gamma}
            if c["stored"]:
                out["P_tau"], out["P_iw"] = torch.stack(pts), torch.stack(pws)
            return out
        qs = range(c["q0"], c["q0"] + c["nq"])
        if kind == "pol":
            return {"P0": torch.stack([x.pol(G, G, q) for q in qs])}
        if kind == "se":
            Pt = _p_tilde(c, seed, x.g["tau"])
            return {"sig_tau": sum(x.se(G, Pt[i], q) for i, q in enumerate(qs))}
        if kind == "hf":
            sinf, gamma = x.hf(G)
            return {"sig_inf": sinf, "gamma": gamma}
        dinf, dtau = _directions(c, seed)
        if kind == "jvp":
            dinf, dtau = x.jvp(G, dtau)
            return {"d_inf": dinf, "d_tau": dtau}
        return {"G_bar": x.vjp(G, dinf, dtau)}
