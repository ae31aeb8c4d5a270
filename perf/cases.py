"""The workloads this library is timed on: what a user's program has it do, through its Python
interface, over the sizes its configurations and benchmark use.

A case is a dict of plain values. listed() gives the named cases, draw(rng) one more of the same
ranges, prepare(case, seed) the inputs and the staged context on the GPU, run(state) one pass,
work(case) the bytes and operations a pass cannot do without, exact(case, seed) the pass's result
from plain FP64 torch / numpy.

Inputs follow the library's synthetic stand-in for molecular density-fitting integrals: occupied
energies U[-1, -0.3], virtual energies U[0, 3], L^P_pq symmetric normal with standard deviation
0.21 / sqrt(naux) (the scale at which the pencils of every size here are definite).
"""
import math

import numpy as np
import torch

import paper_2512_12515_amd as P

BYTES = {"fp64": 8, "fp32": 4, "bf16x6": 6, "bf16x3": 4}  # bytes read per staged integral


def listed():
    return [
        # the smallest call: one trial vector of a small molecule, where launches and latency count
        dict(name="sigma small, 1 vector", kind="sigma", nocc=5, nvir=20, naux=100, mult="singlet",
             prec="fp64", k=1),
        # a few trial vectors of a mid-sized system of no round size
        dict(name="sigma ragged, 7 vectors", kind="sigma", nocc=13, nvir=117, naux=457,
             mult="triplet", prec="fp64", k=7),
        # the block product of the ordinary FP64 solve
        dict(name="sigma 20/200/700 fp64", kind="sigma", nocc=20, nvir=200, naux=700,
             mult="singlet", prec="fp64", k=20),
        # the block product of the headline FP64 solve, the largest call
        dict(name="sigma 50/500/1800 fp64", kind="sigma", nocc=50, nvir=500, naux=1800,
             mult="singlet", prec="fp64", k=20),
        # mixed precision: the largest request of the serving mix (FP32, its default precision)
        dict(name="sigma 40/400/1540 fp32", kind="sigma", nocc=40, nvir=400, naux=1540,
             mult="triplet", prec="fp32", k=12),
        # mixed precision: six- and three-product BF16 splits at the large sizes they are meant for
        dict(name="sigma 50/500/1800 bf16x6", kind="sigma", nocc=50, nvir=500, naux=1800,
             mult="singlet", prec="bf16x6", k=20),
        dict(name="sigma 40/400/1540 bf16x3", kind="sigma", nocc=40, nvir=400, naux=1540,
             mult="triplet", prec="bf16x3", k=16),
        # spin-unrestricted: the density-fitted alpha-beta sector
        dict(name="sigma alpha-beta 200/20/18", kind="sigma_ab", nmo=200, nocc_a=20, nocc_b=18,
             naux=700, prec="fp64", k=16),
        # a whole Davidson solve of the ordinary size
        dict(name="davidson 20/200/700", kind="davidson", nocc=20, nvir=200, naux=700,
             mult="triplet", nroot=10, block=20),
        # the direct solve of a small molecule: its lowest roots with their vectors
        dict(name="direct 5/20/100", kind="direct", nocc=5, nvir=20, naux=100, mult="singlet",
             nroot=5, channel="pp"),
        # the correlation energy of one spin block from its whole spectrum
        dict(name="energy 8/45/150", kind="energy", nocc=8, nvir=45, naux=150, mult="singlet"),
        # analysis of the roots of an ordinary solve: NTO weights and density blocks
        dict(name="nto 20/200, 10 roots", kind="nto", nocc=20, nvir=200, mult="singlet", k=10),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _naux(rng, nmo):
    return max(20, min(1800, int(nmo * rng.uniform(3.0, 4.0))))


def draw(rng):
    kind = rng.choice(["sigma"] * 5 + ["sigma_ab", "davidson", "direct", "energy", "nto"])
    mult = rng.choice(["singlet", "triplet"])
    if kind == "sigma":
        nocc, nvir = _log_int(rng, 4, 50), _log_int(rng, 20, 500)
        return dict(kind=kind, nocc=nocc, nvir=nvir, naux=_naux(rng, nocc + nvir), mult=mult,
                    prec=rng.choice(["fp64", "fp64", "fp32", "bf16x6", "bf16x3"]),
                    k=_log_int(rng, 1, 20))
    if kind == "sigma_ab":
        nmo, nocc = _log_int(rng, 30, 240), _log_int(rng, 4, 24)
        return dict(kind=kind, nmo=nmo, nocc_a=nocc, nocc_b=max(1, nocc - rng.randrange(3)),
                    naux=_naux(rng, nmo), prec=rng.choice(["fp64", "fp64", "fp32", "bf16x6", "bf16x3"]),
                    k=_log_int(rng, 1, 20))
    if kind == "davidson":
        nocc, nvir, nroot = _log_int(rng, 5, 20), _log_int(rng, 30, 200), rng.randrange(3, 13)
        return dict(kind=kind, nocc=nocc, nvir=nvir, naux=_naux(rng, nocc + nvir), mult=mult,
                    nroot=nroot, block=rng.choice([nroot, min(20, 2 * nroot)]))
    if kind == "nto":
        return dict(kind=kind, nocc=_log_int(rng, 4, 40), nvir=_log_int(rng, 20, 400), mult=mult,
                    k=_log_int(rng, 1, 16))
    nocc, nvir = _log_int(rng, 4, 9), _log_int(rng, 10, 62)
    case = dict(kind=kind, nocc=nocc, nvir=nvir, naux=_naux(rng, nocc + nvir), mult=mult)
    if kind == "direct":
        case.update(nroot=rng.randrange(1, 7), channel=rng.choice(["pp", "pp", "hh"]))
    return case


def _pairs(m, mult):
    return m * (m + 1) // 2 if mult == "singlet" else m * (m - 1) // 2


def _order(case):
    if case["kind"] == "sigma_ab":
        a, b, nmo = case["nocc_a"], case["nocc_b"], case["nmo"]
        return (nmo - a) * (nmo - b) + a * b
    return _pairs(case["nvir"], case["mult"]) + _pairs(case["nocc"], case["mult"])


def _generator(seed, stream):
    return torch.Generator(device="cuda").manual_seed(int(seed) * 16 + stream)


def _eps(nocc, nvir, g):
    u = torch.rand(nocc + nvir, generator=g, device="cuda", dtype=torch.float64)
    occ, vir = torch.sort(-1.0 + 0.7 * u[:nocc])[0], torch.sort(3.0 * u[nocc:])[0]
    return torch.cat([occ, vir])


def _integrals(naux, nmo, g):
    x = torch.randn(naux, nmo, nmo, generator=g, device="cuda", dtype=torch.float64)
    x = torch.triu(x.mul_(0.21 / math.sqrt(naux)))
    return x + torch.triu(x, 1).transpose(1, 2)


def _vectors(k, n, g):
    z = torch.randn(k, n, generator=g, device="cuda", dtype=torch.float64)
    return z / z.norm(dim=1, keepdim=True)


def _roots(case, g):
    """Packed vectors like computed roots: a few large pairs over a small background, scaled to
    x.x - y.y = 1."""
    npp, nhh = _pairs(case["nvir"], case["mult"]), _pairs(case["nocc"], case["mult"])
    x = torch.randn(case["k"], npp, generator=g, device="cuda", dtype=torch.float64)
    y = torch.randn(case["k"], nhh, generator=g, device="cuda", dtype=torch.float64)
    fall = torch.arange(npp, device="cuda", dtype=torch.float64).add_(1.0).pow_(-0.75)
    x *= fall
    x /= x.norm(dim=1, keepdim=True)
    y *= 0.1 / y.norm(dim=1, keepdim=True).clamp_min(1e-300)
    x *= (1.0 + (y * y).sum(1, keepdim=True)).sqrt()
    return torch.cat([x, y], 1).contiguous()


def _inputs(case, seed):
    """The numbers of a case: energies, integrals and vectors, all FP64."""
    kind = case["kind"]
    if kind == "nto":  # the analysis reads the vectors only: any integrals of the same orbitals do
        return (_eps(case["nocc"], case["nvir"], _generator(seed, 0)),
                _integrals(2, case["nocc"] + case["nvir"], _generator(seed, 1)),
                _roots(case, _generator(seed, 2)))
    if kind == "sigma_ab":
        nmo, naux = case["nmo"], case["naux"]
        ea = _eps(case["nocc_a"], nmo - case["nocc_a"], _generator(seed, 0))
        eb = _eps(case["nocc_b"], nmo - case["nocc_b"], _generator(seed, 3))
        La, Lb = _integrals(naux, nmo, _generator(seed, 1)), _integrals(naux, nmo, _generator(seed, 4))
        return ea, eb, La, Lb, _vectors(case["k"], _order(case), _generator(seed, 2))
    eps = _eps(case["nocc"], case["nvir"], _generator(seed, 0))
    L = _integrals(case["naux"], case["nocc"] + case["nvir"], _generator(seed, 1))
    z = _vectors(case["k"], _order(case), _generator(seed, 2)) if kind == "sigma" else None
    return eps, L, z


def prepare(case, seed):
    """Inputs and the staged context: what a program keeps from call to call."""
    kind = case["kind"]
    if kind == "sigma_ab":
        ea, eb, La, Lb, z = _inputs(case, seed)
        torch.cuda.synchronize()  # the context is built on a stream of its own
        ctx = P.PpRPA.alpha_beta(ea, eb, La, Lb, case["nocc_a"], case["nocc_b"],
                                 density_fitted=True, prec=case["prec"])
        return dict(case=case, ctx=ctx, z=z)
    eps, L, z = _inputs(case, seed)
    torch.cuda.synchronize()
    ctx = P.PpRPA(eps, L, case["nocc"], mult=case["mult"], prec=case.get("prec", "fp64"),
                  dense=kind in ("direct", "energy"))
    return dict(case=case, ctx=ctx, z=z.cpu().numpy() if kind == "nto" else z)


def run(state):
    case, ctx = state["case"], state["ctx"]
    kind = case["kind"]
    if kind in ("sigma", "sigma_ab"):
        s = ctx.matvec(state["z"])
        # a reduced-precision product carries FP32 accuracy: the program goes on in FP32
        return s if case["prec"] == "fp64" else s.float()
    if kind == "davidson":
        return ctx.davidson(case["nroot"], block=case["block"], tol=1e-6, max_iter=200)["omega"]
    if kind == "direct":
        r = ctx.davidson(case["nroot"], direct=True, vectors=True, channel=case["channel"])
        return dict(omega=r["omega"], vecs=r["vecs"])
    if kind == "energy":
        return ctx.correlation_energy()
    return ctx.nto(state["z"])


def work(case):
    kind, n = case["kind"], _order(case)
    if kind == "sigma_ab":
        nmo, naux, k = case["nmo"], case["naux"], case["k"]
        # both spins' symmetric integrals once, the vectors in and out
        b = naux * nmo * (nmo + 1) * BYTES[case["prec"]] + 16 * k * n
        return dict(bytes=b, flops=4 * naux * n * nmo * k)
    nocc, nvir = case["nocc"], case["nvir"]
    nmo = nocc + nvir
    if kind == "nto":
        k = case["k"]
        sq = nvir * nvir + nocc * nocc
        cub = nvir ** 3 + nocc ** 3
        # vectors in, weights and densities out; T T^t, T^t T (halves) and the tridiagonal forms
        return dict(bytes=8 * k * (n + sq + nmo), flops=k * (2 * cub + 4 * cub // 3))
    if kind in ("direct", "energy"):
        # the matrix once; Cholesky, the reduced matrix and its tridiagonal form
        out = case.get("nroot", 0) * n
        return dict(bytes=8 * (n * n + out), flops=n ** 3 // 3 + n ** 3 + 4 * n ** 3 // 3)
    naux = case["naux"]
    per_vector = 3 * naux * nmo * (nvir * nvir + nocc * nocc)  # triangle of one contraction, the other
    integrals = naux * nmo * (nmo + 1) // 2
    if kind == "davidson":
        # about ten products for each root from a diagonal guess, in blocks
        k = 10 * case["nroot"]
        return dict(bytes=8 * integrals * -(-k // case["block"]) + 16 * k * n, flops=per_vector * k)
    k = case["k"]
    return dict(bytes=integrals * BYTES[case["prec"]] + 16 * k * n, flops=per_vector * k)


# ---- the same results in plain FP64 ---------------------------------------------------------------


def _blocks(case, z):
    """Z = blockdiag over [occupied; virtual] orbitals of the packed vectors, its diagonal weight,
    and the index lists that pack a result again."""
    nocc, nvir, k = case["nocc"], case["nvir"], z.shape[0]
    nmo = nocc + nvir
    off = 0 if case["mult"] == "singlet" else 1
    pv = torch.triu_indices(nvir, nvir, off, device=z.device) + nocc
    po = torch.triu_indices(nocc, nocc, off, device=z.device)
    p, q = torch.cat([pv, po], 1)
    Z = torch.zeros(k, nmo, nmo, dtype=torch.float64, device=z.device)
    if case["mult"] == "singlet":
        same = (p == q).to(torch.float64)
        w = 1.0 + same * (math.sqrt(0.5) - 1.0)
        Z[:, p, q] = z * (1.0 + same * (math.sqrt(2.0) - 1.0))
        Z[:, q, p] = Z[:, p, q].clone()
    else:
        w = torch.ones_like(z[0])
        Z[:, p, q] = z
        Z[:, q, p] = -z
    return Z, p, q, w


def _energies(case, eps, p, q):
    npp = _pairs(case["nvir"], case["mult"])
    e = eps[p] + eps[q]
    e[npp:] *= -1.0
    return e


def _sandwich(La, Z, Lb):
    """sum_P La^P Z_k Lb^P for every k, a few P at a time."""
    k, ma, mb = Z.shape
    S = torch.zeros(ma, k * mb, dtype=torch.float64, device=Z.device)
    step = max(1, int(2e8 // (k * ma * mb)))
    for p0 in range(0, La.shape[0], step):
        A, B = La[p0:p0 + step], Lb[p0:p0 + step]
        np_ = A.shape[0]
        W = B.permute(1, 0, 2).reshape(mb, np_ * mb)  # [d][(P, col)]
        T = (Z.reshape(k * ma, mb) @ W).reshape(k, ma, np_, mb)
        T = T.permute(2, 1, 0, 3).reshape(np_ * ma, k * mb)  # [(P, c)][(k, col)]
        S += A.permute(1, 0, 2).reshape(ma, np_ * ma) @ T
    return S.reshape(ma, k, mb).permute(1, 0, 2)


def _dense(case, eps, L):
    """M, the pair metric's signs and 2 mu."""
    nocc = case["nocc"]
    nmo = nocc + case["nvir"]
    s = 1.0 if case["mult"] == "singlet" else -1.0
    _, p, q, w = _blocks(case, torch.zeros(1, _order(case), dtype=torch.float64, device=L.device))
    V = L.reshape(L.shape[0], nmo * nmo)
    V = (V.T @ V).reshape(nmo, nmo, nmo, nmo)
    n = p.numel()
    M = torch.empty(n, n, dtype=torch.float64, device=L.device)
    for r0 in range(0, n, 512):
        a, b = p[r0:r0 + 512, None], q[r0:r0 + 512, None]
        M[r0:r0 + 512] = (V[a, p, b, q] + s * V[a, q, b, p]) * w[r0:r0 + 512, None] * w
    M += torch.diag(_energies(case, eps, p, q))
    sign = torch.ones(n, dtype=torch.float64, device=L.device)
    sign[_pairs(case["nvir"], case["mult"]):] = -1.0
    return M.cpu().numpy(), sign.cpu().numpy(), float(eps[nocc - 1] + eps[nocc])


def _spectrum(M, sign, mu2, vectors):
    """Roots and vectors of M z = Omega W z by the definite reduction."""
    C = np.linalg.cholesky(M - mu2 * np.diag(sign))
    S = C.T @ (sign[:, None] * C)
    if not vectors:
        return np.linalg.eigvalsh(S) + mu2, None
    lam, U = np.linalg.eigh(S)
    return lam + mu2, np.linalg.solve(C.T, U) * np.sqrt(np.abs(lam))


def exact(case, seed):
    kind = case["kind"]
    if kind == "sigma_ab":
        ea, eb, La, Lb, z = _inputs(case, seed)
        na, nb, nmo, k = case["nocc_a"], case["nocc_b"], case["nmo"], case["k"]
        npp = (nmo - na) * (nmo - nb)
        Z = torch.zeros(k, nmo, nmo, dtype=torch.float64, device=z.device)
        Z[:, na:, nb:] = z[:, :npp].reshape(k, nmo - na, nmo - nb)
        Z[:, :na, :nb] = z[:, npp:].reshape(k, na, nb)
        S = _sandwich(La, Z, Lb)
        ex = (ea[na:, None] + eb[nb:]).reshape(-1)
        ey = -(ea[:na, None] + eb[:nb]).reshape(-1)
        return z * torch.cat([ex, ey]) + torch.cat([S[:, na:, nb:].reshape(k, -1),
                                                    S[:, :na, :nb].reshape(k, -1)], 1)
    eps, L, z = _inputs(case, seed)
    if kind == "sigma":
        Z, p, q, w = _blocks(case, z)
        return z * _energies(case, eps, p, q) + w * _sandwich(L, Z, L)[:, p, q]
    if kind == "nto":
        k, nv, no = case["k"], case["nvir"], case["nocc"]
        off = 0 if case["mult"] == "singlet" else 1
        npp = _pairs(nv, case["mult"])
        out = {}
        for m, part, lam, d, sgn in ((nv, z[:, :npp], "lam_p", "d_vv", 1.0), (no, z[:, npp:], "lam_h", "d_oo", -1.0)):
            X = torch.zeros(k, m, m, dtype=torch.float64)
            a, b = torch.triu_indices(m, m, off)
            X[:, a, b] = part.cpu()
            Xt = X.transpose(1, 2).contiguous()
            out[lam] = (torch.linalg.svdvals(X) ** 2).numpy()
            out[d] = (sgn * (X @ Xt + Xt @ X)).numpy()
        return out
    n = _order(case)
    if n > 2500:
        return None
    M, sign, mu2 = _dense(case, eps, L)
    npp = int((sign > 0).sum())
    roots, U = _spectrum(M, sign, mu2, kind == "direct")
    if kind == "energy":
        ta, tc = float(np.trace(M[:npp, :npp])), float(np.trace(M[npp:, npp:]))
        return dict(ec_pp=float(roots[n - npp:].sum() - ta), ec_hh=float(-roots[:n - npp].sum() - tc),
                    trace_a=ta, trace_c=tc, n_pp_roots=npp, n_hh_roots=n - npp)
    if kind == "davidson":
        return roots[n - npp:n - npp + case["nroot"]].copy()
    nroot = case["nroot"]
    cols = np.arange(n - npp, n - npp + nroot) if case["channel"] == "pp" else n - npp - 1 - np.arange(nroot)
    vecs = U[:, cols].T
    vecs *= np.sign(vecs[np.arange(nroot), np.abs(vecs).argmax(1)])[:, None]
    return dict(omega=roots[cols].copy(), vecs=vecs.copy())
