"""Workloads of the Newton-system library that performance is measured on.

A case is one pass of what a user's program does with a packed arrowhead LP:

  newton    one interior-point iteration's linear algebra: factor at an iterate
            (x, z), then the predictor's and the corrector's solve
  refined   factor, then one solve refined in FP64 on the unregularized system
            (FP64 or FP32 factors; with upper bounds the Q-system)
  gradient  derivatives at a point whose factors are held: one gradient (the
            transposed solve) and two directional derivatives, all refined
  ipm       a whole interior-point solve from its own start point, with a budget
            of eight iterations (a rolling horizon's or a decomposition's solve)

Sizes: the time-block shapes of gen.py's workloads (tiny, n512, uneven, sens,
mid_b) and block counts and ragged shapes in between; m_i ~ U{m_lo..m_hi},
n_i = 2 m_i, link pairs l_j ~ U{l_lo..l_hi}, n0 linking variables, ng global
rows.  A_i and C_i have the stated share of nonzeros and are handed over dense,
as the library takes them; every row of A_i has at least one nonzero.

Iterates lie near the central path at complementarity mu: in each block half
of the variables are large (x ~ U[0.5, 2], z = mu / x), the others small
(z ~ U[0.5, 2], x = mu / z), each product disturbed by up to 30%.
"""
from types import SimpleNamespace

import numpy as np
import torch

from paper_2412_07731_amd import ahlp, autodiff

RHO, DELTA = 1e-8, 1e-6   # the library's default regularization


def _case(kind, N, m, l, n0, density, ng=0, mu=1e-2, fp32=False, bounded=False):
    return dict(kind=kind, N=N, m_lo=m[0], m_hi=m[1], l_lo=l[0], l_hi=l[1], n0=n0, ng=ng,
                density=density, mu=mu, fp32=fp32, bounded=bounded)


def listed():
    def named(name, *a, **k):
        return dict(_case(*a, **k), name=name)
    return [
        # a model of a few small periods, solved often: launches and latency count
        named("tiny newton", "newton", 8, (32, 32), (4, 4), 8, 0.30),
        named("tiny ipm", "ipm", 8, (32, 32), (4, 4), 8, 0.30),
        # many small ragged periods, as in models cut into hours or days
        named("hourly newton", "newton", 2190, (20, 60), (2, 8), 12, 0.15),
        # a mid-size model with bounds and global rows, solved to full accuracy
        named("ragged refined", "refined", 47, (70, 150), (3, 15), 5, 0.50, ng=3, bounded=True),
        # the benchmark shape: one iteration, with FP32 factors, and a whole solve
        named("n512 newton", "newton", 512, (256, 256), (16, 16), 32, 0.10),
        named("n512 fp32", "refined", 512, (256, 256), (16, 16), 32, 0.10, fp32=True),
        named("n512 ipm", "ipm", 512, (256, 256), (16, 16), 32, 0.10),
        # blocks of very different sizes with wide borders
        named("uneven newton", "newton", 512, (64, 512), (4, 32), 64, 0.10),
        # few tall blocks with dense data
        named("tall newton", "newton", 48, (600, 900), (8, 24), 16, 1.0),
        # many quantities carried between periods: pairs of more than 32 rows
        named("wide newton", "newton", 96, (100, 160), (33, 56), 24, 0.25),
        # differentiating a solution with respect to the data
        named("sens gradient", "gradient", 256, (256, 256), (16, 16), 0, 0.10),
        # upper bounds inside the iteration, global rows in the border
        named("bounded ipm", "ipm", 64, (96, 96), (8, 8), 16, 0.10, ng=6, bounded=True),
    ]


def draw(rng):
    def span(lo, hi):   # log-uniform whole number
        return int(round(lo * (hi / lo) ** rng.random()))

    kind = rng.choice(["newton", "newton", "newton", "refined", "gradient", "ipm"])
    m_hi = span(20, 900)
    m_lo = max(16, int(m_hi * rng.uniform(0.3, 1.0)))
    most = 6.0e7 / (2.0 * m_hi * m_hi)           # at most the largest listed case's entries
    N = min(span(8, 2190), max(8, int(most)))
    l_hi = min(span(4, 56 if rng.random() < 0.25 else 32), m_lo)
    l_lo = max(1, int(l_hi * rng.uniform(0.2, 1.0)))
    if l_hi > 32:   # wide pairs: fewer of them
        N = min(N, 96)
    n0 = 0 if kind == "gradient" else rng.randint(1, 64 if l_hi <= 32 else 16)
    ng = rng.choice([0, 0, rng.randint(1, 8)]) if n0 <= 48 else 0
    density = max(round(0.05 * 20.0 ** rng.random(), 3), min(1.0, 6.0 / m_lo))
    return _case(kind, N, (m_lo, m_hi), (l_lo, l_hi), n0, density, ng=ng,
                 mu=10.0 ** rng.uniform(-3, 0), fp32=kind == "refined" and rng.random() < 0.5,
                 bounded=kind in ("refined", "ipm") and rng.random() < 0.4)


def _sizes(case):
    """m_i and l_j, the same for every seed."""
    rs = np.random.RandomState(1)
    m = rs.randint(case["m_lo"], case["m_hi"] + 1, case["N"])
    return m, rs.randint(case["l_lo"], case["l_hi"] + 1, case["N"] - 1)


def _instance(case, seed):
    """The LP (host arrays, as the library takes it) and a random source on the GPU."""
    rs = np.random.RandomState(seed)
    g = torch.Generator(device="cuda").manual_seed(seed)

    def uni(size, lo=0.0, hi=1.0):
        return torch.rand(size, generator=g, device="cuda", dtype=torch.float64) * (hi - lo) + lo

    N, n0, ng = case["N"], case["n0"], case["ng"]
    m, l = _sizes(case)
    n = 2 * m

    def sparse(count):
        v = uni(count, -1.0, 1.0)
        keep = torch.rand(count, generator=g, device="cuda") < case["density"]
        return v * keep

    A = sparse(int((m * n).sum()))
    # entry (r, r) of every block: no empty row
    rows = np.arange(int(m.sum())) - np.repeat(np.cumsum(m) - m, m)
    first = np.repeat(np.cumsum(m * n) - m * n, m) + rows * np.repeat(n, m) + rows
    A[torch.from_numpy(first).cuda()] = uni(len(first), 0.5, 1.0)
    A = A.cpu().numpy()
    C = sparse(int(m.sum()) * n0).cpu().numpy()
    cut_a, cut_c = np.cumsum(m * n)[:-1], np.cumsum(m * n0)[:-1]
    FR, FL = [], []
    for j in range(N - 1):   # storage continuity: the last l_j columns of block j, the first of j + 1
        k = np.arange(l[j])
        FR.append(np.zeros((l[j], n[j])))
        FL.append(np.zeros((l[j], n[j + 1])))
        FR[j][k, n[j] - l[j] + k] = 1.0
        FL[j][k, k] = -1.0
    Wg = Wg0 = None
    if ng:
        Wg = [np.zeros((ng, k)) for k in n]
        for W in Wg:
            for r in range(ng):
                W[r, rs.choice(W.shape[1], 3, replace=False)] = rs.uniform(-1.0, 1.0, 3)
        Wg0 = rs.uniform(-1.0, 1.0, (ng, n0)) * (rs.rand(ng, n0) < 0.5) if n0 else None
    inst = SimpleNamespace(N=N, n0=n0, m=m, n=n, l=l,
                           A=[a.reshape(p, q) for a, p, q in zip(np.split(A, cut_a), m, n)],
                           C=[a.reshape(p, n0) for a, p in zip(np.split(C, cut_c), m)],
                           FR=FR, FL=FL, F0=None, Wg=Wg, Wg0=Wg0, ub=None)
    inst.n_tot, inst.m_tot = int(n.sum()) + n0, int(m.sum()) + int(l.sum()) + ng
    inst.b, inst.c = np.zeros(inst.m_tot), np.zeros(inst.n_tot)
    if case["kind"] == "ipm":
        _optimum(inst, case, rs)
    return inst, uni, rs


def _apply(inst, x, y):
    """(A x, A'y) with the whole constraint matrix."""
    xo, yo = np.concatenate([[0], np.cumsum(inst.n)]), np.concatenate([[0], np.cumsum(inst.m)])
    lo = yo[-1] + np.concatenate([[0], np.cumsum(inst.l)])
    x0 = x[xo[-1]:]
    ax, aty = np.zeros(inst.m_tot), np.zeros(inst.n_tot)
    for i in range(inst.N):
        s, t = slice(xo[i], xo[i + 1]), slice(yo[i], yo[i + 1])
        ax[t] = inst.A[i] @ x[s] + inst.C[i] @ x0
        aty[s] += inst.A[i].T @ y[t]
        aty[xo[-1]:] += inst.C[i].T @ y[t]
    for j in range(inst.N - 1):
        s, s2, t = slice(xo[j], xo[j + 1]), slice(xo[j + 1], xo[j + 2]), slice(lo[j], lo[j + 1])
        ax[t] = inst.FR[j] @ x[s] + inst.FL[j] @ x[s2]
        aty[s] += inst.FR[j].T @ y[t]
        aty[s2] += inst.FL[j].T @ y[t]
    if inst.Wg is not None:
        yg = y[lo[-1]:]
        for i in range(inst.N):
            s = slice(xo[i], xo[i + 1])
            ax[lo[-1]:] += inst.Wg[i] @ x[s]
            aty[s] += inst.Wg[i].T @ yg
        if inst.n0:
            ax[lo[-1]:] += inst.Wg0 @ x0
            aty[xo[-1]:] += inst.Wg0.T @ yg
    return ax, aty


def _optimum(inst, case, rs):
    """b, c (and upper bounds) of a feasible LP with a finite optimum: half of the variables positive."""
    nt = inst.n_tot
    big = np.zeros(nt, bool)
    at = 0
    for k in list(inst.n) + [inst.n0]:   # exactly half of every block's variables, and of x_0's
        big[at + rs.permutation(k)[:k // 2]] = True
        at += k
    x = np.where(big, rs.uniform(0.5, 2.0, nt), 0.0)
    z = np.where(big, 0.0, rs.uniform(0.5, 2.0, nt))
    inst.b, aty = _apply(inst, x, rs.standard_normal(inst.m_tot))
    inst.c = aty + z
    if case["bounded"]:   # 40% of the variables, half of those that are positive at their bound
        at = big & (rs.rand(nt) < 0.5)
        inst.ub = np.where(rs.rand(nt) < 0.4, x + np.where(at, 0.0, rs.uniform(0.5, 2.0, nt)), np.inf)
        inst.c = inst.c - np.where(at & np.isfinite(inst.ub), rs.uniform(0.5, 2.0, nt), 0.0)


def _point(case, inst, uni):
    nt, mt, mu = inst.n_tot, inst.m_tot, case["mu"]
    big = uni(nt) < 0.5
    v, off = uni(nt, 0.5, 2.0), uni(nt, 0.7, 1.3)
    x = torch.where(big, v, mu * off / v)
    z = torch.where(big, mu * off / v, v)
    p = SimpleNamespace(x=x, z=z, q=None)
    if case["bounded"]:   # w / s of the bounded variables
        p.q = torch.where(uni(nt) < 0.4, mu ** uni(nt, -1.0, 1.0), 0.0 * v)
    p.rx, p.ry, p.rz = uni(nt, -1.0, 1.0), uni(mt, -1.0, 1.0), -x * z
    p.rz2 = p.rz + 0.1 * mu - mu * uni(nt, -0.5, 0.5)
    p.gx, p.db, p.dc = uni(nt, -1.0, 1.0), uni(mt, -1.0, 1.0), uni(nt, -1.0, 1.0)
    return p


def prepare(case, seed):
    inst, uni, _ = _instance(case, seed)
    s = SimpleNamespace(case=case, prob=ahlp.Problem(inst))
    if case["kind"] != "ipm":
        s.at = _point(case, inst, uni)
    if case["kind"] == "gradient":
        s.prob.set_bc(s.at.db, s.at.dc)
        s.prob.factor(s.at.x, s.at.z, rho=RHO, delta=DELTA)
    return s


def run(s):
    p, kind = s.prob, s.case["kind"]
    if kind == "ipm":
        x, y, z, res = p.ipm(tol=1e-3, max_iter=8)
        return {"x": x, "y": y, "z": z, "objective": res["primal_obj"]}
    a = s.at
    if kind == "newton":
        p.factor(a.x, a.z, rho=RHO, delta=DELTA)
        pred = p.solve(a.rx, a.ry, a.rz)[:3]
        corr = p.solve(a.rx, a.ry, a.rz2)[:3]
        return {"pred": pred, "corr": corr}
    if kind == "refined":
        prec = ahlp.FP32_REFINE if s.case["fp32"] else ahlp.FP64
        if a.q is None:
            p.factor(a.x, a.z, rho=RHO, delta=DELTA, precision=prec)
        else:
            p.factor_bounded(a.x, a.z, a.q, rho=RHO, delta=DELTA, precision=prec)
        return {"dir": p.solve(a.rx, a.ry, a.rz, max_refine=10, refine_tol=1e-13)[:3]}
    gb, gc, _ = p.lp_gradient(a.gx, 0.5)
    one = autodiff.jvp(p, a.db, a.dc)
    two = autodiff.jvp(p, a.ry, a.rx)
    return {"grad_b": gb, "grad_c": gc, "one": one, "two": two}


def work(case):
    """Nonzeros of A and C, vectors, dense factors of the blocks and of S (LAPACK counts)."""
    m, l = _sizes(case)
    m, l = m.astype(float), float(l.mean())
    n, N, d, nb = 2 * m, case["N"], case["density"], case["n0"] + case["ng"]
    k = 2 * l + nb
    nnz = float((d * m * n + m).sum() + d * m.sum() * case["n0"])
    vec = float(n.sum() + m.sum() + N * l + nb)
    syrk = float((m * m * n * d * d).sum())
    chol = float((m ** 3 / 3 + m * m * k + k * (k + 1) * m).sum()) + (N - 1) * (l ** 3 / 3 + 6 * l ** 3 + 4 * l * l * nb)
    solve = 4.0 * nnz + float((2 * m * m + 4 * m * k).sum()) + (N - 1) * (10 * l * l + 4 * l * nb)
    factors, solves = {"newton": (1, 2), "refined": (1, 1), "gradient": (0, 3), "ipm": (9, 18)}[case["kind"]]
    outs = 1 if case["kind"] == "ipm" else solves
    return {"bytes": 8.0 * (nnz + 2 * vec + 2.5 * vec * outs),
            "flops": factors * (syrk + chol) + solves * solve}


# ------------------------------------------------------------------ 64-bit reference
def _newton64(inst, x, z, q, rhs, rho, delta):
    """Newton directions for several (rx, ry, rz), by block elimination of the normal equations
    (A D A' + delta I on every dual row, D = (z/x + q + rho)^-1) with one correction step."""
    N, n0, ng = inst.N, inst.n0, 0 if inst.Wg is None else inst.Wg[0].shape[0]
    xo, yo = np.concatenate([[0], np.cumsum(inst.n)]), np.concatenate([[0], np.cumsum(inst.m)])
    lo = np.concatenate([[0], np.cumsum(inst.l)])
    nl, nb, l = lo[-1], ng + n0, inst.l
    D = 1.0 / (z / x + q + rho)
    # S over the pairs (block tridiagonal T, couplings U) and the border (global rows, x_0)
    T = [delta * np.eye(k) for k in l]
    U = [np.zeros((l[j + 1], l[j])) for j in range(N - 2)]
    E = [np.zeros((k, nb)) for k in l]
    S00 = np.diag(np.concatenate([np.full(ng, delta), -1.0 / D[xo[-1]:]]))
    if ng and n0:
        S00[:ng, ng:], S00[ng:, :ng] = inst.Wg0, inst.Wg0.T
    Li, W, F = [], [], []
    for i in range(N):
        lL, lR = l[i - 1] if i else 0, l[i] if i < N - 1 else 0
        F.append(np.concatenate([inst.FL[i - 1] if i else np.zeros((0, inst.n[i])),
                                 inst.FR[i] if i < N - 1 else np.zeros((0, inst.n[i])),
                                 inst.Wg[i] if ng else np.zeros((0, inst.n[i]))]))
        d = D[xo[i]:xo[i + 1]]
        AD = inst.A[i] * d
        Li.append(np.linalg.inv(np.linalg.cholesky(AD @ inst.A[i].T + delta * np.eye(inst.m[i]))))
        W.append(Li[i] @ np.concatenate([AD @ F[i].T, inst.C[i]], axis=1))
        G = -W[i].T @ W[i]
        G[:len(F[i]), :len(F[i])] += (F[i] * d) @ F[i].T
        a, b, c = slice(0, lL), slice(lL, lL + lR), slice(lL + lR, None)
        if lL:
            T[i - 1] += G[a, a]
            E[i - 1] += G[a, c]
        if lR:
            T[i] += G[b, b]
            E[i] += G[b, c]
        if lL and lR:
            U[i - 1] += G[b, a]
        S00 += G[c, c]
    border = _arrow(T, U, E, S00, lo)

    def solve(ry, rhx):   # A dx + delta dy = ry, A'dy - dx / D = rhx
        v = D * rhx
        top = np.concatenate([ry[yo[-1]:], rhx[xo[-1]:]])
        at, ts = [], []
        for i in range(N):
            s = slice(xo[i], xo[i + 1])
            at.append(np.concatenate([np.arange(lo[max(i - 1, 0)], lo[min(i + 1, N - 1)]), np.arange(nl, nl + nb)]))
            ts.append(Li[i] @ (ry[yo[i]:yo[i + 1]] + inst.A[i] @ v[s]))
            top[at[i][:len(F[i])]] += F[i] @ v[s]
            top[at[i]] -= W[i].T @ ts[i]
        u = border(top)
        dy = np.concatenate([Li[i].T @ (ts[i] - W[i] @ u[at[i]]) for i in range(N)] + [u[:nl + ng]])
        dx = D * (_apply(inst, np.zeros(inst.n_tot), dy)[1] - rhx)
        dx[xo[-1]:] = u[nl + ng:]
        return dx, dy

    out = []
    for rx, ry, rz in rhs:
        h = rx - rz / x
        dx, dy = solve(ry, h)
        for _ in range(2):   # corrections of the reduced system
            ax, aty = _apply(inst, dx, dy)
            ex, ey = solve(ry - ax - delta * dy, h - (aty - dx / D))
            dx, dy = dx + ex, dy + ey
        out.append((dx, dy, (rz - z * dx) / x))
    return out


def _arrow(T, U, E, S00, lo):
    """Solver for the block tridiagonal (T, U) with the border (E, S00)."""
    P, nl = len(T), lo[-1]
    T, E, inv, low = list(T), list(E), [], []
    for j in range(P):
        inv.append(np.linalg.inv(T[j]))
        S00 = S00 - E[j].T @ inv[j] @ E[j]
        if j + 1 < P:
            low.append(U[j] @ inv[j])
            T[j + 1] = T[j + 1] - low[j] @ U[j].T
            E[j + 1] = E[j + 1] - low[j] @ E[j]

    def solve(r):
        w = [r[lo[j]:lo[j + 1]].copy() for j in range(P)]
        w0 = r[nl:].copy()
        for j in range(P):
            w0 -= E[j].T @ (inv[j] @ w[j])
            if j + 1 < P:
                w[j + 1] -= low[j] @ w[j]
        u0 = np.linalg.solve(S00, w0)
        u = [None] * P
        for j in range(P - 1, -1, -1):
            u[j] = inv[j] @ (w[j] - E[j] @ u0)
            if j + 1 < P:
                u[j] -= low[j].T @ u[j + 1]
        return np.concatenate(u + [u0])
    return solve


def exact(case, seed):
    if case["kind"] == "ipm":
        return None   # the end point depends on the path to it
    inst, uni, _ = _instance(case, seed)
    a = _point(case, inst, uni)
    f = {k: v.cpu().numpy() for k, v in vars(a).items() if v is not None}
    q = f.get("q", 0.0)
    if case["kind"] == "newton":
        one, two = _newton64(inst, f["x"], f["z"], q, [(f["rx"], f["ry"], f["rz"]), (f["rx"], f["ry"], f["rz2"])],
                             RHO, DELTA)
        return {"pred": one, "corr": two}
    if case["kind"] == "refined":
        return {"dir": _newton64(inst, f["x"], f["z"], q, [(f["rx"], f["ry"], f["rz"])], 0.0, 0.0)[0]}
    # K' w = (g, 0, 0) is the Newton system's direction with rz = z * 0
    zx = np.zeros(inst.n_tot)
    g = f["gx"] + 0.5 * f["dc"]
    grad, one, two = _newton64(inst, f["x"], f["z"], 0.0,
                               [(g, np.zeros(inst.m_tot), zx), (f["dc"], f["db"], zx), (f["rx"], f["ry"], zx)], 0.0, 0.0)
    return {"grad_b": grad[1], "grad_c": grad[0] + 0.5 * f["x"], "one": one, "two": two}
