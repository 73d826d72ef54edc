"""Measured cases of the library: the calls a user's program spends its time in.

Every case goes through the public Python entry points over the C ABI, with
what such a program keeps between calls (basis, workspaces, fields, vectors)
prepared beforehand and the outputs returned whole. The kinds:

* ``apply``: y = (H - sigma) x, one realization or R interleaved ones;
* ``minres``: one linear solve, to the tolerance or (on chains whose full
  solves take seconds to minutes) for a bounded number of iterations;
* ``problems``: a disorder campaign in one call, realizations of uneven L;
* ``pairs``: sigma, the eigenpairs nearest it and their observables;
* ``grad``: the derivatives of an eigenpair (the backward direction).

A solve that runs to its tolerance of 1e-12 has a solution that does not
depend on rounding (to 1e-11), and so has one of at most 64 iterations from
L = 16 on; in between, MINRES iterates are not reproducible under a change of
summation order, so no case stops there.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2203_09732_amd as mbl
from paper_2203_09732_amd import tune

FP64, FP32 = "fp64", "fp32"


def listed():
    return [
        # the smallest call: one product on a chain of 12 sites (n = 924),
        # all launch latency, as in inner loops of small studies
        dict(name="apply_L12", kind="apply", L=12, R=0, dtype=FP64, h=3.0),
        # the largest single-GPU chain (n = 10 400 600), one realization
        dict(name="apply_L26", kind="apply", L=26, R=0, dtype=FP64, h=3.8),
        # a middling batch in the single-precision storage form
        dict(name="apply_L20_R16_fp32", kind="apply", L=20, R=16, dtype=FP32, h=3.0),
        # the benchmark's headline: 32 realizations at L = 22, tuned split
        dict(name="apply_L22_R32", kind="apply", L=22, R=32, dtype=FP64, h=3.5),
        # the inner solve of shift-invert Lanczos on one realization, to
        # 1e-12: the smaller and the larger end of what is solved one by one
        dict(name="minres_L14", kind="minres", L=14, R=0, kmax=0, h=3.0, precond="row"),
        dict(name="minres_L18", kind="minres", L=18, R=0, kmax=0, h=3.0, precond="row"),
        # the same on a chain whose vectors leave the L2 caches, bounded
        dict(name="minres_L22", kind="minres", L=22, R=0, kmax=64, h=3.5, precond="row"),
        # batched inner solves: to the tolerance with lanes that end at
        # different times, and the headline batch, bounded
        dict(name="minres_L16_R32", kind="minres", L=16, R=32, kmax=0, h=3.0, precond="row"),
        dict(name="minres_L22_R32", kind="minres", L=22, R=32, kmax=64, h=3.5, precond="row"),
        # a campaign call: realizations of uneven length and disorder
        dict(name="problems_96", kind="problems", count=96, Lmin=10, Lmax=14, nev=2, h=6.0),
        # one realization from its fields to pairs, twist overlaps and entropies
        dict(name="pairs_L14", kind="pairs", L=14, nev=4, h=3.0),
        # dE/dh and d|z|^2/dh of one eigenpair
        dict(name="grad_L14", kind="grad", L=14, h=3.0),
    ]


def draw(rng):
    kind = rng.choice(["apply", "apply", "minres", "minres", "problems", "pairs", "grad"])
    h = round(rng.uniform(1.5, 6.0), 3)
    if kind == "apply":
        L = 2 * rng.randint(4, 13)
        R, dtype = 0, rng.choice([FP64, FP64, FP32])
        if L >= 12 and rng.random() < 0.6:
            R = 2 ** rng.randint(1, 5)
            while math.comb(L, L // 2) * R > math.comb(22, 11) * 32 or (L >= 26 and R > 16):
                R //= 2
            if R < 2:
                R = 0
        return dict(kind="apply", L=L, R=R, dtype=dtype, h=h)
    if kind == "minres":
        if rng.random() < 0.5:   # to the tolerance
            R = rng.choice([0, 0, 2 ** rng.randint(1, 5)])
            L = 2 * (rng.randint(6, 7) if R else rng.randint(4, 8))
            return dict(kind="minres", L=L, R=R, kmax=0, h=max(h, 2.5),
                        precond=rng.choice(["row", "row", "id"]) if L <= 12 else "row")
        R = rng.choice([0, 2 ** rng.randint(1, 5)])
        L = 2 * rng.randint(8, 12)
        while math.comb(L, L // 2) * max(R, 1) > math.comb(22, 11) * 32:
            L -= 2
        return dict(kind="minres", L=L, R=R, kmax=rng.randint(20, 64), h=h, precond="row")
    if kind == "problems":
        Lmax = 2 * rng.randint(4, 6)
        return dict(kind="problems", count=int(round(math.exp(rng.uniform(0.0, math.log(160))))),
                    Lmin=2 * rng.randint(3, Lmax // 2), Lmax=Lmax, nev=rng.randint(1, 4),
                    h=max(h, 2.0))
    if kind == "pairs":
        return dict(kind="pairs", L=2 * rng.randint(4, 6), nev=rng.randint(1, 6), h=max(h, 2.0))
    return dict(kind="grad", L=2 * rng.randint(4, 7), h=max(h, 2.0))


# ---------------------------------------------------------------------------
# inputs

def _fields(case, rng, count):
    """Fields of `count` realizations and a shift inside each one's spectrum."""
    L = case["L"]
    f = rng.uniform(-case["h"], case["h"], (count, L))
    return f, rng.uniform(-0.6, -0.3, count)


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


class _Plain:
    """(H - sigma) in plain torch from the definition of Eq. (1): states by
    popcount, neighbours by a sorted search."""

    def __init__(self, L):
        every = torch.arange(1 << L, dtype=torch.int64, device="cuda")
        pop = torch.zeros_like(every)
        for b in range(L):
            pop += (every >> b) & 1
        self.L, self.states = L, every[pop == L // 2]
        self.n = self.states.numel()
        place = torch.full((1 << L,), -1, dtype=torch.int32, device="cuda")
        place[self.states] = torch.arange(self.n, dtype=torch.int32, device="cuda")
        del every, pop
        self.place = place

    def spin(self, j):
        return ((self.states >> j) & 1).double() - 0.5

    def diagonal(self, f):
        d = torch.zeros(self.n, dtype=torch.float64, device="cuda")
        for j in range(self.L):
            d += self.spin(j) * self.spin((j + 1) % self.L) - float(f[j]) * self.spin(j)
        return d

    def bonds(self):
        """(rows, their neighbours) of every bond's antiparallel states."""
        for j in range(self.L):
            mask = (1 << j) | (1 << ((j + 1) % self.L))
            two = self.states & mask
            rows = torch.nonzero((two != 0) & (two != mask)).ravel()
            yield rows, self.place[self.states[rows] ^ mask].long()

    def product(self, diag, x):
        """diag * x plus the exchange terms; x is (n,) or (n, R)."""
        y = diag * x
        for rows, to in self.bonds():
            y.index_add_(0, rows, x.index_select(0, to), alpha=0.5)
        return y

    def table(self):
        """Neighbour of each row per bond, n where the bond is parallel."""
        t = torch.full((self.L, self.n), self.n, dtype=torch.int64, device="cuda")
        for j, (rows, to) in enumerate(self.bonds()):
            t[j, rows] = to
        return t

    def dense(self, f):
        A = torch.diag(self.diagonal(f))
        for rows, to in self.bonds():
            A[rows, to] += 0.5
        return A

    def twist(self, U):
        """z of the columns of U."""
        theta = sum(2 * math.pi / self.L * (j + 1) * self.spin(j) for j in range(self.L))
        w = U * U
        return torch.complex(w.t() @ torch.cos(theta), w.t() @ torch.sin(theta))


def _nearest(w, sigma, nev):
    idx = torch.argsort((w - sigma).abs())[:nev]
    return idx[torch.argsort(w[idx])]


def _fix_sign(U):
    """Columns of U with their largest-magnitude entry positive."""
    top = U.gather(0, U.abs().argmax(0, keepdim=True))
    return U * torch.where(top < 0, -1.0, 1.0).to(U.dtype)


def _problem_list(case, seed):
    """Chain lengths in turn, disorder and fields from the seed."""
    rng = np.random.default_rng(seed)
    out = []
    for i in range(case["count"]):
        L = case["Lmin"] + 2 * (i % ((case["Lmax"] - case["Lmin"]) // 2 + 1))
        h = case["h"] * float(rng.choice([0.75, 1.0, 1.25]))
        out.append(dict(L=L, h=rng.uniform(-h, h, L), nev=case["nev"]))
    return out


def _eigenpair(case, seed):
    """Fields, and an eigenpair near the middle of the spectrum by Rayleigh
    quotient iteration on the dense matrix."""
    rng = np.random.default_rng(seed)
    f = rng.uniform(-case["h"], case["h"], case["L"])
    A = _Plain(case["L"]).dense(f)
    v = torch.randn(A.shape[0], dtype=torch.float64, device="cuda", generator=_gen(seed))
    E = -0.45
    eye = torch.eye(A.shape[0], dtype=torch.float64, device="cuda")
    for k in range(9):
        v = torch.linalg.solve(A - (E + 1e-13) * eye, v)
        v = v / v.norm()
        if k >= 2:   # a few steps of plain inverse iteration pick the pair first
            E = float(v @ (A @ v))
    return f, E, v.contiguous()


def prepare(case, seed):
    kind = case["kind"]
    if kind == "problems":
        return dict(case=case, problems=_problem_list(case, seed))
    if kind == "grad":
        f, E, psi = _eigenpair(case, seed)
        b = mbl.Basis(case["L"])
        return dict(case=case, basis=b, fields=f, E=E, psi=psi, ws=mbl.Workspace(b, 0))
    rng = np.random.default_rng(seed)
    L, R = case["L"], case.get("R", 0)
    f, sg = _fields(case, rng, max(R, 1))
    if kind == "pairs":
        b = mbl.Basis(L)
        mmax = min(b.n, 3 * case["nev"] + 40)
        return dict(case=case, basis=b, fields=f[0], ws=mbl.Workspace(b, mmax), mmax=mmax,
                    seed=seed)
    prec = case.get("dtype", FP64)
    dtype = torch.float64 if prec == FP64 else torch.float32
    b = mbl.Basis(L, tune.best_lo_bits(L, R, prec) if R else 0)
    state = dict(case=case, basis=b, fields=f, sigma=sg)
    shape = (b.n, R) if R else (b.n,)
    x = torch.randn(shape, dtype=torch.float64, device="cuda", generator=_gen(seed))
    if R:
        state["batch"] = mbl.Batch(b, R)
        tune.apply_schedule(state["batch"], L, R, prec)
    if kind == "apply":
        state["x"] = x.to(dtype)
        state["y"] = torch.empty_like(state["x"])
    else:
        state["b"] = x / x.norm(dim=0, keepdim=bool(R))
        if not R:
            state["ws"] = mbl.Workspace(b, 0)
    return state


# ---------------------------------------------------------------------------
# one pass

def run(state):
    case = state["case"]
    kind, R = case["kind"], case.get("R", 0)
    if kind == "apply":
        if R:
            return mbl.apply_H_batched(state["basis"], state["batch"], state["fields"],
                                       state["sigma"], state["x"], state["y"])
        return mbl.apply_H(state["basis"], state["fields"][0], state["sigma"][0], state["x"],
                           state["y"])
    if kind == "minres":
        # a bounded solve cannot reach its tolerance, so it takes kmax iterations
        kw = dict(tol=1e-12) if case["kmax"] == 0 else dict(tol=1e-30, kmax=case["kmax"])
        if R:
            x, its, phi, _ = mbl.minres_solve_batched(state["basis"], state["batch"],
                                                      state["fields"], state["sigma"], state["b"],
                                                      precond=case["precond"], **kw)
            return dict(x=x) if case["kmax"] == 0 else dict(x=x, iters=its, phi=phi)
        x, info = mbl.minres_solve(state["basis"], state["fields"][0], state["sigma"][0],
                                   state["b"], precond=case["precond"], ws=state["ws"], **kw)
        return dict(x=x) if case["kmax"] == 0 else dict(x=x, iters=info.iters, phi=abs(info.phi))
    if kind == "problems":
        _, res = mbl.si_lanczos_problems(state["problems"], seed=11)
        out = {}
        for L in sorted({r.L for r in res}):
            of = [r for r in res if r.L == L]
            out["L%d" % L] = dict(sigma=np.array([r.sigma for r in of]),
                                  evals=np.stack([r.evals for r in of]),
                                  z=np.stack([r.z for r in of]),
                                  evecs=_fix_sign(torch.cat([r.evecs for r in of], 1)))
        return out
    if kind == "pairs":
        b = state["basis"]
        lo, hi, sg = mbl.sigma_midpoint(b, state["fields"])
        res = mbl.si_lanczos(b, state["fields"], sg, case["nev"], mmax=state["mmax"],
                             escale=max(abs(lo), abs(hi)), seed=state["seed"], ws=state["ws"])
        return dict(emin=lo, emax=hi, sigma=sg, evals=res.evals, evecs=_fix_sign(res.evecs),
                    z=mbl.twist_expect(b, res.evecs), S=mbl.entanglement_entropy(b, res.evecs))
    dE, dz2, z, _ = mbl.eig_grad(state["basis"], state["fields"], state["E"], state["psi"],
                                 tol=1e-12, ws=state["ws"])
    return dict(dE=dE, dz2=dz2, z=np.array([z]))


# ---------------------------------------------------------------------------
# what a pass cannot do without

def work(case):
    """Products: x read, y written. A MINRES iteration: q_k, q_{k-1}, two
    search directions and x read, q_{k+1}, one direction and x written (8
    vectors), one product's arithmetic and 20 operations per element. Solves to
    the tolerance take about n iterations, and a few eigenpairs about
    nev * 3 + 10 solves."""
    kind = case["kind"]
    size = 4 if case.get("dtype") == FP32 else 8

    def solve(L, its, R=1):
        n = math.comb(L, L // 2)
        return np.array([its * 64.0 * n * R, its * (L + 26.0) * n * R])

    if kind == "apply":
        L, R = case["L"], max(case["R"], 1)
        n = math.comb(L, L // 2)
        return dict(bytes=2.0 * size * n * R, flops=(L + 6.0) * n * R)
    if kind == "minres":
        its = case["kmax"] or math.comb(case["L"], case["L"] // 2)
        w = solve(case["L"], its, max(case["R"], 1))
    elif kind == "grad":
        w = solve(case["L"], math.comb(case["L"], case["L"] // 2))
    elif kind == "pairs":
        w = solve(case["L"], (3 * case["nev"] + 10) * math.comb(case["L"], case["L"] // 2))
    else:
        Ls = range(case["Lmin"], case["Lmax"] + 1, 2)
        w = sum(solve(L, (3 * case["nev"] + 10) * math.comb(L, L // 2)) for L in Ls)
        w = w * case["count"] / len(Ls)
    return dict(bytes=float(w[0]), flops=float(w[1]))


# ---------------------------------------------------------------------------
# the same in plain 64-bit torch

def _minres_plain(P, case, f, sg, b):
    """Alg. 2 for a fixed number of iterations; columns of b are realizations."""
    diag = torch.stack([P.diagonal(fr) - float(s) for fr, s in zip(f, sg)], 1)
    nanti = sum((P.spin(j) * P.spin((j + 1) % P.L) < 0).double() for j in range(P.L))
    m = torch.sqrt(diag * diag + 0.25 * nanti[:, None])
    table = P.table() if P.n * P.L <= 4e7 else None

    def product(v):
        if table is None:
            return P.product(diag, v)
        y, ext = diag * v, torch.cat([v, torch.zeros_like(v[:1])])
        for j in range(P.L):
            y += 0.5 * ext[table[j]]
        return y

    z0, z = torch.zeros_like(b), b
    q = z / m
    d1, d2, x = torch.zeros_like(b), torch.zeros_like(b), torch.zeros_like(b)
    beta0, beta = torch.ones_like(b[0]), (q * z).sum(0).sqrt()
    c, s = torch.ones_like(beta), torch.zeros_like(beta)
    dhat, eps, phi = torch.zeros_like(beta), torch.zeros_like(beta), beta
    for _ in range(case["kmax"]):
        p = product(q)
        alpha = (q * p).sum(0) / beta ** 2
        z0, z = z, p / beta - (alpha / beta) * z - (beta / beta0) * z0
        d = q / beta
        q = z / m
        beta0, beta, prev = beta, (q * z).sum(0).sqrt(), eps
        delta, ghat = c * dhat + s * alpha, -s * dhat + c * alpha
        eps, dhat = s * beta, c * beta
        gamma = (ghat * ghat + beta * beta).sqrt()
        c, s = ghat / gamma, beta / gamma
        d = (d - delta * d1 - prev * d2) / gamma
        x = x + (c * phi) * d
        phi = -s * phi
        d2, d1 = d1, d
    return x, phi.abs()


def _solve_refined(A, b):
    lu = torch.linalg.lu_factor(A)
    x = torch.linalg.lu_solve(*lu, b)
    return x + torch.linalg.lu_solve(*lu, b - A @ x)


def _pairs_plain(P, f, nev):
    w, V = torch.linalg.eigh(P.dense(f).cpu())
    sigma = 0.5 * (w[0] + w[-1])
    idx = _nearest(w, sigma, nev)
    U = _fix_sign(V[:, idx].cuda())
    return float(w[0]), float(w[-1]), float(sigma), w[idx].numpy(), U, P.twist(U).cpu().numpy()


def _entropy_plain(P, U):
    A = 1 << (P.L // 2)
    out = []
    for t in range(U.shape[1]):
        C = torch.zeros(A * A, dtype=torch.float64)
        C[P.states.cpu()] = U[:, t].cpu()
        p = torch.linalg.svdvals(C.view(A, A)) ** 2
        p = p[p > 0] / p.sum()
        out.append(float(-(p * p.log()).sum()))
    return np.array(out)


def exact(case, seed):
    kind = case["kind"]
    if kind == "problems":
        probs = _problem_list(case, seed)
        out = {}
        for L in sorted({p["L"] for p in probs}):
            of = [p for p in probs if p["L"] == L]
            if L > 12 or len(of) > 80:   # a dense solver's time
                out["L%d" % L] = dict(sigma=None, evals=None, z=None, evecs=None)
                continue
            P = _Plain(L)
            got = [_pairs_plain(P, p["h"], case["nev"]) for p in of]
            out["L%d" % L] = dict(sigma=np.array([g[2] for g in got]),
                                  evals=np.stack([g[3] for g in got]),
                                  z=np.stack([g[5] for g in got]),
                                  evecs=torch.cat([g[4] for g in got], 1))
        return out
    P = _Plain(case["L"])
    if kind == "pairs":
        f, _ = _fields(case, np.random.default_rng(seed), 1)
        lo, hi, sg, E, U, z = _pairs_plain(P, f[0], case["nev"])
        return dict(emin=lo, emax=hi, sigma=sg, evals=E, evecs=U, z=z, S=_entropy_plain(P, U))
    if kind == "grad":
        f, E, psi = _eigenpair(case, seed)
        z = P.twist(psi[:, None])[0]
        theta = sum(2 * math.pi / P.L * (j + 1) * P.spin(j) for j in range(P.L))
        g = 4 * psi * (z.real * torch.cos(theta) + z.imag * torch.sin(theta))
        g = g - psi * (psi @ g)
        A = P.dense(f) - E * torch.eye(P.n, dtype=torch.float64, device="cuda")
        lam = _solve_refined(A + torch.outer(psi, psi), g[:, None])[:, 0]
        lam = lam - psi * (psi @ lam)
        spins = torch.stack([P.spin(j) for j in range(P.L)], 1)
        return dict(dE=-(psi * psi) @ spins, dz2=(lam * psi) @ spins,
                    z=np.array([complex(z.cpu())]))
    R = case["R"]
    f, sg = _fields(case, np.random.default_rng(seed), max(R, 1))
    x = torch.randn((P.n, R) if R else (P.n,), dtype=torch.float64, device="cuda",
                    generator=_gen(seed))
    if kind == "apply":
        x = x.to(torch.float32).double() if case["dtype"] == FP32 else x
        if not R:
            return P.product(P.diagonal(f[0]) - float(sg[0]), x)
        return P.product(torch.stack([P.diagonal(fr) - float(s) for fr, s in zip(f, sg)], 1), x)
    b = x / x.norm(dim=0, keepdim=bool(R))
    if case["kmax"] == 0:
        if P.n > 13000 or P.n * max(R, 1) > 60000:
            return None   # a dense solver's time
        cols = b if R else b[:, None]
        eye = torch.eye(P.n, dtype=torch.float64, device="cuda")
        X = [_solve_refined(P.dense(fr) - float(s) * eye, cols[:, r:r + 1])
             for r, (fr, s) in enumerate(zip(f, sg))]
        X = torch.cat(X, 1)
        return dict(x=X if R else X[:, 0])
    X, phi = _minres_plain(P, case, f, sg, b if R else b[:, None])
    if R:
        return dict(x=X, iters=None, phi=phi)
    return dict(x=X[:, 0], iters=None, phi=float(phi[0]))
