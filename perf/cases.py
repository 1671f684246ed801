"""Timing cases of the C0IP hot path, called through the package's public
entry points: operator, additive and multiplicative smoother steps, V-cycles,
FGMRES and flexible-CG solves and batched solves, in 2D and 3D.

listed() are the fixed cases, draw(rng) gives further ones of the same ranges.
prepare(case, seed) makes a handle and seeded device vectors, run(state) is one
pass, work(case) what a pass cannot do without, exact(case, seed) the same
outputs in plain float64 PyTorch: every operator is a Kronecker product of
dense 1D matrices built here from quadrature.
"""
import math

import numpy as np
import torch

import paper_2412_05082_amd as P

F64, F32 = "float64", "float32"


def _case(kind, dim, k, N, dtype, **more):
    c = {"kind": kind, "dim": dim, "degree": k, "cells": N, "dtype": dtype, "smoother": "avs",
         "local": "separable", "steps": 1, "x_zero": False}
    c.update(more)
    return c


def listed():
    named = {
        # one operator call on the smallest workload of the benchmark: launch latency
        "apply_2d_q2_16_f64": _case("apply", 2, 2, 16, F64),
        # the operator of the outer Krylov method on the headline mesh
        "apply_2d_q3_512_f64": _case("apply", 2, 3, 512, F64),
        # the dominant kernel of the mixed-precision V-cycle on the headline mesh
        "smooth_2d_q3_512_f32": _case("smooth", 2, 3, 512, F32),
        # a smoother step at high degree (degree sweep), ordinary mesh, double precision
        "smooth_2d_q6_128_f64": _case("smooth", 2, 6, 128, F64),
        # one multiplicative step (8 colours), ordinary mesh
        "mvs_2d_q3_256_f64": _case("smooth", 2, 3, 256, F64, smoother="mvs"),
        # the preconditioner of the headline solve
        "vcycle_2d_q3_512_f32": _case("vcycle", 2, 3, 512, F32),
        # a double-precision V-cycle on an ordinary mesh: mostly launches
        "vcycle_2d_q4_64_f64": _case("vcycle", 2, 4, 64, F64),
        # 3D operator and additive smoother step at the benchmark's 3D size
        "apply_3d_q3_128_f64": _case("apply", 3, 3, 128, F64),
        "smooth_3d_q3_128_f32": _case("smooth", 3, 3, 128, F32),
        # the preconditioner of the 3D mixed-precision workload (multiplicative, 16 colours)
        "vcycle_3d_q2_128_mvs_f32": _case("vcycle", 3, 2, 128, F32, smoother="mvs"),
        # a whole mixed-precision FGMRES solve of an ordinary problem
        "solve_2d_q3_64": _case("solve", 2, 3, 64, F32),
        # many uneven small systems in one batch
        "batch_2d_24": _case("batch", 2, 3, 32, F32, problems=24),
    }
    return [dict(c, name=n) for n, c in named.items()]


def draw(rng):
    kind = rng.choice(["apply", "apply", "smooth", "smooth", "smooth", "vcycle", "vcycle", "solve", "fcg", "batch"])
    dim = rng.choice([2, 2, 3])
    dtype = rng.choice([F64, F32])
    more = {}
    if kind in ("solve", "fcg", "batch"):
        # sizes at which float64 determines the solution to well under 1e-9 (the operator's condition grows as N^4)
        dim, k = 2, rng.choice([2, 3, 4])
        N = 2 ** rng.randint(4, 6 if k <= 3 and kind != "batch" else 5)
        if kind == "batch":
            more["problems"] = rng.randint(5, 40)
        elif kind == "fcg":
            more["steps"] = rng.choice([1, 2])
        elif rng.random() < 0.3:
            more["smoother"] = "mvs"
        return _case(kind, dim, k, N, dtype, **more)
    # float32 residuals are rounded at the local solvers' condition number: steps below degree 5, V-cycles below 4
    top = 7 if dtype == F64 or kind == "apply" else 4 if kind == "smooth" else 3
    k = rng.randint(2, top)
    if dim == 2:
        N = 2 ** rng.randint(3, 9 if k <= 4 else 8)
    else:
        N = 2 ** rng.randint(2, 7 if k <= 3 and kind != "vcycle" else 6 if k <= 4 else 5)
    if kind != "apply" and rng.random() < 0.35:
        more["smoother"] = "mvs"
        if dim == 3:
            N = min(N, 64 if k <= 3 else 32 if k == 4 else 16)
            if kind == "vcycle" and dtype == F32:
                k = 2
    if kind != "apply" and dim == 2 and k <= 3 and rng.random() < 0.2:
        more["local"] = "exact"
    if kind == "smooth" and rng.random() < 0.3:
        more["x_zero"] = True
    if kind == "vcycle":
        more["steps"] = rng.choice([1, 1, 2])
    return _case(kind, dim, k, N, dtype, **more)


def _omega(c):
    if c["smoother"] == "mvs":
        return 1.0 if c["dim"] == 2 else 0.7
    return 0.25 if c["dim"] == 2 else 0.1


def _problems(c):
    """A batch's (cells, degree) list: sizes up to the case's mesh, degrees 2 to 4."""
    top = int(math.log2(c["cells"]))
    return [(2 ** (top - i % 4 if top - i % 4 >= 2 else 2), 2 + (c["degree"] + i // 4) % 3)
            for i in range(c["problems"])]


def _rhs(i):
    return 4 if i == 0 else 1


_RTOL = 1e-10


def _vector(gen, dim, k, N, dtype, device):
    """Uniform [-1, 1] on the interior nodes, 0 on the boundary."""
    n1 = k * N + 1
    v = torch.rand([n1] * dim, generator=gen, dtype=torch.float64, device=device) * 2 - 1
    for d in range(dim):
        v.select(d, 0).zero_()
        v.select(d, n1 - 1).zero_()
    return v.to(dtype).reshape(-1)


def _inputs(c, seed):
    """The case's vectors: b (and x), or a batch's right-hand sides."""
    device = torch.device("cuda" if torch.cuda.is_available() else "cpu")
    gen = torch.Generator(device=device).manual_seed(1000003 * int(seed) + 17)
    if c["kind"] == "batch":
        return [torch.stack([_vector(gen, 2, k, N, torch.float64, device) for _ in range(_rhs(i))])
                for i, (N, k) in enumerate(_problems(c))]
    dtype = torch.float64 if c["dtype"] == F64 or c["kind"] in ("solve", "fcg") else torch.float32
    return [_vector(gen, c["dim"], c["degree"], c["cells"], dtype, device) for _ in range(2)]


def prepare(case, seed):
    v = _inputs(case, seed)
    vdt = P.C0IP_F64 if case["dtype"] == F64 else P.C0IP_F32
    if case["kind"] == "batch":
        handle = P.Batch(_problems(case), [_rhs(i) for i in range(case["problems"])], omega=0.25, vcycle_dtype=vdt)
        return {"case": case, "handle": handle, "b": v, "y": [torch.zeros_like(b) for b in v]}
    handle = P.Problem(case["dim"], case["cells"], case["degree"], omega=_omega(case), pre_steps=case["steps"],
                       post_steps=case["steps"], vcycle_dtype=vdt, smoother=int(case["smoother"] == "mvs"),
                       local_solver=int(case["local"] == "exact"))
    return {"case": case, "handle": handle, "b": v[0], "x": v[1], "y": torch.zeros_like(v[0])}


def run(state):
    c, h, b, y = state["case"], state["handle"], state["b"], state["y"]
    kind = c["kind"]
    if kind == "apply":
        h.apply_A(state["x"], y)
    elif kind == "smooth":
        h.smoother_step(b, None if c["x_zero"] else state["x"], y)
    elif kind == "vcycle":
        h.vcycle(b, y)
    elif kind == "solve":
        h.solve(b, y, rtol=_RTOL)
    elif kind == "fcg":
        h.solve_fcg(b, y, rtol=_RTOL)
    else:
        h.solve(b, y, rtol=_RTOL)
    return y


# ---------------------------------------------------------------- work

def _fma_apply(dim, k):
    m, b = k + 2, 3 * k + 2  # mean row lengths of the 1D mass/Laplace and bi-Laplace factors
    return 4 * m + 2 * b if dim == 2 else 9 * m + 3 * b


def _fma_patches(dim, k, exact):
    """Local solves per DoF: about one patch per cell of k^dim nodes."""
    n = 2 * k - 1
    return (n ** (2 * dim) if exact else 2 * dim * n ** (dim + 1) + n ** dim) / k ** dim


def _work_step(c, dim, k, n, size, x_zero):
    """Bytes and FMAs of one smoother step."""
    solve = _fma_patches(dim, k, c["local"] == "exact")
    apply = _fma_apply(dim, k)
    if c["smoother"] == "mvs":  # each colour's residual on its own patch nodes
        share = ((2 * k - 1) / k) ** dim
        return 3 * n * size, n * (solve + apply * share)
    return (2 if x_zero else 3) * n * size, n * (solve + (0 if x_zero else apply))


def _work_vcycle(c, dim, k, N):
    """Per level: the smoothing steps, the residual with its restriction, the correction."""
    size = 8 if c["dtype"] == F64 else 4
    byt = fma = 0.0
    while N >= 4:
        n = (k * N + 1) ** dim
        for s in range(2 * c["steps"]):
            b1, f1 = _work_step(c, dim, k, n, size, s == 0)
            byt, fma = byt + b1, fma + f1
        byt, fma = byt + 2 * n * size, fma + n * (_fma_apply(dim, k) + 4 * (k + 1))
        N //= 2
    return byt, fma


def _work_solve(c, dim, k, N):
    its = 50  # about what the additive smoother takes to this tolerance
    if c["smoother"] == "mvs" or c["steps"] == 2:
        its = 20
    n = (k * N + 1) ** dim
    byt, fma = _work_vcycle(c, dim, k, N)
    basis = its / 2 if c["kind"] != "fcg" else 5
    return its * (byt + 16 * n + 16 * n * basis), its * (fma + n * _fma_apply(dim, k) + 4 * n * basis)


def work(case):
    dim, k, N = case["dim"], case["degree"], case["cells"]
    n = (k * N + 1) ** dim
    size = 8 if case["dtype"] == F64 else 4
    if case["kind"] == "apply":
        byt, fma = 2 * n * size, n * _fma_apply(dim, k)
    elif case["kind"] == "smooth":
        byt, fma = _work_step(case, dim, k, n, size, case["x_zero"])
    elif case["kind"] == "vcycle":
        byt, fma = _work_vcycle(case, dim, k, N)
    elif case["kind"] == "batch":
        byt = fma = 0.0
        for i, (Ni, ki) in enumerate(_problems(case)):
            b1, f1 = _work_solve(case, 2, ki, Ni)
            byt, fma = byt + _rhs(i) * b1, fma + _rhs(i) * f1
    else:
        byt, fma = _work_solve(case, dim, k, N)
    return {"bytes": float(byt), "flops": 2.0 * fma}


# ---------------------------------------------------------------- float64 reference

def _nodes(k):
    """Gauss-Lobatto nodes on [0, 1]."""
    inner = np.polynomial.legendre.Legendre.basis(k).deriv().roots()
    z = np.concatenate([[-1.0], np.sort(inner.real), [1.0]])
    return (z + 1) / 2


def _basis(k):
    z = _nodes(k)
    out = []
    for j in range(k + 1):
        r = np.delete(z, j)
        out.append(np.polynomial.Polynomial.fromroots(r) / np.prod(z[j] - r))
    return z, out


class _Level:
    """Dense 1D matrices of one mesh level: mass M, Laplace L, interior-penalty
    bi-Laplace B, the patch eigentransform E (all patches' eigenmodes as rows),
    and the embedding from the next coarser level."""

    def __init__(self, dim, k, N, device):
        self.dim, self.k, self.N, self.n1 = dim, k, N, k * N + 1
        h, n1 = 1.0 / N, self.n1
        z, phi = _basis(k)
        t, w = np.polynomial.legendre.leggauss(k + 2)
        t, w = (t + 1) / 2, w / 2
        val = [np.array([f.deriv(m)(t) if m else f(t) for f in phi]) for m in range(3)]
        el = [(val[m] * w) @ val[m].T * h ** (1 - 2 * m) for m in range(3)]
        d1 = np.array([[f.deriv(1)(e) for f in phi] for e in (0.0, 1.0)]) / h
        d2 = np.array([[f.deriv(2)(e) for f in phi] for e in (0.0, 1.0)]) / h ** 2
        M, L, B = (np.zeros((n1, n1)) for _ in range(3))
        for c in range(N):
            s = slice(c * k, c * k + k + 1)
            for G, e in zip((M, L, B), el):
                G[s, s] += e
        for f in range(N + 1):
            lo, hi = max(0, (f - 1) * k), min(n1, (f + 1) * k + 1)
            jump, mean = np.zeros(hi - lo), np.zeros(hi - lo)
            both = 0.5 if 0 < f < N else 1.0
            if f > 0:
                jump[:k + 1] += d1[1]
                mean[:k + 1] += both * d2[1]
            if f < N:
                jump[-(k + 1):] -= d1[0]
                mean[-(k + 1):] += both * d2[0]
            B[lo:hi, lo:hi] += (k * (k + 1) / h * np.outer(jump, jump) - np.outer(jump, mean) - np.outer(mean, jump))
        for G in (M, L, B):
            G[[0, -1], :] = 0
            G[:, [0, -1]] = 0
        n = 2 * k - 1
        E, lam = np.zeros(((N - 1) * n, n1)), np.zeros((N - 1) * n)
        for v in range(1, N):
            s = slice((v - 1) * k + 1, (v - 1) * k + 1 + n)
            C = np.linalg.inv(np.linalg.cholesky(M[s, s]))
            lv, U = np.linalg.eigh(C @ B[s, s] @ C.T)
            r = slice((v - 1) * n, v * n)
            E[r, s], lam[r] = U.T @ C, lv
        dev = lambda a: torch.from_numpy(a).to(device)  # noqa: E731
        self.M, self.L, self.B, self.E, self.lam = dev(M), dev(L), dev(B), dev(E), dev(lam)
        self.embed = None
        if N > 2:
            Pr = np.zeros((n1, k * (N // 2) + 1))
            for c in range(N):
                for p in range(k + 1):
                    Pr[c * k + p, (c // 2) * k:(c // 2) * k + k + 1] = [f((c % 2 + z[p]) / 2) for f in phi]
            self.embed = dev(Pr)
        self.blocks = {}

    def along(self, G, X, d):
        """G applied along axis d of X."""
        Y = torch.tensordot(G, X, dims=([1], [d]))
        return Y.movedim(0, d).contiguous()

    def each(self, G, X):
        for d in range(self.dim):
            X = self.along(G, X, d)
        return X

    def apply(self, X):
        M, L, B = self.M, self.L, self.B
        if self.dim == 2:
            XL, XB, XM = (self.along(G, X, 1) for G in (L, B, M))
            return self.along(M, XB, 0) + 2 * self.along(L, XL, 0) + self.along(B, XM, 0)
        XM, XL, XB = (self.along(G, X, 2) for G in (M, L, B))
        S1 = self.along(M, XB, 1) + self.along(B, XM, 1) + 2 * self.along(L, XL, 1)
        S2 = self.along(M, XM, 1)
        S3 = 2 * (self.along(L, XM, 1) + self.along(M, XL, 1))
        return self.along(M, S1, 0) + self.along(B, S2, 0) + self.along(L, S3, 0)

    def colours(self):
        """Per patch: its colour, from its vertex's parities and their red-black split."""
        v = torch.arange(1, self.N, device=self.M.device)
        col = half = 0
        for d in range(self.dim):
            shape = [1] * self.dim
            shape[self.dim - 1 - d] = self.N - 1
            col = col + ((v % 2) << d).reshape(shape)
            half = half + (v // 2).reshape(shape)
        return col + (half % 2) * 2 ** self.dim

    def solves(self, R, exact, mask=None):
        """Sum over the patches (of the mask) of the local solves of R."""
        n = 2 * self.k - 1
        if exact:
            return self._solves_exact(R, mask)
        T = self.each(self.E, R)
        s = 0
        for d in range(self.dim):
            shape = [1] * self.dim
            shape[d] = -1
            s = s + self.lam.reshape(shape)
        T = T / s
        if mask is not None:
            for d in range(self.dim):
                mask = mask.repeat_interleave(n, dim=d)
            T = T * mask
        return self.each(self.E.T, T)

    def _solves_exact(self, R, mask):
        """2D: dense solves with the restriction of the operator to each patch."""
        k, N, n = self.k, self.N, 2 * self.k - 1
        out = torch.zeros_like(R)
        variant = lambda v: (v == 1) + 2 * (v == N - 1)  # noqa: E731
        vs = {}
        for v in range(1, N):
            vs.setdefault(variant(v), []).append(v)
        for ty, ys in vs.items():
            for tx, xs in vs.items():
                if (ty, tx) not in self.blocks:
                    a, b = ((w[0] - 1) * k + 1 for w in (ys, xs))
                    G = [[m[o:o + n, o:o + n].contiguous() for m in (self.M, self.L, self.B)] for o in (a, b)]
                    A = torch.kron(G[0][0], G[1][2]) + 2 * torch.kron(G[0][1], G[1][1]) + torch.kron(G[0][2], G[1][0])
                    self.blocks[ty, tx] = torch.linalg.inv(A)
                y, x = (torch.tensor(w, device=R.device) for w in (ys, xs))
                o = torch.arange(n, device=R.device)
                iy = ((y - 1) * k + 1)[:, None, None, None] + o[None, None, :, None]
                ix = ((x - 1) * k + 1)[None, :, None, None] + o[None, None, None, :]
                U = R[iy, ix].reshape(-1, n * n) @ self.blocks[ty, tx].T
                if mask is not None:
                    U = U * mask[y - 1][:, x - 1].reshape(-1, 1)
                flat = (iy * self.n1 + ix).reshape(-1)
                out.view(-1).index_add_(0, flat, U.reshape(-1))
        return out

    def step(self, c, omega, X, b):
        ex = c["local"] == "exact"
        if c["smoother"] != "mvs":
            R = b if X is None else b - self.apply(X)
            return omega * self.solves(R, ex) + (0 if X is None else X)
        X = torch.zeros_like(b) if X is None else X
        col = self.colours()
        for q in range(2 ** (self.dim + 1)):
            X = X + omega * self.solves(b - self.apply(X), ex, col == q)
        return X


def _levels(dim, k, N, device):
    lv = []
    while N >= 2:
        lv.insert(0, _Level(dim, k, N, device))
        N //= 2
    return lv


def _vcycle(c, omega, lv, b):
    top = lv[-1]
    if top.N == 2:  # one patch: solve with the operator itself
        k, n = top.k, 2 * top.k - 1
        s = slice(1, 1 + n)
        M, L, B = (m[s, s].contiguous() for m in (top.M, top.L, top.B))
        kr = lambda *m: m[0] if len(m) == 1 else torch.kron(m[0], kr(*m[1:]))  # noqa: E731
        if top.dim == 2:
            A = kr(B, M) + 2 * kr(L, L) + kr(M, B)
        else:
            A = kr(B, M, M) + kr(M, B, M) + kr(M, M, B) + 2 * (kr(L, L, M) + kr(L, M, L) + kr(M, L, L))
        X = torch.zeros_like(b)
        at = (s,) * top.dim
        X[at] = torch.linalg.solve(A, b[at].reshape(-1, 1)).reshape(b[at].shape)
        return X
    X = None
    for _ in range(c["steps"]):
        X = top.step(c, omega, X, b)
    X = X + top.each(top.embed, _vcycle(c, omega, lv[:-1], top.each(top.embed.T.contiguous(), b - top.apply(X))))
    for _ in range(c["steps"]):
        X = top.step(c, omega, X, b)
    return X


def _solve(dim, k, N, b):
    """A x = b by conjugate gradients with the additive V-cycle, to stagnation, then one more correction."""
    lv = _levels(dim, k, N, b.device)
    plain = {"smoother": "avs", "local": "separable", "steps": 2}
    omega = 0.25 if dim == 2 else 0.1
    x = torch.zeros_like(b)
    for _ in range(2):
        r = b - lv[-1].apply(x)
        stop, p, rz = float(r.norm()) * 1e-13, None, None
        for _ in range(80):
            z = _vcycle(plain, omega, lv, r)
            new = (r * z).sum()
            p = z if p is None else z + (new / rz) * p
            rz = new
            q = lv[-1].apply(p)
            alpha = rz / (p * q).sum()
            x, r = x + alpha * p, r - alpha * q
            if not float(r.norm()) > stop:
                break
    return x


def exact(case, seed):
    if not torch.cuda.is_available() and case["dim"] == 3 and case["cells"] > 16:
        return None
    dim, k, N = case["dim"], case["degree"], case["cells"]
    v = _inputs(case, seed)
    if case["kind"] == "batch":
        out = []
        for (Ni, ki), b in zip(_problems(case), v):
            n1 = ki * Ni + 1
            out.append(torch.stack([_solve(2, ki, Ni, q.reshape(n1, n1)).reshape(-1) for q in b]))
        return out
    shape = [k * N + 1] * dim
    b, x = (t.double().reshape(shape) for t in v)
    if case["kind"] == "apply":
        y = _Level(dim, k, N, b.device).apply(x)
    elif case["kind"] == "smooth":
        y = _Level(dim, k, N, b.device).step(case, _omega(case), None if case["x_zero"] else x, b)
    elif case["kind"] == "vcycle":
        y = _vcycle(case, _omega(case), _levels(dim, k, N, b.device), b)
    else:
        y = _solve(dim, k, N, b)
    return y.reshape(-1)
