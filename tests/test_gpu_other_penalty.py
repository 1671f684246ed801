"""Penalties other than k(k+1) through the public entry points: they take the
kernels that read coefficient tables (the default penalty has its own, with
compile-time coefficients).  Operator, additive and multiplicative steps with
separable and exact local solves, V-cycles with and without the one-launch
tail, single and batched solves, in both precisions, against the oracle
assembled with the same penalty.  Bars: those of gpu_util.py, with their
condition numbers and float32 floors taken for this penalty."""
import functools

import numpy as np
import pytest
import scipy.sparse as sp
import torch

import oracle as O
import paper_2412_05082_amd as P
from gpu_util import EPS64, _row_order_shuffled, check, dev, fp64_vcycle_tol, host, rel_l2, vectors

pytestmark = pytest.mark.gpu
FACTOR = 1.5
DTYPES = [torch.float64, torch.float32]


@functools.lru_cache(maxsize=None)
def _ops(dim, k, N, exact):
    gamma = FACTOR * k * (k + 1)
    A, idx = O.assemble(dim, k, N, gamma=gamma), O.patch_indices(dim, k, N)
    local = A if exact else O.assemble(dim, k, N, gamma=gamma, bulk="diag")
    return A, O.patch_blocks(local, idx), idx, O.mvs_colors(dim, N)


def _rounded_operator(dim, k, N, gamma):
    """The operator with the 1D factors rounded to float32, as the library holds them: a systematic change of A of a
    rounding's size, which the V-cycle amplifies on smooth modes."""
    M, L, B = (sp.csr_matrix(v.astype(np.float32).astype(np.float64)) for v in P.host_matrices_1d(k, N, gamma))
    if dim == 2:
        terms = [(1, B, M), (2, L, L), (1, M, B)]
    else:
        terms = [(1, B, M, M), (1, M, B, M), (1, M, M, B), (2, L, L, M), (2, L, M, L), (2, M, L, L)]
    return sum(c * functools.reduce(sp.kron, f) for c, *f in terms).tocsr()


def _inputs(dim, k, N, dtype):
    x, b = vectors(dim, k, N)
    if dtype == torch.float32:
        x, b = (v.astype(np.float32).astype(np.float64) for v in (x, b))
    return x, b


def _step(dim, k, N, exact, mvs, omega, x, b, low=False):
    """One step in float64; low: with the float32 floor's rounding (gpu_util.py: the residual rounded to float32 for
    the additive step, all of a multiplicative one in float32)."""
    A, blocks, idx, col = _ops(dim, k, N, exact)
    if mvs:
        if low:
            A, blocks = A.astype(np.float32), blocks.astype(np.float32)
        return O.mvs_apply(A, blocks, idx, col, x, b, omega, x_is_zero=x is None).astype(np.float64)
    if not low or x is None:
        return O.avs_apply(A, blocks, idx, x, b, omega, x_is_zero=x is None)
    r = (b.astype(np.float32) - A.astype(np.float32) @ x.astype(np.float32)).astype(np.float64)
    return x + O.avs_apply(A, blocks, idx, None, r, omega, x_is_zero=True)


def _bar(dim, k, N, exact, mvs, omega, x, b, dtype, ref):
    if dtype == torch.float64:
        _, blocks, _, _ = _ops(dim, k, min(N, 4), exact)
        kappa = max(np.linalg.cond(blocks[i]) for i in range(0, len(blocks), max(1, len(blocks) // 8)))
        return (2 ** (dim + 1) if mvs else 1) * max(1e-12, 2.0 * kappa * EPS64)
    if exact and mvs:  # one bar of the additive step with exact solves per colour
        add = [_step(dim, k, N, 1, 0, omega, x, b, low=low) for low in (True, False)]
        return 2 ** (dim + 1) * max(1e-5, 2.0 * rel_l2(*add))
    return max(1e-5, 2.0 * rel_l2(_step(dim, k, N, exact, mvs, omega, x, b, low=True), ref))


def _check_step(dim, k, N, dtype, omega, exact=0, mvs=0, variants=(0,), modes=(0,)):
    x, b = _inputs(dim, k, N, dtype)
    f64 = dtype == torch.float64
    y = torch.empty(x.size, dtype=dtype, device="cuda")
    for mode in modes:
        p = P.Problem(dim, N, k, gamma=FACTOR * k * (k + 1), omega=omega, smoother=mvs, local_solver=exact,
                      mvs_residual=mode)
        for name, xi in (("S(0,b)", None), ("S(x,b)", x)):
            ref = _step(dim, k, N, exact, mvs, omega, xi, b)
            bar = _bar(dim, k, N, exact, mvs, omega, xi, b, dtype, ref)
            for v in variants if xi is not None else (0,):
                if dim == 2:
                    p.set_variant(v, dtype=P.C0IP_F64 if f64 else P.C0IP_F32)
                y.fill_(7.0)
                p.smoother_step(dev(b, dtype), None if xi is None else dev(xi, dtype), y)
                check(f"{name} {dim}D Q{k} {N} {dtype} mvs {mvs} exact {exact} mode {mode} variant {v}",
                      rel_l2(host(y), ref), bar)
        p.close()


@pytest.mark.parametrize("dim,k,N", [(2, 2, 2), (2, 2, 32), (2, 3, 16), (2, 4, 16), (2, 5, 8), (2, 6, 8), (2, 7, 2),
                                     (2, 7, 8), (3, 2, 8), (3, 3, 4), (3, 4, 4), (3, 5, 4), (3, 6, 2), (3, 7, 2)])
@pytest.mark.parametrize("dtype", DTYPES)
def test_operator_and_additive_step(dim, k, N, dtype):
    x, _ = _inputs(dim, k, N, dtype)
    p = P.Problem(dim, N, k, gamma=FACTOR * k * (k + 1))
    y = torch.full((x.size,), 7.0, dtype=dtype, device="cuda")
    p.apply_A(dev(x, dtype), y)
    check(f"A x {dim}D Q{k} {N} {dtype}", rel_l2(host(y), _ops(dim, k, N, 0)[0] @ x),
          1e-12 if dtype == torch.float64 else 1e-5)
    p.close()
    _check_step(dim, k, N, dtype, 0.25 if dim == 2 else 0.1, variants=range(3 if k <= 3 else 2) if dim == 2 else (0,))


@pytest.mark.parametrize("exact", [0, 1])
@pytest.mark.parametrize("k,N", [(2, 2), (2, 16), (3, 16), (4, 8), (5, 8), (6, 4), (7, 4)])
@pytest.mark.parametrize("dtype", DTYPES)
def test_multiplicative_step_2d(k, N, exact, dtype):
    _check_step(2, k, N, dtype, 1.0, exact=exact, mvs=1, modes=(1, 2))


@pytest.mark.parametrize("k,N", [(2, 2), (2, 8), (3, 4), (4, 4), (5, 2)])
@pytest.mark.parametrize("dtype", DTYPES)
def test_multiplicative_step_3d(k, N, dtype):
    _check_step(3, k, N, dtype, 0.7, mvs=1)


@pytest.mark.parametrize("k,N", [(2, 8), (3, 8), (5, 4)])
@pytest.mark.parametrize("dtype", DTYPES)
def test_exact_additive_step(k, N, dtype):
    _check_step(2, k, N, dtype, 0.25, exact=1)


@pytest.mark.parametrize("dim,k,N,mvs", [(2, 2, 64, 0), (2, 3, 32, 0), (2, 4, 16, 0), (2, 5, 8, 0), (2, 3, 16, 1),
                                         (3, 2, 8, 0), (3, 2, 8, 1)])
@pytest.mark.parametrize("dtype", DTYPES)
def test_vcycle(dim, k, N, mvs, dtype):
    """With the tail (2D, k <= 4) and without it, one and two steps."""
    _, b = _inputs(dim, k, N, dtype)
    om = (1.0 if dim == 2 else 0.7) if mvs else (0.25 if dim == 2 else 0.1)
    for pre, post in ((1, 1), (2, 1)):
        kw = dict(gamma=FACTOR * k * (k + 1), omega=om, pre=pre, post=post, smoother="mvs" if mvs else "avs")
        H = O.Hierarchy(dim, k, N, **kw)
        if dtype == torch.float32:
            H.Alow = [_rounded_operator(dim, k, 2 << l, kw["gamma"]) for l in range(len(H.Alow))]
        ref = H.vcycle(b)
        if dtype == torch.float64:
            bar = (2 ** (dim + 1) if mvs else 1) * fp64_vcycle_tol(dim, k, N, pre, post)
        else:  # the oracle's own float32 V-cycle over four summation orders, as in gpu_util.py
            exact = O.Hierarchy(dim, k, N, **kw).vcycle(b)
            low = O.Hierarchy(dim, k, N, dtype=np.float32, **kw)
            errs, stored = [rel_l2(low.vcycle(b), exact)], list(low.Alow)
            for seed in range(3):
                rng = np.random.default_rng(seed)
                low.Alow = [_row_order_shuffled(a, rng) for a in stored]
                errs.append(rel_l2(low.vcycle(b), exact))
            bar = max(1e-5, 2.0 * max(errs))
        for tail in (-1, 0):
            p = P.Problem(dim, N, k, gamma=kw["gamma"], omega=om, pre_steps=pre, post_steps=post, smoother=mvs,
                          tail_levels=tail, vcycle_dtype=P.C0IP_F64 if dtype == torch.float64 else P.C0IP_F32)
            z = torch.full((b.size,), 7.0, dtype=dtype, device="cuda")
            p.vcycle(dev(b, dtype), z)
            check(f"V-cycle {dim}D Q{k} {N} {dtype} mvs {mvs} steps {pre}+{post} tail {tail}", rel_l2(host(z), ref), bar)
            p.close()


def test_batched_and_single_solves():
    """Uneven problems in one batch: the single solves' iteration counts, and true residuals of 1e-8."""
    problems, n_rhs, gamma = [(16, 2), (8, 3), (16, 3), (8, 2)], [2, 1, 1, 1], FACTOR * 12
    rng = np.random.default_rng(5)
    bs = []
    for (N, k), r in zip(problems, n_rhs):
        v = np.zeros((r, k * N + 1, k * N + 1))
        v[:, 1:-1, 1:-1] = rng.uniform(-1.0, 1.0, (r, k * N - 1, k * N - 1))
        bs.append(v.reshape(r, -1))
    batch = P.Batch(problems, n_rhs, gamma=gamma, vcycle_dtype=P.C0IP_F32)
    db = [dev(v) for v in bs]
    dx = [torch.zeros_like(v) for v in db]
    infos, i = batch.solve(db, dx, rtol=1e-8), 0
    for (N, k), v, xs in zip(problems, bs, dx):
        A = O.assemble(2, k, N, gamma=gamma)
        p = P.Problem(2, N, k, gamma=gamma, vcycle_dtype=P.C0IP_F32)
        for row, x in zip(v, host(xs)):
            xd = torch.zeros(row.size, dtype=torch.float64, device="cuda")
            one = p.solve(dev(row), xd, rtol=1e-8)
            assert infos[i]["converged"] == 1 and infos[i]["iterations"] == one["iterations"]
            for name, u in (("batched", x), ("single", host(xd))):
                check(f"residual Q{k} {N} {name}", np.linalg.norm(row - A @ u) / np.linalg.norm(row), 1.05e-8)
            i += 1
        p.close()
    batch.close()
