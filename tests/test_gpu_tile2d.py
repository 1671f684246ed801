"""The 2D operator and additive smoother on both sides of their switches
between small and large tiles, and on meshes that cut the tiles (one patch, a
mesh smaller than a tile, remainders), against the Kronecker form with dense
1D factors of the library (pinned to the exact ones in test_lib_host.py) and
SciPy's local eigenbases.  Boundary entries of the inputs hold large values:
they must not count."""
import functools

import numpy as np
import pytest
import scipy.linalg
import torch

import oracle as O
import paper_2412_05082_amd as P
from gpu_util import check, dev, fp32_mvs_tol, fp32_tol, fp64_mvs_tol, fp64_tol, fp64_vcycle_tol, host, rel_l2, vectors

pytestmark = pytest.mark.gpu
OMEGA = 0.25


@functools.lru_cache(maxsize=None)
def _factors(k, N):
    M, L, B = P.host_matrices_1d(k, N)
    n1, n = k * N + 1, 2 * k - 1
    E, lam = np.zeros(((N - 1) * n, n1)), np.zeros((N - 1) * n)
    for v in range(1, N):
        s, r = slice((v - 1) * k + 1, (v - 1) * k + 1 + n), slice((v - 1) * n, v * n)
        lam[r], Q = scipy.linalg.eigh(B[s, s], M[s, s])
        E[r, s] = Q.T
    return M, L, B, E, lam


def _apply(k, N, X):
    M, L, B, _, _ = _factors(k, N)
    return M @ X @ B + 2.0 * (L @ X @ L) + B @ X @ M


def _solves(k, N, R):
    _, _, _, E, lam = _factors(k, N)
    return E.T @ ((E @ R @ E.T) / (lam[:, None] + lam[None, :])) @ E


LARGE = {2: 256, 3: 256, 4: 256, 5: 128, 6: 128, 7: 128}


@pytest.mark.parametrize("k,N", [(k, N) for k in range(2, 8) for N in (2, 4, 16, LARGE[k])])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_operator_and_smoother_2d_tiles(k, N, dtype):
    n1 = k * N + 1
    rng = np.random.default_rng(10 * k + N)
    inner, full = [], []
    for _ in range(2):
        v = rng.uniform(-1.0, 1.0, (n1, n1))
        if dtype == torch.float32:
            v = v.astype(np.float32).astype(np.float64)
        z = np.zeros_like(v)
        z[1:-1, 1:-1] = v[1:-1, 1:-1]
        inner.append(z)
        full.append(np.where(z == 0.0, 1e6 * v, v))
    (x, b), (xf, bf) = inner, full
    f64 = dtype == torch.float64
    bar = fp64_tol(2, k, min(N, 8)) if f64 else fp32_tol(2, k, min(N, 8))
    p = P.Problem(2, N, k, omega=OMEGA)
    y = torch.full((n1 * n1,), 7.0, dtype=dtype, device="cuda")
    p.apply_A(dev(xf.ravel(), dtype), y)
    check(f"A x Q{k} {N}^2 {dtype}", rel_l2(host(y), _apply(k, N, x).ravel()), 1e-12 if f64 else 1e-5)
    y.fill_(7.0)
    p.smoother_step(dev(bf.ravel(), dtype), None, y)
    check(f"S(0,b) Q{k} {N}^2 {dtype}", rel_l2(host(y), OMEGA * _solves(k, N, b).ravel()), bar)
    ref = (x + OMEGA * _solves(k, N, b - _apply(k, N, x))).ravel()
    for variant in range(3 if k <= 3 else 2):
        p.set_variant(variant, dtype=P.C0IP_F64 if f64 else P.C0IP_F32)
        y.fill_(7.0)
        p.smoother_step(dev(bf.ravel(), dtype), dev(xf.ravel(), dtype), y)
        check(f"S(x,b) Q{k} {N}^2 {dtype} variant {variant}", rel_l2(host(y), ref), bar)
        edge = host(y).reshape(n1, n1)
        assert np.all(edge[[0, -1], :] == 0.0) and np.all(edge[:, [0, -1]] == 0.0)


@pytest.mark.parametrize("k,N", [(2, 16), (3, 32), (5, 8)])
def test_other_penalty_2d(k, N):
    """Another penalty constant takes the kernels with coefficient tables:
    operator, smoother step and V-cycle against the oracle."""
    gamma = 1.5 * k * (k + 1)
    x, b = vectors(2, k, N)
    A = O.assemble(2, k, N, gamma=gamma)
    idx = O.patch_indices(2, k, N)
    blocks = O.patch_blocks(O.assemble(2, k, N, gamma=gamma, bulk="diag"), idx)
    p = P.Problem(2, N, k, gamma=gamma, omega=OMEGA, vcycle_dtype=P.C0IP_F64)
    y = torch.empty(x.size, dtype=torch.float64, device="cuda")
    p.apply_A(dev(x), y)
    check("A x", rel_l2(host(y), A @ x), 1e-12)
    p.smoother_step(dev(b), dev(x), y)
    check("S(x,b)", rel_l2(host(y), O.avs_apply(A, blocks, idx, x, b, OMEGA)), fp64_tol(2, k, N))
    p.vcycle(dev(b), y)
    ref = O.Hierarchy(2, k, N, gamma=gamma, omega=OMEGA).vcycle(b)
    check("V-cycle", rel_l2(host(y), ref), fp64_vcycle_tol(2, k, N))


@pytest.mark.parametrize("k,N", [(2, 2), (2, 64), (3, 8), (3, 64), (4, 4), (4, 32), (5, 16), (6, 16), (7, 2), (7, 16)])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_multiplicative_step_2d(k, N, dtype):
    """The coloured step with the residual in the colour's launch: one patch
    (seven empty colours), patches that fill part of a workgroup, and several
    workgroups per colour."""
    n1, n = k * N + 1, 2 * k - 1
    rng = np.random.default_rng(100 * k + N)
    x, b = (np.pad(rng.uniform(-1.0, 1.0, (n1 - 2, n1 - 2)).astype(np.float32).astype(np.float64), 1)
            for _ in range(2))
    _, _, _, E, lam = _factors(k, N)
    v = np.repeat(np.arange(1, N), n)
    ref = x.copy()
    for c in range(8):
        on = (((v[:, None] // 2 + v[None, :] // 2) % 2 == c // 4) & (v[:, None] % 2 == c // 2 % 2)
              & (v[None, :] % 2 == c % 2))
        ref = ref + E.T @ (on * (E @ (b - _apply(k, N, ref)) @ E.T) / (lam[:, None] + lam[None, :])) @ E
    p = P.Problem(2, N, k, omega=1.0, smoother=1, mvs_residual=1)
    y = torch.full((n1 * n1,), 7.0, dtype=dtype, device="cuda")
    p.smoother_step(dev(b.ravel(), dtype), dev(x.ravel(), dtype), y)
    small = min(N, 8)
    bar = fp64_mvs_tol(2, k, small) if dtype == torch.float64 else fp32_mvs_tol(2, k, small, 1.0)
    check(f"MVS Q{k} {N}^2 {dtype}", rel_l2(host(y), ref.ravel()), bar)
