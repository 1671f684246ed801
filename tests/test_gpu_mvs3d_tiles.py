"""The 3D coloured multiplicative step with the residual formed in each
colour's launch, on meshes that fill its workgroups in every way (one patch
and 15 empty colours, one partial row, full and remainder chunks of a row),
from x and from 0, against the coloured sweep in Kronecker form: dense 1D
factors of the library (pinned to the exact ones in test_lib_host.py), local
eigenbases from SciPy.  Boundary entries of the inputs hold large values: they
must not count, and the ones of x stay."""
import numpy as np
import pytest
import scipy.linalg
import torch

import paper_2412_05082_amd as P
from gpu_util import check, dev, fp32_mvs_tol, fp64_mvs_tol, host, rel_l2

pytestmark = pytest.mark.gpu
OMEGA = 0.7


def _kron3(F, X):
    for d, A in enumerate(F):
        X = np.moveaxis(np.tensordot(A, X, axes=(1, d)), 0, d)
    return X


def _step(k, N, x, b):
    M, L, B = P.host_matrices_1d(k, N)
    n1, n = k * N + 1, 2 * k - 1
    E, lam = np.zeros(((N - 1) * n, n1)), np.zeros((N - 1) * n)
    for v in range(1, N):
        s, r = slice((v - 1) * k + 1, (v - 1) * k + 1 + n), slice((v - 1) * n, v * n)
        lam[r], Q = scipy.linalg.eigh(B[s, s], M[s, s])
        E[r, s] = Q.T
    v = np.repeat(np.arange(1, N), n)
    z, y, xx = v[:, None, None], v[None, :, None], v[None, None, :]
    for c in range(16):
        on = (z // 2 + y // 2 + xx // 2) % 2 == c // 8
        on = on & (z % 2 == c // 4 % 2) & (y % 2 == c // 2 % 2) & (xx % 2 == c % 2)
        if not on.any():
            continue
        r = b - sum(_kron3(f, x) for f in ((B, M, M), (M, B, M), (M, M, B)))
        r -= 2.0 * sum(_kron3(f, x) for f in ((L, L, M), (L, M, L), (M, L, L)))
        T = on * _kron3((E, E, E), r) / (lam[:, None, None] + lam[None, :, None] + lam[None, None, :])
        x = x + OMEGA * _kron3((E.T, E.T, E.T), T)
    return x


@pytest.mark.parametrize("k,N", [(2, 2), (2, 4), (2, 8), (2, 32), (3, 2), (3, 4), (3, 16), (4, 2), (4, 8)])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_multiplicative_step_3d_tiles(k, N, dtype):
    n1 = k * N + 1
    rng = np.random.default_rng(1000 * k + N)
    inner, full = [], []
    for _ in range(2):
        v = rng.uniform(-1.0, 1.0, (n1, n1, n1)).astype(np.float32).astype(np.float64)
        z = np.zeros_like(v)
        z[1:-1, 1:-1, 1:-1] = v[1:-1, 1:-1, 1:-1]
        inner.append(z)
        full.append(np.where(z == 0.0, 1e6 * v, v))
    (x, b), (xf, bf) = inner, full
    small = min(N, 4)
    bar = fp64_mvs_tol(3, k, small) if dtype == torch.float64 else fp32_mvs_tol(3, k, small, OMEGA)
    p = P.Problem(3, N, k, omega=OMEGA, smoother=1)
    out = torch.full((n1 ** 3,), 7.0, dtype=dtype, device="cuda")
    p.smoother_step(dev(b.ravel(), dtype), None, out)
    check(f"MVS S(0,b) 3D Q{k} {N}^3 {dtype}", rel_l2(host(out), _step(k, N, np.zeros_like(b), b).ravel()), bar)
    xs = dev(xf.ravel(), dtype)
    p.apply_smoother(dev(bf.ravel(), dtype), xs)
    got, edge = host(xs).reshape(n1, n1, n1), np.ones((n1, n1, n1), bool)
    edge[1:-1, 1:-1, 1:-1] = False
    assert np.array_equal(got[edge], dev(xf.ravel(), dtype).cpu().double().numpy().reshape(n1, n1, n1)[edge])
    check(f"MVS S(x,b) 3D Q{k} {N}^3 {dtype}", rel_l2(np.where(edge, 0.0, got).ravel(), _step(k, N, x, b).ravel()), bar)
