"""The 3D additive smoother on meshes that meet its tiles and z chunks in every
way (one patch, a tile cut by the mesh, several chunks, one cell per chunk),
against the Kronecker form of the step: dense 1D factors of the library (pinned
to the exact ones in test_lib_host.py), local eigenbases from SciPy."""
import numpy as np
import pytest
import scipy.linalg
import torch

import paper_2412_05082_amd as P
from gpu_util import check, dev, fp32_tol, fp64_tol, host, rel_l2

pytestmark = pytest.mark.gpu
OMEGA = 0.1


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
    res = b.copy()
    if x is not None:
        res -= sum(_kron3(f, x) for f in ((B, M, M), (M, B, M), (M, M, B)))
        res -= 2.0 * sum(_kron3(f, x) for f in ((L, L, M), (L, M, L), (M, L, L)))
    T = _kron3((E, E, E), res)
    T /= lam[:, None, None] + lam[None, :, None] + lam[None, None, :]
    # E^T per axis; the modes of every patch scatter back to its nodes
    return (0 if x is None else x) + OMEGA * _kron3((E.T, E.T, E.T), T)


@pytest.mark.parametrize("k,N", [(2, 2), (2, 8), (2, 16), (2, 32), (3, 2), (3, 4), (3, 8), (3, 16), (3, 32), (4, 2),
                                 (4, 4), (4, 8), (4, 16)])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_smoother_3d_tiles(k, N, dtype):
    n1 = k * N + 1
    rng = np.random.default_rng(10 * k + N)
    x, b = np.zeros((n1, n1, n1)), np.zeros((n1, n1, n1))
    for v in (x, b):
        v[1:-1, 1:-1, 1:-1] = rng.uniform(-1.0, 1.0, (n1 - 2, n1 - 2, n1 - 2))
        if dtype == torch.float32:
            v[...] = v.astype(np.float32)
    bar = fp64_tol(3, k, min(N, 4)) if dtype == torch.float64 else fp32_tol(3, k, min(N, 4))
    p = P.Problem(3, N, k, omega=OMEGA)
    out = torch.full((n1 ** 3,), 7.0, dtype=dtype, device="cuda")
    for name, xi in (("S(0,b)", None), ("S(x,b)", x)):
        p.smoother_step(dev(b.ravel(), dtype), None if xi is None else dev(xi.ravel(), dtype), out)
        check(f"{name} 3D Q{k} {N}^3 {dtype}", rel_l2(host(out), _step(k, N, xi, b).ravel()), bar)
    xs = dev(x.ravel(), dtype)  # in place
    p.apply_smoother(dev(b.ravel(), dtype), xs)
    assert torch.equal(xs, out)
