"""Rounding of the float32 local solves S(0, b).  The kernels share transforms
between overlapping patches and multiply by reciprocal eigenvalue sums; they
may round no worse for it than the plain form, every patch for itself with one
division per mode (in float32 on the CPU, one rounding per multiply-add, as on
the device).  Errors are rms over the mesh and over the nodes of the x axis's
first cell, where the boundary patches' share shows.  Smooth right-hand sides:
a few low modes carry the result, so the rounding of a constant that all
patches share does not average out.  Each form has one such rounding per mode
(of the eigenvalue sum, or of its reciprocal), uniform within a unit roundoff
u: u / sqrt(3) of slack."""
import numpy as np
import pytest
import scipy.linalg
import torch

import paper_2412_05082_amd as P
from gpu_util import check, dev, host

pytestmark = pytest.mark.gpu


def _eigen(k, N):
    """Eigenbases and eigenvalues of every vertex's 1D patch."""
    M, _, B = P.host_matrices_1d(k, N)
    n, kinds, Q, lam = 2 * k - 1, {}, [], []
    for v in range(1, N):
        s, t = slice((v - 1) * k + 1, (v - 1) * k + 1 + n), (v == 1, v == N - 1)
        if t not in kinds:
            kinds[t] = scipy.linalg.eigh(B[s, s], M[s, s])
        lam.append(kinds[t][0])
        Q.append(kinds[t][1])
    return np.array(Q), np.array(lam)


def _plain(dim, k, N, b, omega, dtype):
    """omega sum_v R_v^T A~_v^{-1} R_v b, patch by patch, in `dtype`."""
    n, V = 2 * k - 1, N - 1
    Q, lam = (a.astype(dtype) for a in _eigen(k, N))
    win = np.lib.stride_tricks.sliding_window_view(b.astype(dtype)[(slice(1, -1),) * dim], (n,) * dim)
    t = np.ascontiguousarray(win[(slice(None, None, k),) * dim])  # vertices, then nodes

    def along(t, axis, forward):
        t = np.moveaxis(t, dim + axis, -1)
        out = np.zeros_like(t)
        shape = [1] * t.ndim
        shape[axis], shape[-1] = V, n
        for j in range(n):
            q = (Q[:, j, :] if forward else Q[:, :, j]).reshape(shape)
            out = (q.astype(np.float64) * t[..., j:j + 1] + out).astype(dtype)
        return np.moveaxis(out, -1, dim + axis)

    axes = range(dim - 1, -1, -1)  # x first
    for a in axes:
        t = along(t, a, True)
    d = np.zeros((1,) * (2 * dim), dtype)
    for a in axes:
        shape = [1] * (2 * dim)
        shape[a], shape[dim + a] = V, n
        d = (d + lam.reshape(shape)).astype(dtype)
    t = t / d
    for a in axes:
        t = along(t, a, False)
    out = np.zeros(b.shape, dtype)
    for v in np.ndindex((V,) * dim):
        out[tuple(slice(i * k + 1, i * k + 1 + n) for i in v)] += t[v]
    return (omega * out).astype(dtype)


@pytest.mark.parametrize("dim,k,N", [(2, 4, 128), (2, 5, 128), (2, 6, 128), (2, 7, 128), (3, 3, 16), (3, 5, 16),
                                     (3, 7, 8)])
def test_float32_solves_round_like_plain_ones(dim, k, N):
    n1, omega = k * N + 1, 0.25 if dim == 2 else 0.1
    x = np.linspace(0.0, 1.0, n1)
    errs = np.zeros((2, 2))
    for tilt in (1.0, 2.0):
        b = (16.0 * (x * (1.0 - x)) ** 2 * (1.0 + tilt * x)).astype(np.float64)
        for _ in range(dim - 1):
            b = np.multiply.outer(b, 16.0 * (x * (1.0 - x)) ** 2 * (1.0 + tilt * x))
        b = b.astype(np.float32).astype(np.float64)
        ref = _plain(dim, k, N, b, omega, np.float64)
        p = P.Problem(dim, N, k, omega=omega)
        y = torch.full((b.size,), 7.0, dtype=torch.float32, device="cuda")
        p.smoother_step(dev(b.ravel(), torch.float32), None, y)
        for i, out in enumerate((host(y).reshape(b.shape), _plain(dim, k, N, b, omega, np.float32))):
            e = out - ref
            for j, part in enumerate((slice(None), slice(1, k + 1))):
                errs[i, j] += 0.5 * np.sum(e[..., part] ** 2) / np.sum(ref[..., part] ** 2)
        p.close()
    errs = np.sqrt(errs)
    for j, name in enumerate(("mesh", "first cell")):
        check(f"S(0,b) {dim}D Q{k} {N} {name}", errs[0, j], errs[1, j] + 2.0 ** -24 / np.sqrt(3.0))
