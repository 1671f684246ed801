"""The 3D operator's march along z at every degree that takes it (2 to 4), on
the smallest meshes that do (32^3 at degree 2, 64^3 above): A x and the
residual form, the latter through a smoother step, against the Kronecker form
in float64 with the library's dense 1D factors (pinned to the exact ones in
test_lib_host.py) and SciPy's local eigenbases.  Boundary entries of the inputs
hold large values: they must not count."""
import numpy as np
import pytest
import scipy.linalg
import torch

import paper_2412_05082_amd as P
from gpu_util import check, fp32_tol, fp64_tol

pytestmark = pytest.mark.gpu
OMEGA = 0.1


def _kron3(F, X):
    for d, A in enumerate(F):
        X = torch.movedim(torch.tensordot(A, X, dims=([1], [d])), 0, d).contiguous()
    return X


def _apply(F, X):
    M, L, B = F
    return (sum(_kron3(f, X) for f in ((B, M, M), (M, B, M), (M, M, B)))
            + 2.0 * sum(_kron3(f, X) for f in ((L, L, M), (L, M, L), (M, L, L))))


def _factors(k, N):
    M, L, B = P.host_matrices_1d(k, N)
    n1, n = k * N + 1, 2 * k - 1
    E, lam = np.zeros(((N - 1) * n, n1)), np.zeros((N - 1) * n)
    for v in range(1, N):
        s, r = slice((v - 1) * k + 1, (v - 1) * k + 1 + n), slice((v - 1) * n, v * n)
        lam[r], Q = scipy.linalg.eigh(B[s, s], M[s, s])
        E[r, s] = Q.T
    return [torch.from_numpy(a).cuda() for a in (M, L, B)], *(torch.from_numpy(a).cuda() for a in (E, lam))


def _inputs(n1, seed, dtype, count):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    for _ in range(count):
        full = torch.rand((n1, n1, n1), generator=gen, dtype=torch.float64, device="cuda") * 2 - 1
        full = full.to(dtype).double()
        inner = torch.zeros_like(full)
        inner[1:-1, 1:-1, 1:-1] = full[1:-1, 1:-1, 1:-1]
        yield inner, torch.where(inner == 0.0, 1e6 * full, full)


@pytest.mark.parametrize("k,N", [(2, 32), (3, 64), (4, 64)])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_march_at_every_degree(k, N, dtype):
    n1, f64 = k * N + 1, dtype == torch.float64
    F, E, lam = _factors(k, N)
    (x, xf), (b, bf) = _inputs(n1, 10 * k + N, dtype, 2)
    ax = _apply(F, x)
    # rounding of a sum: a few eps of the sum of its terms' sizes
    size = _apply([a.abs() for a in F], x.abs())
    bar = 4.0 * torch.finfo(dtype).eps * (size.norm() / ax.norm()).item()
    p = P.Problem(3, N, k, omega=OMEGA, vcycle_dtype=P.C0IP_F64 if f64 else P.C0IP_F32)
    y = torch.full((n1 ** 3,), 7.0, dtype=dtype, device="cuda")
    p.apply_A(xf.to(dtype).reshape(-1), y)
    out = y.double().reshape(n1, n1, n1)
    check(f"A x 3D Q{k} {N}^3 {dtype}", ((out - ax).norm() / ax.norm()).item(), bar)
    assert all(bool((out.select(d, e) == 0.0).all()) for d in range(3) for e in (0, n1 - 1))
    p.smoother_step(bf.to(dtype).reshape(-1), xf.to(dtype).reshape(-1), y)
    T = _kron3((E, E, E), b - ax) / (lam[:, None, None] + lam[None, :, None] + lam[None, None, :])
    ref = x + OMEGA * _kron3([E.T.contiguous()] * 3, T)
    out = y.double().reshape(n1, n1, n1)
    check(f"S(x,b) 3D Q{k} {N}^3 {dtype}", ((out - ref).norm() / ref.norm()).item(),
          fp64_tol(3, k, 4) if f64 else fp32_tol(3, k, 4))
