"""The 3D transfers on meshes that fill a part of their tiles, one tile or
several: without smoothing steps the V-cycle is P ... P A_0^{-1} P^T ... P^T b,
compared with the oracle's dense 1D embeddings and the Kronecker form of A_0."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2412_05082_amd as P
from gpu_util import EPS64, check, dev, host, rel_l2
from test_gpu_op3d_boundary import _kron3

pytestmark = pytest.mark.gpu


def _inner(v):
    z = np.zeros_like(v)
    z[1:-1, 1:-1, 1:-1] = v[1:-1, 1:-1, 1:-1]
    return z


@pytest.mark.parametrize("k,N", [(2, 4), (2, 8), (2, 32), (3, 4), (3, 16), (4, 8), (5, 8), (6, 4), (6, 8), (7, 4)])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_transfers_3d(k, N, dtype):
    n1 = k * N + 1
    b = _inner(np.random.default_rng(k + N).uniform(-1.0, 1.0, (n1, n1, n1)).astype(np.float32).astype(np.float64))
    E, Nc, r = [], N, b
    while Nc > 2:
        Nc //= 2
        E.append(np.asarray(O.prolongation_1d(k, Nc)))
        r = _inner(_kron3((E[-1].T,) * 3, r))
    M, L, B = (m[1:-1, 1:-1] for m in P.host_matrices_1d(k, 2))
    k3 = lambda f: np.kron(f[0], np.kron(f[1], f[2]))  # noqa: E731
    A0 = sum(map(k3, ((B, M, M), (M, B, M), (M, M, B)))) + 2.0 * sum(map(k3, ((L, L, M), (L, M, L), (M, L, L))))
    x = np.zeros_like(r)
    x[1:-1, 1:-1, 1:-1] = np.linalg.solve(A0, r[1:-1, 1:-1, 1:-1].ravel()).reshape([2 * k - 1] * 3)
    for e in reversed(E):
        x = _inner(_kron3((e, e, e), x))
    p = P.Problem(3, N, k, omega=0.1, pre_steps=0, post_steps=0, vcycle_dtype=P.C0IP_F64)
    y = torch.full((n1 ** 3,), 7.0, dtype=dtype, device="cuda")
    p.vcycle(dev(b.ravel(), dtype), y)
    # the dense inverse's rounding; in float32 the transferred values', damped or not
    kap = np.linalg.cond(A0)
    check(f"transfers Q{k} {N}^3 {dtype}", rel_l2(host(y), x.ravel()),
          max(1e-12, 4.0 * kap * EPS64) if dtype == torch.float64 else 2e-5)
