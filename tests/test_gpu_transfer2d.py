"""The 2D transfers on meshes that fill a part of their tiles, one tile or
several: without smoothing steps and without the one-launch tail the V-cycle is
P ... P A_0^{-1} P^T ... P^T b, compared with the oracle's dense 1D embeddings
and the Kronecker form of A_0."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2412_05082_amd as P
from gpu_util import EPS64, check, dev, host, rel_l2

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k,N", [(2, 4), (2, 64), (3, 8), (3, 32), (4, 4), (4, 32), (5, 8), (6, 16), (7, 4), (7, 16)])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_transfers_2d(k, N, dtype):
    n1 = k * N + 1
    b = np.pad(np.random.default_rng(k + N).uniform(-1.0, 1.0, (n1 - 2, n1 - 2)).astype(np.float32), 1).astype(float)
    E, Nc, r = [], N, b
    while Nc > 2:
        Nc //= 2
        E.append(np.asarray(O.prolongation_1d(k, Nc)))
        r = np.pad((E[-1].T @ r @ E[-1])[1:-1, 1:-1], 1)
    M, L, B = (m[1:-1, 1:-1] for m in P.host_matrices_1d(k, 2))
    A0 = np.kron(M, B) + 2.0 * np.kron(L, L) + np.kron(B, M)
    x = np.pad(np.linalg.solve(A0, r[1:-1, 1:-1].ravel()).reshape([2 * k - 1] * 2), 1)
    for e in reversed(E):
        x = np.pad((e @ x @ e.T)[1:-1, 1:-1], 1)
    p = P.Problem(2, N, k, omega=0.25, pre_steps=0, post_steps=0, tail_levels=0, vcycle_dtype=P.C0IP_F64)
    y = torch.full((n1 * n1,), 7.0, dtype=dtype, device="cuda")
    p.vcycle(dev(b.ravel(), dtype), y)
    kap = np.linalg.cond(A0)  # of the dense inverse
    check(f"transfers Q{k} {N}^2 {dtype}", rel_l2(host(y), x.ravel()),
          max(1e-12, 4.0 * kap * EPS64) if dtype == torch.float64 else 2e-5)
