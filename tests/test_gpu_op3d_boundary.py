"""The 3D operator on meshes whose tiles meet the boundary in every way (a
single cell row, tiles cut by the mesh, first and last cell in one tile or in
different ones, one cell per z chunk), against the Kronecker form with the
library's dense 1D factors (pinned to the exact ones in test_lib_host.py).
Boundary entries of the input hold large values: they must not count."""
import numpy as np
import pytest
import torch

import paper_2412_05082_amd as P
from gpu_util import check, dev, host, rel_l2

pytestmark = pytest.mark.gpu


def _kron3(F, X):
    for d, A in enumerate(F):
        X = np.moveaxis(np.tensordot(A, X, axes=(1, d)), 0, d)
    return X


@pytest.mark.parametrize("k,N", [(2, 2), (2, 8), (2, 16), (2, 32), (3, 2), (3, 4), (3, 16), (3, 32), (4, 2), (4, 8),
                                 (4, 16)])
@pytest.mark.parametrize("dtype,bar", [(torch.float64, 1e-12), (torch.float32, 1e-5)])
def test_operator_3d_at_the_boundary(k, N, dtype, bar):
    n1 = k * N + 1
    x = np.random.default_rng(k * 100 + N).uniform(-1.0, 1.0, (n1, n1, n1))
    inner = np.zeros_like(x)
    inner[1:-1, 1:-1, 1:-1] = x[1:-1, 1:-1, 1:-1]
    if dtype == torch.float32:
        inner = inner.astype(np.float32).astype(np.float64)
    full = np.where(inner == 0.0, 1e6 * x, inner)
    M, L, B = P.host_matrices_1d(k, N)
    ref = sum(_kron3(f, inner) for f in ((B, M, M), (M, B, M), (M, M, B)))
    ref += 2.0 * sum(_kron3(f, inner) for f in ((L, L, M), (L, M, L), (M, L, L)))
    p = P.Problem(3, N, k, omega=0.1)
    y = torch.full((n1 ** 3,), 7.0, dtype=dtype, device="cuda")
    p.apply_A(dev(full.ravel(), dtype), y)
    check(f"A x 3D Q{k} {N}^3 {dtype}", rel_l2(host(y), ref.ravel()), bar)
    out = host(y).reshape(n1, n1, n1)
    assert all(np.all(np.take(out, e, axis=d) == 0.0) for d in range(3) for e in (0, n1 - 1))
