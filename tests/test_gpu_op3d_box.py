"""The 3D operator on both sides of its switch between boxes of cells and the
march along z, and at high degrees (boxes of one layer that touch opposite
faces, first and last cell in one box or in different ones), against the
Kronecker form with the library's dense 1D factors (pinned to the exact ones
in test_lib_host.py).  Boundary entries of the input hold large values: they
must not count."""
import numpy as np
import pytest
import torch

import paper_2412_05082_amd as P
from gpu_util import check, dev, host, rel_l2
from test_gpu_op3d_boundary import _kron3

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k,N", [(2, 16), (2, 32), (3, 64), (4, 32), (5, 2), (5, 4), (5, 8), (6, 2), (6, 8), (7, 2),
                                 (7, 4), (7, 8)])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_operator_3d_boxes(k, N, dtype):
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
    # rounding of a sum: a few eps of the sum of its terms' sizes
    aM, aL, aB, ax = (np.abs(v) for v in (M, L, B, inner))
    size = sum(_kron3(f, ax) for f in ((aB, aM, aM), (aM, aB, aM), (aM, aM, aB)))
    size += 2.0 * sum(_kron3(f, ax) for f in ((aL, aL, aM), (aL, aM, aL), (aM, aL, aL)))
    bar = 4.0 * torch.finfo(dtype).eps * np.linalg.norm(size) / np.linalg.norm(ref)
    p = P.Problem(3, N, k, omega=0.1)
    y = torch.full((n1 ** 3,), 7.0, dtype=dtype, device="cuda")
    p.apply_A(dev(full.ravel(), dtype), y)
    check(f"A x 3D Q{k} {N}^3 {dtype}", rel_l2(host(y), ref.ravel()), bar)
    out = host(y).reshape(n1, n1, n1)
    assert all(np.all(np.take(out, e, axis=d) == 0.0) for d in range(3) for e in (0, n1 - 1))
