"""The 3D additive smoother at degrees 5 to 7 on one patch, on boxes that touch
opposite faces and on boxes with and without neighbours, from 0, from x and in
place, against the Kronecker form of the step."""
import numpy as np
import pytest
import torch

import paper_2412_05082_amd as P
from gpu_util import check, dev, fp32_tol, fp64_tol, host, rel_l2
from test_gpu_smooth3d_tiles import OMEGA, _step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k,N", [(5, 2), (5, 4), (5, 8), (6, 2), (6, 4), (6, 8), (7, 2), (7, 4), (7, 8)])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_smoother_3d_boxes(k, N, dtype):
    n1 = k * N + 1
    rng = np.random.default_rng(10 * k + N)
    x, b = np.zeros((n1, n1, n1)), np.zeros((n1, n1, n1))
    for v in (x, b):
        v[1:-1, 1:-1, 1:-1] = rng.uniform(-1.0, 1.0, (n1 - 2, n1 - 2, n1 - 2)).astype(np.float32)
    bar = fp64_tol(3, k, 2) if dtype == torch.float64 else fp32_tol(3, k, 2)
    p = P.Problem(3, N, k, omega=OMEGA)
    out = torch.full((n1 ** 3,), 7.0, dtype=dtype, device="cuda")
    for name, xi in (("S(0,b)", None), ("S(x,b)", x)):
        p.smoother_step(dev(b.ravel(), dtype), None if xi is None else dev(xi.ravel(), dtype), out)
        check(f"{name} 3D Q{k} {N}^3 {dtype}", rel_l2(host(out), _step(k, N, xi, b).ravel()), bar)
    xs = dev(x.ravel(), dtype)  # in place
    p.apply_smoother(dev(b.ravel(), dtype), xs)
    assert torch.equal(xs, out)
