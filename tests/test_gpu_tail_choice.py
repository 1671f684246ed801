"""The tail V-cycle in float64 on both sides of the choice between its kernel
with compile-time coefficients and the one with tables (by degree, top level
and number of smoothing steps), against the oracle, and a batch whose systems
enter one tail at levels on both sides."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2412_05082_amd as P
from gpu_util import check, dev, fp64_vcycle_tol, host, rel_l2, vectors

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k,N", [(2, 4), (2, 8), (2, 16), (2, 32), (3, 4), (3, 8), (3, 16), (4, 4), (4, 8)])
@pytest.mark.parametrize("pre,post", [(1, 1), (1, 2), (2, 2)])
def test_tail_on_both_sides_of_the_choice(k, N, pre, post):
    _, b = vectors(2, k, N)
    ref = O.Hierarchy(2, k, N, omega=0.25, pre=pre, post=post).vcycle(b)
    for coarse in (0, 1) if (pre, post) == (2, 2) else (0,):
        p = P.Problem(2, N, k, omega=0.25, pre_steps=pre, post_steps=post, coarse_mode=coarse,
                      vcycle_dtype=P.C0IP_F64)
        z = torch.full((b.size,), 7.0, dtype=torch.float64, device="cuda")
        p.vcycle(dev(b), z)
        if coarse:
            ref = O.Hierarchy(2, k, N, omega=0.25, pre=pre, post=post, coarse="smoother").vcycle(b)
        check(f"V-cycle Q{k} {N}^2 {pre}+{post} coarse {coarse}", rel_l2(host(z), ref),
              fp64_vcycle_tol(2, k, N, pre, post))
        p.close()


def test_batch_over_both_sides():
    problems = [(16, 3), (8, 3), (4, 3), (8, 2), (4, 4)]
    rng = np.random.default_rng(9)
    bs = []
    for N, k in problems:
        v = np.zeros((1, k * N + 1, k * N + 1))
        v[:, 1:-1, 1:-1] = rng.uniform(-1.0, 1.0, (1, k * N - 1, k * N - 1))
        bs.append(v.reshape(1, -1))
    batch = P.Batch(problems, [1] * len(problems), vcycle_dtype=P.C0IP_F64)
    dx = [torch.zeros_like(dev(v)) for v in bs]
    for (N, k), v, x, info in zip(problems, bs, dx, batch.solve([dev(v) for v in bs], dx, rtol=1e-8)):
        r = v[0] - O.assemble(2, k, N) @ host(x)[0]
        assert info["converged"] == 1
        check(f"residual Q{k} {N}^2", np.linalg.norm(r) / np.linalg.norm(v), 1.05e-8)
    batch.close()
