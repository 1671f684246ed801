"""The automatic choice of where a 2D multiplicative step forms its residual,
on both sides of the size that it turns on: degree 7 with the default penalty,
and another penalty at degree 2.  The automatic mode launches what the full
residual pass does on the finest level and what the in-launch residual does on
the level below, and every mode agrees with the coloured sweep in Kronecker
form: dense 1D factors of the library (pinned to the exact ones in
test_lib_host.py) and SciPy's local eigenbases."""
import numpy as np
import pytest
import scipy.linalg
import torch

import paper_2412_05082_amd as P
from capture_util import launches
from gpu_util import check, fp32_mvs_tol, fp64_mvs_tol, rel_l2

pytestmark = pytest.mark.gpu
SWITCH = 3 * 2 ** 19  # DoFs of a level


def _sweep(k, N, gamma, x, b):
    M, L, B = P.host_matrices_1d(k, N, gamma)
    n1, n = k * N + 1, 2 * k - 1
    E, lam = np.zeros(((N - 1) * n, n1)), np.zeros((N - 1) * n)
    kinds = {}  # local eigenbases: the first, the inner and the last vertex
    for v in range(1, N):
        s, r = slice((v - 1) * k + 1, (v - 1) * k + 1 + n), slice((v - 1) * n, v * n)
        t = 0 if v == 1 else 2 if v == N - 1 else 1
        if t not in kinds:
            kinds[t] = scipy.linalg.eigh(B[s, s], M[s, s])
        lam[r], E[r, s] = kinds[t][0], kinds[t][1].T
    M, L, B, E, lam = (torch.from_numpy(a).cuda() for a in (M, L, B, E, lam))
    v = torch.arange(1, N, device="cuda").repeat_interleave(n)
    for c in range(8):
        on = (((v[:, None] // 2 + v[None, :] // 2) % 2 == c // 4) & (v[:, None] % 2 == c // 2 % 2)
              & (v[None, :] % 2 == c % 2))
        r = b - (M @ x @ B + 2.0 * (L @ x @ L) + B @ x @ M)
        x = x + E.T @ (on * (E @ r @ E.T) / (lam[:, None] + lam[None, :])) @ E
    return x


@pytest.mark.parametrize("k,N,gamma", [(7, 256, 0.0), (2, 1024, 9.0)])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_automatic_residual_on_both_sides_of_the_switch(k, N, gamma, dtype):
    assert (k * N + 1) ** 2 >= SWITCH > (k * N // 2 + 1) ** 2
    gen = torch.Generator(device="cuda").manual_seed(11 * k)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        handles = [P.Problem(2, N, k, gamma=gamma, omega=1.0, smoother=1, mvs_residual=m,
                             vcycle_dtype=P.C0IP_F64 if dtype == torch.float64 else P.C0IP_F32) for m in (0, 1, 2)]
        top = handles[0].num_levels() - 1
        for level, Nl, same, other in ((top, N, 2, 1), (top - 1, N // 2, 1, 2)):
            n1 = k * Nl + 1
            x, b = (torch.nn.functional.pad(torch.rand((n1 - 2, n1 - 2), generator=gen, dtype=torch.float64,
                                                       device="cuda") * 2 - 1, (1, 1, 1, 1)).to(dtype).double()
                    for _ in range(2))
            ref = _sweep(k, Nl, gamma, x, b).cpu().numpy()
            xd, bd = (v.to(dtype).reshape(-1) for v in (x, b))
            y, counts = torch.empty_like(xd), []
            for m, p in enumerate(handles):
                y.fill_(7.0)
                p.smoother_step(bd, xd, y, level=level)
                # the floors depend on k, hardly on N
                bar = fp64_mvs_tol(2, k, 8) if dtype == torch.float64 else fp32_mvs_tol(2, k, 8, 1.0)
                check(f"Q{k} {Nl}^2 {dtype} mode {m}", rel_l2(y.double().cpu().numpy().reshape(n1, n1), ref), bar)
                counts.append(launches(stream, lambda: p.smoother_step(bd, xd, y, level=level)))
            assert counts[0] == counts[same] != counts[other]
        for p in handles:
            p.close()
