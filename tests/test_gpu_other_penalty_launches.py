"""Launches of a V-cycle with another penalty than k(k+1): on small levels the
first pre-smoothing step and the residual after it are one launch where that
is the faster form, as they are for the default penalty."""
import pytest
import torch

import paper_2412_05082_amd as P
from capture_util import launches

pytestmark = pytest.mark.gpu


def _vcycle_launches(gamma, k, N, vdt):
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        p = P.Problem(2, N, k, gamma=gamma, vcycle_dtype=vdt, tail_levels=0)
        b = torch.ones((k * N + 1) ** 2, dtype=torch.float64 if vdt == P.C0IP_F64 else torch.float32, device="cuda")
        z = torch.empty_like(b)
        p.vcycle(b, z)  # sets the levels up
        n = launches(s, lambda: p.vcycle(b, z))
        p.close()
    return n


@pytest.mark.parametrize("k,N", [(2, 8), (2, 128), (2, 256), (3, 8), (3, 64)])
@pytest.mark.parametrize("vdt", [P.C0IP_F64, P.C0IP_F32])
def test_pre_smoothing_and_residual_are_one_launch(k, N, vdt):
    assert _vcycle_launches(1.5 * k * (k + 1), k, N, vdt) == _vcycle_launches(0.0, k, N, vdt)
