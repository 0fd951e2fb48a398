"""The temporal stage on both sides of the up-sampling factor at which its windows no
longer fit LDS (48), several volumes and samples that leave a remainder of its
work-groups, against the oracle: tolerances and rows as in test_gpu_parity."""
import pytest

import oracle as O
import pat_inputs as P
from test_gpu_parity import check, run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("U,B,L", [(47, 1, 200), (48, 2, 257), (49, 1, 200), (49, 2, 257), (64, 1, 200)])
def test_fine_arrival_grids(gpu, U, B, L, prec):
    p = P.small_case(P.PLANAR, n=4, K=3, L=L, U=U, B=B, seed=31)
    s, z = run_gpu(p, "closed", prec)
    check(f"{p.name} U={U} B={B} {prec}", prec, s, O.forward(p), z, O.adjoint(p))
