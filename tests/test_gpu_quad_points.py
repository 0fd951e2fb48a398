"""Point-method kernels at point grids whose columns leave a remainder of their
step (odd, one) and at ones of one row, against the oracle: tolerances and rows
as in test_gpu_parity (the bins are decided in FP64 on both sides)."""
import pytest

import oracle as O
import pat_inputs as P
from test_gpu_parity import check, run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("shape", [P.PLANAR, P.CYLINDER])
@pytest.mark.parametrize("quad_n", [(1, 1), (3, 5), (7, 2), (1, 33)])
def test_point_grids(gpu, quad_n, shape, prec):
    p = P.small_case(shape, n=9, K=3, L=260, U=2, seed=21)
    p.quad_n = quad_n
    s, z = run_gpu(p, "quadrature", prec)
    check(f"{p.name} {quad_n} {prec}", prec, s, O.forward(p, mode=O.MODE_POINT), z, O.adjoint(p, mode=O.MODE_POINT))
