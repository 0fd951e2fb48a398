"""The sparse forward's items (groups of 64 nonzeros x some transducers), whose
number of transducers follows from the number of nonzeros: one, two and sixteen
a piece, with transducers that do not divide among them, against the full
forward.  Both sum the same FP64 terms in other orders: 1e-12, as for the other
supports; 1e-6 with FP32 output.
"""
import numpy as np
import pytest
import torch

import pat_inputs as P
from conftest import rel_l2

pytestmark = pytest.mark.gpu

DT = {"fp32": torch.float32, "fp64": torch.float64}
SELF = {"fp32": 1e-6, "fp64": 1e-12}


@pytest.mark.parametrize("shape", ["planar", "cylinder"])
@pytest.mark.parametrize("nonzeros,K,prec", [(1, 5, "fp64"), (64, 17, "fp64"), (65, 17, "fp64"), (33000, 63, "fp32"),
                                             (33000, 65, "fp64"), (48 ** 3, 301, "fp32")])
def test_items_of_every_size(gpu, shape, nonzeros, K, prec):
    from paper_2609_29253_amd.operator import PatOperator
    p = P.small_case(P.CYLINDER if shape == "cylinder" else P.PLANAR, n=48, K=K, L=700, seed=11)
    coef = np.zeros_like(p.coef)
    rng = np.random.default_rng(5)
    at = rng.permutation(p.N)[:nonzeros]
    coef[0, at] = rng.uniform(0.5, 1.5, at.size)
    op = PatOperator.from_problem(p, mode="closed", precision=prec)
    c = torch.tensor(coef, dtype=DT[prec], device=gpu)
    full = op.forward(c).cpu().numpy()
    sparse = op.forward(c, sparse=True).cpu().numpy()
    op.close()
    assert np.linalg.norm(full) > 0 and rel_l2(sparse, full) < SELF[prec]
