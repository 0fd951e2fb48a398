"""A window of few samples: transducers none of whose shells it keeps, ones whose
shells it cuts and ones it sees whole, in one array, against the oracle
(tolerances and rows as in test_gpu_parity)."""
import numpy as np
import pytest

import oracle as O
import pat_inputs as P
from test_gpu_parity import check, run_gpu

pytestmark = pytest.mark.gpu


def cut_case(shapes, L, B=1):
    p = P.mixed_case(n=9, K_planar=3, K_cyl=3, L=L, seed=12, B=B)
    rows = p.tr.packed[np.isin(p.tr.packed[:, 0], shapes)].copy()
    out = rows[:, 1:4] + (rows[:, 0] == 1)[:, None] * rows[:, 12:13] * rows[:, 7:10]     # centre of the surface
    out /= np.linalg.norm(out, axis=1)[:, None]
    rows[:, 1:4] += np.linspace(0.0, 4e-3, len(rows))[:, None] * out
    q = P._finish("cut", P.Transducers(rows), p.grid, p.fs, L, p.coef, 13)
    assert not q.meta["window_covers_signal"]
    return q


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("shapes,L,B", [((0,), 110, 1), ((1,), 100, 1), ((0, 1), 90, 2), ((0, 1), 130, 1)])
def test_short_window(gpu, shapes, L, B, prec):
    p = cut_case(shapes, L, B)
    s_ref, z_ref = O.forward(p), O.adjoint(p)
    rows = np.abs(s_ref).max(axis=(0, 2))
    assert rows.max() > 0 and rows.min() < 1e-3 * rows.max()
    s, z = run_gpu(p, "closed", prec)
    silent = rows == 0
    assert not np.any(s[:, silent])
    check(f"{p.name} {shapes} {L} {prec}", prec, s[:, ~silent], s_ref[:, ~silent], z, z_ref)
