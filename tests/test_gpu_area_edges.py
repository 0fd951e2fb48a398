"""Bin edges on the voxels' projections, on the GPU against the oracle: everything
is a whole number of radial steps (c / fs = 2^-15 m) except r0, one rounding above
a whole number.  Tolerances and rows as in test_gpu_parity."""
import math

import numpy as np
import pytest

import oracle as O
import pat_inputs as P
from test_gpu_parity import check, run_gpu

pytestmark = pytest.mark.gpu

FS = float(2 ** 25)
DR = 1024.0 / FS


def lattice(rows, r0):
    grid = P.Grid.centred(9, DR)
    coef = np.random.default_rng(8).random((1, grid.N))
    p = P._finish("lattice", P.Transducers(np.array(rows)), grid, FS, 160, coef, 9)
    p.sound_speed, p.t0 = 1024.0, r0 / FS
    return p


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("r0", [math.nextafter(112.0, 200.0), math.nextafter(112.0, 0.0)])
def test_rectangles(gpu, r0, prec):
    x, y, z = [1.0, 0, 0], [0, 1.0, 0], [0, 0, 1.0]
    p = lattice([P.planar([0, 0, -130 * DR], x, y, 13.3 * DR, 9 * DR),
                 P.planar([125 * DR, 2 * DR, 0], y, z, 20 * DR, 6.4 * DR)], r0)
    s, z = run_gpu(p, "closed", prec)
    assert np.isfinite(s).all() and np.isfinite(z).all()
    check(f"{p.name} {r0} {prec}", prec, s, O.forward(p), z, O.adjoint(p))
