"""The rectangles' areas on the CPU at the distances and bin numbers of real
geometries (thousands to a hundred thousand bins, on the axis and far off it),
against 30 digits.

Tolerance with FP64 input and output, of the pair's largest area: an edge counts
from the quadrant's nearest corner, so what rounds are the corner's distance D
(2^-53 D twice, which shifts a bin by that share of it at either edge) and the
area nearer than the edge (at most the element's, 32 roundings of it).  With FP32,
whose differences are of r^2 - |x3|^2: half a unit in the last place of the output."""
import math

import mpmath as mp
import numpy as np
import pytest

from test_arc_areas import areas, below, pytestmark  # noqa: F401


def errors(areas, L1, L2, x, r0):
    d = np.maximum(0, np.abs(x[:2]) - [L1, L2])
    near = math.hypot(np.linalg.norm(d), x[2])
    far = math.hypot(np.linalg.norm(np.abs(x[:2]) + [L1, L2]), x[2])
    lo, hi = math.floor(near - r0) - 1, math.ceil(far - r0) + 1
    tr = [0, L1, L2, 0]
    bins = sorted({*range(lo, min(lo + 5, hi)), *range(max(hi - 5, lo), hi + 1),
                   *np.linspace(lo, hi, 9).round().astype(int).tolist()})
    with mp.workdps(30):
        at = lambda m: below(tr, x, max(mp.mpf(r0) + m, 0))  # noqa: E731
        ref = np.array([float(at(m) - at(m - 1)) for m in bins])
    out = []
    for kind in (0, 1):
        got, _ = areas(tr, x, r0, lo, hi, kind)
        assert np.isfinite(got).all()
        out.append((np.abs(got[np.array(bins) - lo] - ref).max(), got.max()))
    return out, far


@pytest.mark.parametrize("distance", [2e3, 2e4, 1e5])
@pytest.mark.parametrize("angle", [0, 30, 60, 85])
@pytest.mark.parametrize("half", [(8.3, 50.0), (36.7, 36.7), (101.7, 101.7)])
def test_oblique_rectangles(areas, half, angle, distance):
    L1, L2 = half
    rng = np.random.default_rng(int(angle + distance))
    for r0 in (0.0, 250.25, math.nextafter(120.0, 200.0)):
        a, phi = math.radians(angle), rng.uniform(0, 2 * math.pi)
        x = [distance * math.sin(a) * math.cos(phi) + rng.uniform(-3, 3),
             distance * math.sin(a) * math.sin(phi) + rng.uniform(-3, 3), distance * math.cos(a)]
        (e32, t32), (e64, t64) = errors(areas, L1, L2, x, r0)[0]
        assert e64 <= 4 * 2.0 ** -53 * distance * t64 + 32 * 2.0 ** -53 * 4 * L1 * L2, (x, r0)
        assert e32 <= 2.0 ** -24 * t32, (x, r0)


def test_edges_on_every_corner(areas):
    """Corners at whole distances (multiples of 3, 4, 5 and 300, 400, 1200, 1300): the edge
    between two bins passes through them."""
    for L, z in (((300.0, 300.0), 400.0), ((300.0, 1200.0), 400.0), ((9.0, 9.0), 12.0)):
        for u, v in ((0.0, 0.0), (L[0], 0.0), (0.0, L[1]), (L[0], L[1])):
            out, far = errors(areas, *L, [u, v, z], 0.0)
            e64, t64 = out[1]
            assert e64 <= 4 * 2.0 ** -53 * far * t64 + 32 * 2.0 ** -53 * 4 * L[0] * L[1], (L, z, u, v)


@pytest.mark.parametrize("r0", [math.nextafter(120.0, 200.0), (112 / 50e6) * 50e6, math.nextafter(120.0, 0.0), 100.1,
                                0.3])
def test_edge_on_the_projection(areas, r0):
    """r0 one rounding off a whole number of bins (t0 fs U is) and voxels at whole
    distances in front of the element: the shell has radius zero in its plane."""
    L1, L2 = 13.3, 9.0
    for z in [float(int(r0) + 1 + i) for i in range(24)] + [r0 + 1 + i for i in range(24)]:
        for u, v in ((0.0, 0.0), (5.0, -3.0)):
            out, far = errors(areas, L1, L2, [u, v, z], r0)
            e64, t64 = out[1]
            assert e64 <= 4 * 2.0 ** -53 * far * t64 + 32 * 2.0 ** -53 * 4 * L1 * L2, (z, u, v)
