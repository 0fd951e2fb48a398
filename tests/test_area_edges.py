"""The kernels' area sweeps on the CPU where a bin edge falls on a quadrant's
nearest corner, which the voxel's projection is: r0 one rounding off a whole
number of bins (t0 fs U is), voxels at whole distances.  There the shell through
that edge has radius zero in the element's plane.

Tolerance, of the pair's largest area: that of test_arc_areas (64 roundings of the
variant in terms of the size of r^2 - |x|^2 at the farthest corner, the weight
polynomial's error) and the rounding of r^2 - |x|^2 itself, 2^-52 r^2, which
moves an area by at most that much."""
import math

import mpmath as mp
import numpy as np
import pytest

from test_arc_areas import POLY, UNIT, areas, below, pytestmark  # noqa: F401

R0 = [math.nextafter(120.0, 200.0), (112 / 50e6) * 50e6, math.nextafter(120.0, 0.0), 100.1, 0.3]


def compare(areas, tr, x, r0, near, far, kind, poly):
    lo, hi = math.floor(near - r0) - 1, math.ceil(far - r0) + 2
    got, _ = areas(tr, x, r0, lo, hi, kind)
    assert np.isfinite(got).all(), (tr, x, r0, kind)
    with mp.workdps(30):
        at = [below(tr, x, max(mp.mpf(r0) + m, 0)) for m in range(lo - 1, hi + 1)]
        ref = np.array([float(b - a) for a, b in zip(at, at[1:])])
    tol = 64 * UNIT[kind] * (far ** 2 - near ** 2) + 2.0 ** -52 * far ** 2 + poly * ref.max()
    assert np.abs(got - ref).max() <= tol, (tr, x, r0, kind, np.abs(got - ref).max(), tol)
    # the same where a window starts at the edge on the corner and after it
    for a in range(lo, lo + 4):
        assert np.array_equal(areas(tr, x, r0, a, hi, kind)[0], got[a - lo:])


@pytest.mark.parametrize("kind", [0, 1])
@pytest.mark.parametrize("r0", R0)
def test_planar_edge_on_the_projection(areas, r0, kind):
    L1, L2 = 13.3, 9.0
    for z in [float(int(r0) + 1 + i) for i in range(24)] + [r0 + 1 + i for i in range(24)]:
        for u, v in ((0.0, 0.0), (5.0, -3.0)):
            far = math.sqrt((L1 + u) ** 2 + (L2 + abs(v)) ** 2 + z * z)
            compare(areas, [0, L1, L2, 0], [u, v, z], r0, z, far, kind, 0.0)


@pytest.mark.parametrize("kind", [0, 1])
@pytest.mark.parametrize("r0", R0)
def test_cylinder_edge_on_the_projection(areas, r0, kind):
    R, th, hl = 300.0, 0.05, 21.0
    for d in [float(int(r0) + 1 + i) for i in range(8)] + [r0 + 1 + i for i in range(8)]:
        rho = R - d
        far = math.sqrt(d * d + 4 * R * rho * math.sin(th / 2) ** 2 + hl * hl)
        compare(areas, [1, R, th, hl], [rho, 0.0, 0.0], r0, d, far, kind, POLY[kind])


@pytest.mark.parametrize("kind", [0, 1])
def test_far_side_of_the_cylinder(areas, kind):
    """The interval's end at u = pi up to rounding, and a bin edge there (r = R + rho)."""
    R, hl, rho = 300.0, 21.0, 150.0
    for th in np.linspace(0.05, 0.6, 56):
        for phi in (math.pi - th, np.nextafter(math.pi - th, 0), np.nextafter(math.pi - th, 4)):
            got, _ = areas([1, R, th, hl], [rho * math.cos(phi), rho * math.sin(phi), 0.0], 0.0, 100, 480, kind)
            assert np.isfinite(got).all() and got.min() > -1e-6 * got.max()
