"""The polynomial weight of the cylinder's areas on the CPU, FP32 input and output:
the areas of all bins of a pair add up to the element's, 4 R theta L, within the
weight's relative error (2.3e-11, what an evaluation by elliptic integrals leaves in
the bins of a scan's element) and 64 roundings of the variant."""
import math

import numpy as np
import pytest

from test_arc_areas import UNIT, areas, pytestmark  # noqa: F401


@pytest.mark.parametrize("theta,half", [(math.asin(0.15), 0.125e-3), (math.asin(0.12), 1.5e-3), (0.03, 1.5e-3)])
def test_areas_add_up_to_the_element(areas, theta, half):
    rng = np.random.default_rng(2)
    da = 1500 / 62.5e6
    R, hl, worst = 25e-3 / da, half / da, 0.0
    for _ in range(200):
        rho, phi, z = rng.uniform(1e-3, 8e-3) / da, rng.uniform(0, math.pi - theta), rng.uniform(-1.5e-3, 1.5e-3) / da
        near, far = int(R - rho) - 2, int(math.hypot(R + rho, abs(z) + hl)) + 3
        got, _ = areas([1, R, theta, hl], [rho * math.cos(phi), rho * math.sin(phi), z], 0.0, near, far, 0)
        worst = max(worst, abs(got.sum() / (4 * R * theta * hl) - 1))
    assert worst <= 2.3e-11 + 64 * UNIT[0], worst
