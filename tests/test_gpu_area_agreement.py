"""A cylinder pair's areas do not depend on the other voxels of its wave having
coefficients: a volume of one voxel gives the same FP64 signals alone and beside
a dense volume in the same batch (one voxel's bins have one order of summation).
The cubes of 4 x 4 x 4 voxels span several levels of the weight's polynomials, whose
areas differ by 6e-14 and more; the wave also picks the series of the arc's angle,
all of which round at 2^-53 of it, a few 1e-15 of a signal: 1e-14."""
import numpy as np
import pytest
import torch

import pat_inputs as P

pytestmark = pytest.mark.gpu


def test_one_voxel_alone_and_beside_a_dense_volume(gpu):
    from paper_2609_29253_amd.operator import PatOperator
    rows = []
    for a in np.radians([25.0, 35.0, 45.0, 55.0]):     # the volume's angle from the element's direction
        d = np.array([np.cos(a), np.sin(a), 0.0])
        rows.append(P.cylinder(-10e-3 * d, [0, 0, 1.0], [1.0, 0, 0], 25e-3, 0.15, 0.5e-3))
    grid = P.Grid.centred(8, 0.5e-3)
    dense = np.random.default_rng(1).random(grid.N)
    p = P._finish("levels", P.Transducers(np.array(rows)), grid, 40e6, 1200, np.stack([dense, dense]), 2)
    op = PatOperator.from_problem(p, mode="closed", precision="fp64", max_batch=2)
    dense = torch.tensor(dense, dtype=torch.float64, device=gpu)
    worst = 0.0
    for i in range(0, grid.N, 37):
        one = torch.zeros(2, grid.N, dtype=torch.float64, device=gpu)
        one[0, i] = 1.0
        alone = op.forward(one)[0].cpu().numpy()
        one[1] = dense
        beside = op.forward(one)[0].cpu().numpy()
        assert np.any(alone)
        worst = max(worst, np.abs(alone - beside).max() / np.abs(alone).max())
    op.close()
    assert worst <= 1e-14
