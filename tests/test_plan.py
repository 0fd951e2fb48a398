"""The launch plan's rules on the CPU (plan.h compiled for the host)."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

import pat_inputs as P
from conftest import ROOT

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
pd = ctypes.POINTER(ctypes.c_double)


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("plan") / "plan.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-w", "-shared", "-fPIC", "-I", os.path.join(ROOT, "tests", "hip_shim"),
                    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2609_29253_amd", "csrc"),
                    os.path.join(ROOT, "tests", "plan_driver.cpp"), "-o", so], check=True)
    return ctypes.CDLL(so)


def chunk(plan, K, volumes=1, n=128, rad=23.6, kept=2000, points=0, one_shape=True):
    """The adjoint's chunk: elements of radius `rad` shells on a sphere of 40 mm at 50 MHz."""
    s = np.concatenate([P.fibonacci_points(K, 40e-3) / 30e-6, np.full((K, 1), rad)], 1)
    s = np.ascontiguousarray(s)
    fn = plan.adjoint_chunk_of
    fn.argtypes = [pd, ctypes.c_int, ctypes.c_int, ctypes.c_double, ctypes.c_double] + [ctypes.c_int] * 5
    return fn(s.ctypes.data_as(pd), K, n, 0.1e-3 / 30e-6, 800.0, -40, kept, points, int(one_shape), volumes)


def test_adjoint_stays_whole_where_its_work_is_small(plan):
    """Two chunks cost the clearing, the adding and the cast of FP64 sums: 1.2 to 7 times
    the whole adjoint's time with few transducers, many volumes or a short window."""
    for K, volumes in ((1, 1), (2, 1), (8, 1), (2, 8), (8, 8), (32, 8)):
        assert chunk(plan, K, volumes) == K
    assert chunk(plan, 32, 1, kept=0) == 32 and chunk(plan, 32, 8, kept=100) == 32     # few samples kept
    assert chunk(plan, 2, 8, rad=112.0) == 2 and chunk(plan, 4, 8, points=16) == 4
    assert chunk(plan, 256, 8, n=256) == 256 and chunk(plan, 24, 1, one_shape=False) == 24


def test_adjoint_splits_where_it_pays(plan):
    for K, volumes, kw in ((256, 1, {}), (256, 8, {}), (33, 1, {}), (8, 1, dict(rad=112.0)), (64, 8, dict(rad=112.0)),
                           (8, 1, dict(points=16))):
        assert chunk(plan, K, volumes, **kw) == (K + 1) // 2, (K, volumes, kw)
    assert chunk(plan, 64, 1, n=32) == 2       # below 4096 bricks by their number, as many chunks as fill the device


def test_clearing_launch_fills_the_device(plan):
    """Bins few and sums many: as many work-groups as a fill takes (4096, or one per 256 sums);
    never fewer than the bins need, and no more where there is nothing to clear."""
    fn = plan.adjw_blocks_of
    fn.argtypes, fn.restype = [ctypes.c_long] * 3, ctypes.c_long
    for bins in (1, 190, 256, 257, 2200, 30000):
        for rows in (1, 2, 3, 64, 2048):
            need = -(-bins // 256)
            assert fn(bins, rows, 0) == need
            for sums in (1, 1000, 8 * 128 ** 3, 256 ** 3):
                got, fill = fn(bins, rows, sums), min(4096, -(-sums // 256))
                assert got >= need and got * rows >= fill
                assert got == need or (got - 1) * rows < fill


def share(plan, cyl, n=16, w=1.0, fp64=1):
    fn = plan.arc_share_of
    fn.argtypes, fn.restype = [pd, ctypes.c_int, ctypes.c_int, ctypes.c_double, ctypes.c_int], ctypes.c_double
    c = np.ascontiguousarray(cyl, float)
    return fn(c.ctypes.data_as(pd), len(c), n, w, fp64)


def test_share_of_the_weighted_areas_from_a_bounded_sample(plan):
    """At most 32 elements are looked at, the first and the last among them: the set-up of
    20000 does not grow (it did: 1.3 us an element)."""
    served, wide = [800.0, 0.1, 20.0, 300.0, 100.0, 0.0], [800.0, 1.2, 20.0, 300.0, 100.0, 0.0]
    assert share(plan, [served]) == 1.0 and share(plan, [wide]) == 0.0
    for K in (2, 31, 32, 33, 257, 20000):
        seen = [k for k in sorted({0, 1, K // 3, K // 2, K - 2, K - 1})
                if share(plan, [wide if j == k else served for j in range(K)]) < 1.0]
        assert 0 in seen and K - 1 in seen
        assert K > 32 or len(seen) == len({0, 1, K // 3, K // 2, K - 2, K - 1})
    hidden = sum(share(plan, [wide if j == k else served for j in range(200)]) == 1.0 for k in range(200))
    assert hidden == 200 - 32


@pytest.mark.parametrize("fp64,few", [(0, 16384), (1, 24576)])
def test_groups_that_the_weight_does_not_serve_keep_one_kind_of_pair(plan, fp64, few):
    fn = plan.carlson_only_of
    fn.argtypes = [ctypes.c_double, ctypes.c_long, ctypes.c_int]
    assert fn(0.0, 100, fp64) and fn(0.0, 10 ** 6, fp64) and fn(0.99, few - 1, fp64)
    assert not fn(0.99, few, fp64) and not fn(1.0, 100, fp64) and not fn(0.25, 10 ** 6, fp64)
    axis = [800.0, 0.12, 270.0, -3.0, -3.0, -3.0]      # voxels within 4 bins of the focal line
    assert share(plan, [axis], n=12, w=0.5, fp64=fp64) == 0.0
