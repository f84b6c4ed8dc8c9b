"""Registered detectors that are coarse against the grid: a tile of 256 points
whose brick exceeds the LDS budget is staged in two or four parts, and a
wavefront whose own brick does not fit reads the grid."""
import numpy as np
import pytest
import torch

import paper_2109_05339_amd as spfel
import synth

from tests._common import DEV, detector, gpu, host, model

pytestmark = pytest.mark.gpu


# The detector of 50^2 points (nine whole tiles and one of 196) has its corner
# at the Nyquist radius, neighbouring points 0.89 cells apart on the 66^3 grid;
# scaled it runs from whole tiles (0.5) over pairs of wavefronts and single
# ones (1 .. 2) to reads of the grid (3 .. 8, bricks past 64 cells a side at
# 8), from 1.5 on with supports that wrap around the grid's ends.
@pytest.mark.parametrize("scale", [0.5, 0.8, 1.0, 1.3, 1.6, 2.0, 3.0, 8.0])
@pytest.mark.parametrize("w,domain", [(6, spfel.REAL), (6, spfel.COMPLEX), (4, spfel.REAL),
                                      (8, spfel.REAL), (7, spfel.COMPLEX)])
def test_parts_of_a_tile_equal_the_per_point_path(w, domain, scale):
    """Same cells, weights and order of sums: bitwise equal."""
    det = detector(50) * scale
    q = synth.quaternions(synth.config(1), "ref_quats", 5)
    q[3] = 0.0
    plan = spfel.Plan(33, kernel_width=w, domain=domain, device=DEV)
    m = model(1)
    if domain == spfel.REAL:
        plan.set_model(gpu(m))
    else:
        plan.set_model(gpu(synth.complex_perturbation(synth.config(4), m), torch.complex64))
    plan.set_detector(gpu(det))
    a = host(plan.slice(gpu(q))[0])
    b = host(plan.slice(gpu(q), gpu(det))[0])
    np.testing.assert_array_equal(a, b)
    assert np.all(np.isnan(a[3])) and np.all(np.isfinite(a[[0, 1, 2, 4]]))


# (blocks = 10 tiles per row) on both sides of the launches that read the grid
# instead of staging parts: REAL 250 and 260 blocks, COMPLEX 1,020 and 1,030
@pytest.mark.parametrize("w,domain,rows", [(6, spfel.REAL, 25), (6, spfel.REAL, 26), (6, spfel.COMPLEX, 102),
                                           (6, spfel.COMPLEX, 103), (4, spfel.REAL, 30), (8, spfel.COMPLEX, 104),
                                           (7, spfel.REAL, 26)])
@pytest.mark.parametrize("scale", [0.5, 1.0, 1.6, 3.0])
def test_many_and_few_blocks_equal_the_per_point_path(w, domain, rows, scale):
    det = detector(50) * scale
    q = synth.quaternions(synth.config(1), "ref_quats", rows)
    q[3] = 0.0
    plan = spfel.Plan(33, kernel_width=w, domain=domain, device=DEV)
    m = model(1)
    if domain == spfel.REAL:
        plan.set_model(gpu(m))
    else:
        plan.set_model(gpu(synth.complex_perturbation(synth.config(4), m), torch.complex64))
    plan.set_detector(gpu(det))
    a = host(plan.slice(gpu(q))[0])
    b = host(plan.slice(gpu(q), gpu(det))[0])
    np.testing.assert_array_equal(a, b)
    assert np.all(np.isnan(a[3])) and np.all(np.isfinite(np.delete(a, 3, axis=0)))
