"""The binned spread at the edges of its tiling, against the oracle's type 1:
every kernel width (each has its own bins, rows and matrix tiles) in both
domains, image counts around the eight images a binning block takes, ragged
detector tiles, a grid smaller than a brick, points crowded into a few bins
(several subproblems and full wavefront batches per bin) and spread over many
(runs shorter than a matrix step).  Bar: the parity bar of the merge tests
(1e-5 relative L2); a float32 sum of n terms in any order is off by at most
n u, about 1e-5 only for n above a hundred terms per cell of random signs."""
import numpy as np
import pytest
import torch

import paper_2109_05339_amd as spfel
import synth
from oracle import geometry, nufft
from tests._common import DEV, f32, gpu, host, rel

pytestmark = pytest.mark.gpu


def check(N, w, real, n_img, n_det, shrink, weights=False, drop=0):
    q = synth.quaternions(synth.config(4), "image_quats", n_img).astype(np.float32)
    det = (synth.detector_q(n_det) * shrink).astype(np.float32)[drop:]
    P = len(det)
    x = geometry.slice_points(f32(q), f32(det)).reshape(-1, 3)
    g = np.random.default_rng(N * 100 + w)
    y = g.standard_normal((n_img, P)).astype(np.float32)
    if not real:
        y = (y + 1j * g.standard_normal((n_img, P))).astype(np.complex64)
    wt = (0.5 + 0.5 * g.random((n_img, P))).astype(np.float32) if weights else None
    plan = spfel.Plan(N, kernel_width=w, domain=spfel.REAL if real else spfel.COMPLEX, device=DEV)
    plan.set_detector(gpu(det))
    dt = torch.float32 if real else torch.complex64
    wide = y.astype(np.float64 if real else np.complex128)
    want = nufft.nufft1((wide if wt is None else wide * f32(wt)).ravel(), x, N, w=w, real=real)
    for _ in range(2):   # the second merge finds the first's counts and accumulator cleared
        out = plan.merge_adjoint(gpu(q), None, gpu(y, dt), None if wt is None else gpu(wt))
        assert rel(host(out), want) <= 1e-5


@pytest.mark.parametrize("w", [4, 5, 6, 7, 8])
@pytest.mark.parametrize("real", [True, False])
def test_widths(w, real):
    check(17, w, real, 9, 20, 1.0, weights=True, drop=13)


@pytest.mark.parametrize("n_img", [1, 7, 8, 9, 17])
def test_image_counts_and_ragged_tiles(n_img):
    check(15, 6, True, n_img, 17, 1.0, drop=1)


@pytest.mark.parametrize("N,w", [(5, 4), (5, 5), (7, 6), (7, 7)])
def test_grids_smaller_than_a_brick(N, w):
    check(N, w, True, 3, 9, 1.0)


@pytest.mark.parametrize("w", [4, 5, 6, 7, 8])
@pytest.mark.parametrize("real", [True, False])
def test_crowded_bins(w, real):
    # 40 x 400 points within two cells of the origin: a few bins of
    # thousands of points each, cut into several subproblems
    check(13, w, real, 40, 20, 0.08)


@pytest.mark.parametrize("domain", [spfel.REAL, spfel.COMPLEX])
def test_recorded_merges_do_not_count_as_run(domain):
    """A plan keeps its accumulator and bin counts cleared between merges.  A
    merge that is captured has not run: an eager one right after the capture,
    before any replay, and replays between eager ones give the same sums."""
    det = synth.detector_q(24).astype(np.float32)
    q = gpu(synth.quaternions(synth.config(4), "image_quats", 9))
    dtype = torch.float32 if domain == spfel.REAL else torch.complex64
    v = gpu(np.random.default_rng(3).standard_normal((9, len(det))), dtype)
    other = spfel.Plan(25, domain=domain, device=DEV)   # loads the kernels before the capture
    other.set_detector(gpu(det))
    ref = host(other.merge_adjoint(q, None, v))
    plan = spfel.Plan(25, domain=domain, device=DEV)
    plan.set_detector(gpu(det))
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = plan.merge_adjoint(q, None, v)
    eager = [host(plan.merge_adjoint(q, None, v))]
    for _ in range(3):
        graph.replay()
        torch.cuda.synchronize()
        eager.append(host(out.clone()))
        eager.append(host(plan.merge_adjoint(q, None, v)))
    for got in eager:   # float atomics in any order: a few roundings per cell
        assert rel(got, ref) <= 1e-5


@pytest.mark.parametrize("domain", [spfel.REAL, spfel.COMPLEX])
def test_replays_of_a_recorded_deferred_merge_stay_out_of_later_merges(domain):
    """A deferred merge that is recorded leaves its sums in the accumulator on
    each replay.  After an eager merge has finished it, a replay that nothing
    finishes is not part of the next complete merge."""
    det = synth.detector_q(24).astype(np.float32)
    q = gpu(synth.quaternions(synth.config(4), "image_quats", 9))
    dtype = torch.float32 if domain == spfel.REAL else torch.complex64
    v = gpu(np.random.default_rng(3).standard_normal((9, len(det))), dtype)
    plan = spfel.Plan(25, domain=domain, device=DEV)
    plan.set_detector(gpu(det))
    ref = host(plan.merge_adjoint(q, None, v))
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        plan.merge_adjoint(q, None, v, flags=spfel.MERGE_DEFER)
    graph.replay()
    assert rel(host(plan.merge_adjoint(q, None, v)), 2 * ref) <= 1e-5   # finishes the deferred one
    for _ in range(2):
        graph.replay()
        torch.cuda.synchronize()
        for _ in range(2):
            assert rel(host(plan.merge_adjoint(q, None, v)), ref) <= 1e-5
