"""The line transforms behind the separable 3D DFTs at the sizes where their
tiling changes: below, at and just past whole tiles of 16 output rows and
steps of 4 input slots, lengths whose tables take two, four and eight
wavefronts and more row tiles than wavefronts, and lengths whose fused axis-0
pass does not fit the LDS.

Reference: the same operator through float64 FFTs (torch, on the device).
Tolerance: every output passes six (three) transforms whose sums hold at most
K = N/2 + 1 float32 products per folded half; a sum's rounding error is below
(K/4 + 4) u of the root sum of squares of its terms for the worst order and
about sqrt(K) u for random signs, so six passes at K <= 202 give about
6 * 14 * 2^-24 = 5e-6 relative to the output norm; the bar is 2e-5.
"""
import numpy as np
import pytest
import torch

import paper_2109_05339_amd as spfel
import synth
from oracle import geometry, nufft
from tests._common import DEV, f32, gpu, host
from tests._common import rel as rel_np

pytestmark = pytest.mark.gpu


def randn(seed, shape, real):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    x = torch.randn(shape, generator=g, device=DEV)
    return x if real else torch.complex(x, torch.randn(shape, generator=g, device=DEV))


def rel(a, b):
    a, b = a.to(torch.complex128), b.to(torch.complex128)
    return float((a - b).norm() / b.norm())


# (N, real, systems): 3 the smallest; 31/33/35 around one tile; 63..67 around
# two; 97 (three tiles on four wavefronts); 129/131 around four, with more
# systems than one group; 259 (nine tiles on eight wavefronts); 403 complex
# (unfused axis-0 pass)
@pytest.mark.parametrize("N,real,n", [
    (3, True, 2), (3, False, 1), (5, True, 1), (31, True, 2), (33, False, 2), (35, True, 3),
    (63, False, 1), (65, True, 2), (67, True, 1), (97, True, 1), (129, False, 3), (131, True, 6),
    (259, True, 1), (403, False, 1),
])
def test_normal_operator_against_float64_ffts(N, real, n):
    L, M = 2 * N, 2 * N - 1
    psf = randn(N, (M, M, M), real)      # no symmetry: every folded part counts
    v = randn(N + 1, (n, N, N, N), real)
    lams = [0.25 * (s + 1) * M ** 1.5 for s in range(n)]
    nm = spfel.Normal(N, domain=spfel.REAL if real else spfel.COMPLEX, max_systems=n, device=DEV)
    nm.set_psf(psf)
    y = nm.apply(v, lams)
    m = (torch.arange(M, device=DEV) - (N - 1)) % L
    big = torch.zeros((L, L, L), dtype=torch.complex128, device=DEV)
    big[m[:, None, None], m[None, :, None], m[None, None, :]] = psf.to(torch.complex128)
    big = torch.fft.fftn(big)
    for s in range(n):
        x = v[s].to(torch.complex128)
        e = 0.5 * (x + x.flip(0, 1, 2)) if real else x
        want = torch.fft.ifftn(torch.fft.fftn(e, s=(L, L, L)) * big)[:N, :N, :N]
        want = (want.real if real else want) + lams[s] * x
        assert rel(y[s], want) <= 2e-5, (s, rel(y[s], want))


def phase_step(rho, amp, seen, sup, beta):
    """One HIO step without positivity in float64, and its error."""
    F = torch.fft.fftn(rho.double())
    mag = F.abs()
    a = amp.double()
    d = seen.double()
    err = ((mag - a).square() * d).sum() / (a.square() * d).sum()
    G = torch.where(seen.bool(), a * F / mag, F)
    v = torch.fft.ifftn(G).real
    return torch.where(sup.bool(), v, rho.double() - beta * v), err


# even and odd lengths: 2 and 3 the smallest; around one, two, four and eight
# tiles of 16 rows; 602 (unfused axis-0 pass).  Amplitudes and mask have no
# symmetry, so a coefficient and its mirror image are told apart.
@pytest.mark.parametrize("N", [2, 3, 4, 7, 31, 32, 33, 34, 64, 65, 66, 100, 128, 129, 130, 258, 602])
def test_phase_step_against_float64_ffts(N):
    rho = randn(N, (N, N, N), True)
    amp = randn(N + 1, (N, N, N), True).abs() * N ** 1.5
    seen = (randn(N + 2, (N, N, N), True) > -0.7).to(torch.uint8)
    sup = (randn(N + 3, (N, N, N), True) > 0).to(torch.uint8)
    beta = 0.75
    want, err = phase_step(rho, amp, seen, sup, beta)
    got = rho.clone()
    p = spfel.Phase(N, device=DEV)
    e = p.iterate(got, amp, sup, 1, mode=spfel.PHASE_HIO, beta=beta, positivity=False, measured=seen,
                  errors=True)
    # a projected coefficient keeps its relative error unless |F| is small
    # against its rounding; 2e-5 covers six passes as above
    assert rel(got, want) <= 2e-5, rel(got, want)
    assert abs(float(e[0]) - float(err)) <= 1e-5 * float(err)
    # all coefficients measured
    want, err = phase_step(rho, amp, torch.ones_like(seen), sup, beta)
    got = rho.clone()
    e = p.iterate(got, amp, sup, 1, mode=spfel.PHASE_HIO, beta=beta, positivity=False, errors=True)
    assert rel(got, want) <= 2e-5, rel(got, want)
    assert abs(float(e[0]) - float(err)) <= 1e-5 * float(err)


# Model to fine grid (through slices) and fine grid to modes (through merges,
# twice into one output: the transform leaves the accumulator zeroed), against
# the oracle at the parity bar of the NUFFT tests; the model is not even.
@pytest.mark.parametrize("N", [5, 7, 31, 33, 35, 63, 65, 67])
@pytest.mark.parametrize("real", [True, False])
def test_grid_transforms_against_oracle(real, N):
    w = 4 if N < 9 else 6
    m = synth.random_model(3, N, complex_model=not real)
    m = m.astype(np.float32 if real else np.complex64)
    q = synth.quaternions(synth.config(4), "image_quats", 3).astype(np.float32)
    det = synth.detector_q(8).astype(np.float32)
    x = geometry.slice_points(f32(q), f32(det)).reshape(-1, 3)
    plan = spfel.Plan(N, kernel_width=w, domain=spfel.REAL if real else spfel.COMPLEX, device=DEV)
    dt = torch.float32 if real else torch.complex64
    plan.set_model(gpu(m, dt))
    s = host(plan.slice(gpu(q), gpu(det))[0]).reshape(-1)
    wide = m.astype(np.float64 if real else np.complex128)
    assert rel_np(s, nufft.nufft2(wide, x, w=w, real=real)) <= 1e-5
    g = np.random.default_rng(N)
    y = g.standard_normal((3, 64)).astype(np.float32)
    y = y if real else (y + 1j * g.standard_normal((3, 64))).astype(np.complex64)
    want = nufft.nufft1(y.astype(np.float64 if real else np.complex128).ravel(), x, N, w=w, real=real)
    out = plan.merge_adjoint(gpu(q), gpu(det), gpu(y, dt))
    assert rel_np(host(out), want) <= 1e-5
    plan.merge_adjoint(gpu(q), gpu(det), gpu(y, dt), out=out, flags=spfel.MERGE_ACCUMULATE)
    assert rel_np(host(out), 2 * want) <= 1e-5


@pytest.mark.parametrize("N", [3, 7, 33, 65, 131])
def test_normal_operator_takes_the_even_part_before_it_rounds(N):
    """REAL: A^T D A acts on the even part of a vector, so an odd one leaves
    lambda v alone, exactly; and a vector whose odd part is 1e4 times its even
    part is as accurate as any other (halved sums of opposite elements carry one
    rounding; the bar of the operator's test above)."""
    L, M = 2 * N, 2 * N - 1
    psf = randn(N, (M, M, M), True)
    w = randn(N + 1, (N, N, N), True)
    odd = w - w.flip(0, 1, 2)
    mixed = w + 1e4 * odd
    lam = 0.25 * M ** 1.5
    nm = spfel.Normal(N, max_systems=2, device=DEV)
    nm.set_psf(psf)
    y = nm.apply(torch.stack([odd, mixed]), [lam, 0.0])
    assert torch.equal(y[0], np.float32(lam) * odd)
    m = (torch.arange(M, device=DEV) - (N - 1)) % L
    big = torch.zeros((L, L, L), dtype=torch.complex128, device=DEV)
    big[m[:, None, None], m[None, :, None], m[None, None, :]] = psf.to(torch.complex128)
    x = mixed.double()
    e = 0.5 * (x + x.flip(0, 1, 2))
    want = torch.fft.ifftn(torch.fft.fftn(e, s=(L, L, L)) * torch.fft.fftn(big))[:N, :N, :N].real
    assert rel(y[1], want) <= 2e-5, rel(y[1], want)


def reduction_step(rho, amp, seen, sup):
    """One error reduction step without positivity in float64, and its error."""
    v, err = phase_step(rho, amp, seen, torch.ones_like(sup), 0.0)
    return torch.where(sup.bool(), v, torch.zeros_like(v)), err


# Error reduction runs on the line transforms (HIO on full tables): their cyclic
# form with one to nineteen tiles of 16 rows, more tiles than wavefronts from 258
# on, and at 602 the axis-0 passes and the projection apart.  Tolerances as above.
@pytest.mark.parametrize("N", [2, 3, 4, 7, 31, 32, 33, 34, 64, 65, 66, 100, 128, 129, 130, 258, 602])
def test_error_reduction_step_against_float64_ffts(N):
    rho = randn(N, (N, N, N), True)
    amp = randn(N + 1, (N, N, N), True).abs() * N ** 1.5
    seen = (randn(N + 2, (N, N, N), True) > -0.7).to(torch.uint8)
    sup = (randn(N + 3, (N, N, N), True) > 0).to(torch.uint8)
    p = spfel.Phase(N, device=DEV)
    for mask in (seen, None):   # None: all coefficients measured
        want, err = reduction_step(rho, amp, torch.ones_like(seen) if mask is None else mask, sup)
        got = rho.clone()
        e = p.iterate(got, amp, sup, 1, mode=spfel.PHASE_ER, positivity=False, measured=mask, errors=True)
        assert float(want.norm()) == 0 or rel(got, want) <= 2e-5, rel(got, want)
        assert abs(float(e[0]) - float(err)) <= 1e-5 * float(err)


@pytest.mark.parametrize("N", [7, 34, 65, 130])
def test_errors_of_a_burst_of_error_reduction_steps(N):
    """Each step's error is summed by the launch after its projection.  Error
    reduction does not amplify: five steps carry at most five times a step's
    bar, and the error, of order 1 here, twice that."""
    rho = randn(N, (N, N, N), True)
    amp = randn(N + 1, (N, N, N), True).abs() * N ** 1.5
    seen = (randn(N + 2, (N, N, N), True) > -0.7).to(torch.uint8)
    sup = (randn(N + 3, (N, N, N), True) > 0).to(torch.uint8)
    got, want, errs = rho.clone(), rho, []
    e = spfel.Phase(N, device=DEV).iterate(got, amp, sup, 5, mode=spfel.PHASE_ER, positivity=False,
                                           measured=seen, errors=True)
    for _ in range(5):
        want, err = reduction_step(want, amp, seen, sup)
        errs.append(float(err))
    assert rel(got, want) <= 1e-4, rel(got, want)
    assert np.all(np.abs(host(e) - errs) <= 2e-4 * np.array(errs))


def test_real_normal_operator_past_the_fused_pass():
    """REAL, N = 483: the axis-0 pass does not fit the LDS and runs as two line
    transforms with the product between them.  Sampled outputs against direct
    sums over the kernel, each with the bar of the sampled test at N = 129 (1e-5
    of the root of the sums of squares)."""
    N, M = 483, 965
    g = torch.Generator(device=DEV)
    g.manual_seed(N)
    psf = torch.randn((M, M, M), generator=g, device=DEV)
    v = torch.randn((1, N, N, N), generator=g, device=DEV)
    nm = spfel.Normal(N, max_systems=1, device=DEV)
    nm.set_psf(psf)
    y = nm.apply(v, [0.5])[0]
    ve = 0.5 * (v[0].double() + v[0].flip(0, 1, 2).double())
    for k in ((0, 0, 0), (N - 1, 3, 200), (241, 241, 241), (100, N - 1, N - 2), (17, 311, 0)):
        win = psf[k[0]:k[0] + N, k[1]:k[1] + N, k[2]:k[2] + N].flip(0, 1, 2).double()
        want = float((win * ve).sum()) + 0.5 * float(v[0][k])
        scale = float((win.square().sum() * ve.square().sum()).sqrt())
        assert abs(float(y[k]) - want) <= 1e-5 * scale, k
