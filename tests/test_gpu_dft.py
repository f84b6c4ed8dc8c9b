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
from tests._common import DEV

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
