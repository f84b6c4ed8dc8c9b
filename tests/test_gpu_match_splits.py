"""Matcher launches of few tiles (FP32: tiles of 64 and K split over blocks;
BF16: tiles of 32 images) and rows at every alignment (row lengths that are
not a multiple of 4 or 8), against the oracle's float64 distances.  Images are
Poisson counts of picked rows, so almost every image is decided; the distance
bounds are the documented chains (FP32: 36 + ceil(P/32) roundings of the
expanded form, BF16: P/64 + 16 of the direct sum)."""
import numpy as np
import pytest
import torch

import paper_2109_05339_amd as spfel
from oracle import match as om
from tests._common import DEV, gpu, host

pytestmark = pytest.mark.gpu


# one tile at 1 and at 128 rows and images, one past, P below the split length
# of 1,024 (unsplit), at and just past two splits, ragged by 1, 2 and 7, whole
# K steps that the splits do not divide evenly, a launch of 289 128-row tiles,
# and BF16 launches on both sides of the 256-row tiles' range (136, 144 and 306
# of them)
@pytest.mark.parametrize("M,N,P", [
    (1, 1, 1024), (3, 2, 1023), (128, 128, 1025), (129, 127, 1030), (257, 130, 5121),
    (300, 40, 8199), (64, 200, 16390), (40, 9, 511), (2100, 2050, 700), (300, 17400, 64), (4400, 1990, 64), (4100, 4400, 64),
])
@pytest.mark.parametrize("mode", [spfel.MATCH_FP32, spfel.MATCH_BF16_RESCORE8])
def test_split_and_ragged_launches(mode, M, N, P):
    g = np.random.default_rng(M + N + P)
    S = g.gamma(2.0, 15.0, (M, P)).astype(np.float32)
    D = g.poisson(S[g.integers(0, M, N)]).astype(np.float32)
    St, Dt = gpu(S), gpu(D)
    bi, bd = spfel.new_best(N, DEV)
    S64, D64 = S.astype(np.float64), D.astype(np.float64)
    ex = om.distances_expanded(S64, D64)
    cols = np.arange(N)
    if mode == spfel.MATCH_FP32:
        spfel.match(St, spfel.row_norm2(St), Dt, spfel.row_norm2(Dt), bi, bd)
        absdot = np.abs(S64) @ np.abs(D64).T
        E = om.fp32_distance_bound((S64 ** 2).sum(1)[:, None], (D64 ** 2).sum(1)[None, :], absdot,
                                   36 + -(-P // 32))
    else:
        im = spfel.ImagesBF16(Dt, centre=gpu(om.centre_rounded_mean(D)))
        spfel.match_bf16(St, im, bi, bd)
        E = 2 * om.gamma(P // 64 + 16) * ex + 1e-30
    bi, bd = host(bi), host(bd)
    am = om.argmin_first(ex)
    # images whose exact gap exceeds the bounds (all, but for very short rows)
    order = np.argpartition(ex, min(1, M - 1), axis=0) if M > 1 else np.zeros((2, N), int)
    second = np.where(order[0] == am, order[1], order[0]) if M > 1 else am
    decided = ex[second, cols] - ex[am, cols] > E[second, cols] + E[am, cols] if M > 1 else np.ones(N, bool)
    assert decided.mean() >= 0.99
    assert np.array_equal(bi[decided], am[decided])
    am = bi
    assert np.all(np.abs(bd - ex[am, cols]) <= E[am, cols])


@pytest.mark.parametrize("P", [31, 96, 700, 736])
def test_fp32_distances_do_not_depend_on_the_tile_size(P):
    """A launch of 2,100 x 2,050 runs in tiles of 128, its first 100 rows and 50
    images alone in tiles of 64: the same sums in the same order, so the same
    distances bit for bit (P with and without a ragged K step, and shorter than
    the four steps that the small tiles load ahead)."""
    g = np.random.default_rng(P)
    S = g.gamma(2.0, 15.0, (2100, P)).astype(np.float32)
    D = g.poisson(S[g.integers(0, 100, 2050)]).astype(np.float32)
    got = []
    for s, d in ((gpu(S), gpu(D)), (gpu(S[:100]), gpu(D[:50]))):
        best = spfel.new_best(len(d), DEV)
        spfel.match(s, spfel.row_norm2(s), d, spfel.row_norm2(d), *best)
        got.append([host(b) for b in best])
    same = got[0][0][:50] == got[1][0]   # a row past the first 100 may be nearer at short P
    assert same.mean() >= (0.9 if P >= 96 else 0.1)
    np.testing.assert_array_equal(got[0][1][:50][same], got[1][1][same])


@pytest.mark.parametrize("mode", [spfel.MATCH_FP32, spfel.MATCH_BF16_RESCORE8])
@pytest.mark.parametrize("M,N", [(3, 5), (300, 200), (1500, 1500), (3400, 3400)])
def test_rows_of_no_pixels(mode, M, N):
    """P = 0 through the C ABI (a tensor of no columns has no address): every
    distance is 0 and model image 0 the nearest, and no row is read, also where
    rows of whole K steps would go to the large tiles (3,400 x 3,400)."""
    none = torch.zeros(64, device=DEV)
    zm, zn = torch.zeros(M, device=DEV), torch.zeros(N, device=DEV)
    bi, bd = spfel.new_best(N, DEV)
    ws = torch.empty(spfel.match_workspace_bytes(M, N, 0, mode), dtype=torch.uint8, device=DEV)
    p = none.data_ptr()
    code = spfel.lib().spfel_match(p, zm.data_ptr(), p, zn.data_ptr(), M, N, 0, 0, mode, p, p, zm.data_ptr(),
                                   zn.data_ptr(), bi.data_ptr(), bd.data_ptr(), None, ws.data_ptr(), ws.numel(),
                                   torch.cuda.current_stream().cuda_stream)
    assert code == 0
    assert np.all(host(bi) == 0) and np.all(host(bd) == 0.0)


# BF16 launches on both sides of the rule for the 256-row tiles: one round of
# them (182 and 196 of short rows, 132 and 144 of long ones) and two rounds of
# which 0.87 and 0.95 are used, at a row length that needs 0.93
@pytest.mark.parametrize("M,N,P", [(3500, 3300, 64), (3500, 3500, 64), (3000, 2800, 3072), (3000, 3000, 3072),
                                   (5500, 5300, 1088), (5500, 5600, 1088)])
def test_sizes_of_the_large_tiles(M, N, P):
    test_split_and_ragged_launches(spfel.MATCH_BF16_RESCORE8, M, N, P)
