// Binned type-1 spreading over the registered detector (merging A*, section
// II-C Eq. (2)): every value y at a rotated Ewald-sphere point adds
// y psi psi psi to the w^3 fine-grid cells of its support.
//
// Points of many images are grouped by the fine-grid bin of their support
// origin, so that one block accumulates the stencils of thousands of
// points (from any image) into one brick before a single flush:
//   * bins: (H + 1 - w) x (17 - w) x (17 - w) support origins, each with an
//     H x 16 x 16 brick that holds every support cell of its points, H = 8
//     (16 at w = 8);
//   * pass 1 counts the points per bin, a scan turns the counts into offsets
//     and cuts the bins into subproblems, and pass 2 scatters each point's
//     value, kernel offsets and origin to a slot of its bin;
//   * one block per subproblem sorts its points in LDS by axis-1 origin; the
//     brick lives in registers as v_mfma_f32_16x16x4f32 accumulators, rows
//     (16 / H axis-1 planes x H cells of axis 0) by columns (16 cells of axis
//     2); four points per matrix step, each contributing (y psi0 psi1) (row)
//     times psi2 (column); only the tiles a group of points reaches are
//     stepped;
//   * the four wavefronts' bricks are summed in LDS in a fixed order and
//     added to the fine grid with one global atomic per nonzero cell.
//
// Two planes per tile: at w = 6 four points take three matrix instructions
// (four at odd origins) where 16 x 16 planes took six with 6 of 16 rows in
// use, for bins of a third of the origins.
#include <algorithm>
#include <type_traits>

#include "device_common.h"
#include "internal.h"

namespace spfel {

typedef float floatx4 __attribute__((ext_vector_type(4)));

// Brick cells of axis 0 and support origins of a bin along axis 0 and along
// axes 1 and 2.
constexpr int brick0(int w) { return w <= 7 ? 8 : 16; }
constexpr int origins0(int w) { return brick0(w) - w + 1; }
constexpr int origins12(int w) { return kBrick - w + 1; }

// Support origin (wrapped into [0, nf)) and kernel offsets of point q of
// the registered template under the scaled rotation Rs = R n_f / (2 pi)
// (the slicing kernels' coordinates, so both directions take the same
// support decisions).
template <int W>
__device__ inline bool point_support(const double *__restrict__ Rs, const double (&q)[3], int nf,
                                     int (&L)[3], float (&frac)[3]) {
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    // (explicit: the count and the scatter must round it alike)
    const double t = fma(Rs[3 * d + 2], q[2], fma(Rs[3 * d + 1], q[1], Rs[3 * d] * q[0]));
    if (!(fabs(t) < 1e8)) return false;
    const double c = ceil(t - 0.5 * W);
    frac[d] = (float)(t - c);
    // c mod nf (|c| < 1e8 + W fits an int); points within one period of
    // the grid take the conditional add only
    int ci = (int)c;
    ci += ci < 0 ? nf : 0;
    if ((unsigned)ci >= (unsigned)nf) {
      ci %= nf;
      ci += ci < 0 ? nf : 0;
    }
    L[d] = ci;
  }
  return true;
}

struct BinPoint {
  bool ok;
  int key, o0, o1, o2;
  float frac[3];
};

// Bin and origin in it of point q (template coordinates) under the scaled
// rotation Rs; nb: bins along axes 1 and 2.
template <int W>
__device__ inline BinPoint bin_point(const double *__restrict__ Rs, const double (&q)[3], bool inb, int nf,
                                     int nb) {
  BinPoint b;
  b.ok = false;
  b.key = b.o0 = b.o1 = b.o2 = 0;
  if (!inb || !(Rs[0] == Rs[0])) return b;
  int L[3];
  if (!point_support<W>(Rs, q, nf, L, b.frac)) return b;
  const int b0 = L[0] / origins0(W), b1 = L[1] / origins12(W), b2 = L[2] / origins12(W);
  b.o0 = L[0] - b0 * origins0(W);
  b.o1 = L[1] - b1 * origins12(W);
  b.o2 = L[2] - b2 * origins12(W);
  b.key = (b0 * nb + b1) * nb + b2;
  b.ok = true;
  return b;
}

// A binning block takes one tile of the registered template in kImages
// consecutive images.  Near the origin the images' tiles fall into the same
// few bins whatever their orientation, and the global atomics of one bin are
// served one after the other (about 20 million a second), so the block's
// points of a bin are counted in LDS first: one global atomic per block and
// bin instead of one per wavefront (which took 238 us instead of 88 for the
// count of 512 images of 128^2 pixels).
constexpr int kImages = 8;
constexpr int kHash = kImages * kTile;   // as many slots as points: never full

__device__ inline int table_slot(int *tkey, int key) {
  int h = (int)(((unsigned)key * 2654435761u) >> 21) & (kHash - 1);
  for (int probe = 0; probe < kHash; ++probe) {
    const int prev = atomicCAS(&tkey[h], -1, key);
    if (prev == -1 || prev == key) return h;
    h = (h + 1) & (kHash - 1);
  }
  return 0;   // unreachable: at most kHash distinct keys per block
}

// Adds the wavefront's points to the table, one lane per distinct bin (a
// wavefront's points are a compact patch and fall into one to a few bins).
// Returns this lane's slot and its rank among the block's points of the bin.
__device__ inline void table_add(int *tkey, int *tcnt, bool ok, int key, int &slot, int &rank) {
  const int lane = threadIdx.x & 63;
  unsigned long long left = __ballot(ok);
  while (left) {   // wavefront-uniform
    const int leader = __builtin_ctzll(left);
    const int k = __builtin_amdgcn_readlane(key, leader);
    const unsigned long long m = __ballot(ok && key == k);
    int h = 0, first = 0;
    if (lane == leader) {
      h = table_slot(tkey, k);
      first = atomicAdd(&tcnt[h], (int)__popcll(m));
    }
    h = __builtin_amdgcn_readlane(h, leader);
    first = __builtin_amdgcn_readlane(first, leader);
    if (ok && key == k) {
      slot = h;
      rank = first + (int)__popcll(m & ((1ull << lane) - 1));
    }
    left &= ~m;
  }
}

// The block's tile of the template: this thread's point.
__device__ inline bool tile_point(const float *__restrict__ dets, int64_t P, int tile, double (&q)[3]) {
  const int64_t i = (int64_t)tile * kTile + threadIdx.x;
  const bool inb = i < P;
#pragma unroll
  for (int d = 0; d < 3; ++d) q[d] = inb ? dets[3 * i + d] : 0.0;
  return inb;
}

// Pass 1: points per bin.
template <int W>
__global__ __launch_bounds__(kTile) void bin_count_kernel(
    const double *__restrict__ rot, int images, const float *__restrict__ dets, int64_t P, int tiles,
    int nf, int nb, int32_t *__restrict__ counts) {
  __shared__ int tkey[kHash], tcnt[kHash];
  const uint32_t vb = (uint32_t)xcd_contiguous_block();
  const int n0 = (int)(vb / tiles) * kImages, tile = (int)(vb % tiles);
  for (int e = threadIdx.x; e < kHash; e += kTile) {
    tkey[e] = -1;
    tcnt[e] = 0;
  }
  double q[3];
  const bool inb = tile_point(dets, P, tile, q);
  __syncthreads();
  for (int k = 0; k < kImages && n0 + k < images; ++k) {
    const BinPoint b = bin_point<W>(rot + 9 * (n0 + k), q, inb, nf, nb);
    int slot, rank;
    table_add(tkey, tcnt, b.ok, b.key, slot, rank);
  }
  __syncthreads();
  for (int e = threadIdx.x; e < kHash; e += kTile)
    if (tkey[e] >= 0) atomicAdd(&counts[tkey[e]], tcnt[e]);
}

// Pass 2: each point to its bin's next slot.  aux = (packed origin,
// imaginary value bits); REAL stores the packed origin alone, as an array
// of 32-bit words.
template <int W, bool CPLX>
__global__ __launch_bounds__(kTile) void bin_scatter_kernel(
    const double *__restrict__ rot, int images, int64_t first_image, const float *__restrict__ dets,
    const int32_t *__restrict__ perm, int64_t P, int tiles, int nf, int nb,
    const void *__restrict__ values, const float *__restrict__ weights,
    int32_t *__restrict__ cursor, float4 *__restrict__ pts, uint2 *__restrict__ aux) {
  __shared__ int tkey[kHash], tcnt[kHash];
  const uint32_t vb = (uint32_t)xcd_contiguous_block();
  const int n0 = (int)(vb / tiles) * kImages, tile = (int)(vb % tiles);
  for (int e = threadIdx.x; e < kHash; e += kTile) {
    tkey[e] = -1;
    tcnt[e] = 0;
  }
  double q[3];
  const bool inb = tile_point(dets, P, tile, q);
  const int64_t pixel = inb ? perm[(int64_t)tile * kTile + threadIdx.x] : 0;
  __syncthreads();
  BinPoint b[kImages];
  int slot[kImages], rank[kImages];
  float yr[kImages], yi[kImages], wt[kImages];
#pragma unroll
  for (int k = 0; k < kImages; ++k) {
    const bool in = inb && n0 + k < images;
    const int64_t o = (first_image + (in ? n0 + k : n0)) * P + pixel;
    yr[k] = yi[k] = 0.f;
    wt[k] = 1.f;
    if (in) {
      if (CPLX) {
        const float2 v = static_cast<const float2 *>(values)[o];
        yr[k] = v.x;
        yi[k] = v.y;
      } else {
        yr[k] = static_cast<const float *>(values)[o];
      }
      if (weights) wt[k] = weights[o];
    }
  }
#pragma unroll
  for (int k = 0; k < kImages; ++k) {
    slot[k] = -1;
    rank[k] = 0;
    b[k].ok = false;
    if (n0 + k < images) {   // block-uniform
      b[k] = bin_point<W>(rot + 9 * (n0 + k), q, inb, nf, nb);
      table_add(tkey, tcnt, b[k].ok, b[k].key, slot[k], rank[k]);
    }
  }
  __syncthreads();
  for (int e = threadIdx.x; e < kHash; e += kTile)
    if (tkey[e] >= 0) tcnt[e] = atomicAdd(&cursor[tkey[e]], tcnt[e]);
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kImages; ++k) {
    if (!b[k].ok) continue;
    const int pos = tcnt[slot[k]] + rank[k];
    if (weights) {
      yr[k] *= wt[k];
      yi[k] *= wt[k];
    }
    pts[pos] = make_float4(yr[k], b[k].frac[0], b[k].frac[1], b[k].frac[2]);
    const uint32_t packed = (uint32_t)(b[k].o0 | (b[k].o1 << 4) | (b[k].o2 << 8));
    if (CPLX)
      aux[pos] = make_uint2(packed, __float_as_uint(yi[k]));
    else
      reinterpret_cast<uint32_t *>(aux)[pos] = packed;   // REAL: one word per point
  }
}

// Scan of the bins' counts in two launches.  bin_scan_kernel: each block sums
// kScanBins bins' points and subproblems (runs of at most `cap` points).
// bin_offsets_kernel: each block adds the sums of the blocks before it, and
// writes its bins' scatter cursors and subproblems (in bin order) and clears
// their counts for the next batch; the last block writes the number of
// subproblems.
constexpr int kScanThreads = 256, kScanBins = 4 * kScanThreads;

// Exclusive sums of s over the block's threads; `all` receives the total.
__device__ inline int2 block_scan(int2 s, int2 *wsum, int2 &all) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int2 inc = s;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int x = __shfl_up(inc.x, off), y = __shfl_up(inc.y, off);
    if (lane >= off) {
      inc.x += x;
      inc.y += y;
    }
  }
  if (lane == 63) wsum[wave] = inc;
  __syncthreads();
  int2 run = make_int2(inc.x - s.x, inc.y - s.y);
  all = make_int2(0, 0);
#pragma unroll
  for (int w = 0; w < kScanThreads / 64; ++w) {
    if (w < wave) {
      run.x += wsum[w].x;
      run.y += wsum[w].y;
    }
    all.x += wsum[w].x;
    all.y += wsum[w].y;
  }
  __syncthreads();
  return run;
}

__global__ __launch_bounds__(kScanThreads) void bin_scan_kernel(const int32_t *__restrict__ counts, int nbins,
                                                                int cap, int2 *__restrict__ sums) {
  __shared__ int2 wsum[kScanThreads / 64];
  int2 s = make_int2(0, 0), all;
  for (int k = threadIdx.x; k < kScanBins; k += kScanThreads) {
    const int bin = (int)blockIdx.x * kScanBins + k;
    const int c = bin < nbins ? counts[bin] : 0;
    s.x += c;
    s.y += (c + cap - 1) / cap;
  }
  block_scan(s, wsum, all);
  if (threadIdx.x == 0) sums[blockIdx.x] = all;
}

__global__ __launch_bounds__(kScanThreads) void bin_offsets_kernel(
    int32_t *__restrict__ counts, int nbins, int cap, const int2 *__restrict__ sums,
    int32_t *__restrict__ cursor, int4 *__restrict__ sub, int32_t *__restrict__ nsub) {
  __shared__ int2 wsum[kScanThreads / 64];
  int2 before = make_int2(0, 0), base, all;
  for (int k = threadIdx.x; k < (int)blockIdx.x; k += kScanThreads) {
    before.x += sums[k].x;
    before.y += sums[k].y;
  }
  block_scan(before, wsum, base);
  const int bin0 = (int)blockIdx.x * kScanBins + (int)threadIdx.x * 4;
  int c[4], q[4];
  int2 s = make_int2(0, 0);
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    c[k] = bin0 + k < nbins ? counts[bin0 + k] : 0;
    q[k] = (c[k] + cap - 1) / cap;
    s.x += c[k];
    s.y += q[k];
  }
  int2 run = block_scan(s, wsum, all);
  run.x += base.x;
  run.y += base.y;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if (bin0 + k < nbins) {
      cursor[bin0 + k] = run.x;
      if (c[k]) counts[bin0 + k] = 0;
      for (int j = 0; j < q[k]; ++j)
        sub[run.y + j] = make_int4(bin0 + k, run.x + j * cap, min(run.x + c[k], run.x + (j + 1) * cap), 0);
    }
    run.x += c[k];
    run.y += q[k];
  }
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) *nsub = base.y + all.y;
}

// One block per subproblem.  The points are sorted by axis-1 origin v; each wavefront takes a quarter of
// them, 64 at a time: its lanes turn the points into weight rows in the
// wavefront's own LDS rows, then it steps its accumulators over them, four
// points per matrix step, with the tiles of planes v .. v + w - 1 chosen at
// compile time (one code path per v).  One wavefront's transcendental weights
// overlap another's matrix steps.
//
// What bounds it (REAL, w = 6, 2,048 images of 256^2 pixels on the 258^3 grid:
// 4.64 ms by one plane per tile, 3.67 ms here, 36e9 points/s): the matrix
// instructions take 1.64 ms at the 2.2 GHz held, the vector instructions (430
// per 64 points, 36 of them transcendental) about as long, and the two
// overlap only across the three wavefronts of a SIMD (4.4 ms with two), which
// the staged rows in LDS limit.
//
// LDS words of a staged point: y psi0 over the brick's H cells (COMPLEX:
// psi0 alone), psi1 three times as the matrix steps read it, psi2 over the 16
// cells (COMPLEX: then y).  psi1 of the planes of tile t (H = 8), for the
// lanes of the tile's first and second plane: v even psi1[2 t], psi1[2 t + 1];
// v odd psi1[2 t - 1], psi1[2 t].  Row pitches are 4 or 12 modulo 32, so the
// lanes' 16-byte row writes fall in distinct banks.
template <int W, bool CPLX>
struct Row {
  static constexpr int H = brick0(W), kPlanes = 16 / H;
  static constexpr int k1 = H, k1Words = H == 8 ? 12 : 8;      // psi1
  static constexpr int k2 = k1 + k1Words;                      // psi2
  static constexpr int kY = k2 + 16;
  static constexpr int kPitch = CPLX ? 44 : H == 8 ? 36 : 44;
  static_assert(kY + (CPLX ? 2 : 0) <= kPitch, "row");
};
constexpr int64_t kSpreadGrid = 16 * 768;   // blocks of a launch at most (768 fit the chip at once)
constexpr int kStaged = 64 + 4;   // rows per wavefront: a step reads up to three rows past the last point

template <int W, bool CPLX>
__global__ __launch_bounds__(256, CPLX && W == 8 ? 1 : CPLX || W == 8 ? 2 : 3) void spread_binned_kernel(
    float *__restrict__ grid, int nf, float beta, int nb, const float4 *__restrict__ pts,
    const uint2 *__restrict__ aux, const int4 *__restrict__ sub, const int32_t *__restrict__ nsub) {
  typedef Row<W, CPLX> R;
  constexpr int H = R::H, kPlanes = R::kPlanes, kRow = R::kPitch;
  constexpr int Bo = origins12(W);
  constexpr int kT = 16 / kPlanes;         // accumulator tiles
  constexpr int kA = CPLX ? 2 : 1;
  constexpr int kCap = sub_cap(CPLX), kPer = kCap / 256;
  __shared__ __attribute__((aligned(16))) float rows[4][kStaged][kRow];
  __shared__ uint32_t order[kCap];         // sorted points: index in the subproblem | packed origin << 16
  __shared__ int colOff[Bo + 1];
  const int tid = threadIdx.x, lane = tid & 63;
  const int total = *nsub;
  // (a bounded grid walks over the subproblems: their number is known on the
  // device alone, and its bound on the host counts every bin)
  for (int sb = blockIdx.x; sb < total; sb += gridDim.x) {
    const int4 sp = sub[sb];
    const int bin = sp.x, start = sp.y, count = sp.z - sp.y;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i = lane & 15, g = lane >> 4;

    // ---- sort by axis-1 origin: one LDS atomic per point gives its rank ----
    if (tid <= Bo) colOff[tid] = 0;
    for (int k = lane; k < 4 * kRow; k += 64) rows[wave][64 + k / kRow][k % kRow] = 0.f;
    __syncthreads();
    {
      uint32_t packed[kPer];
      int rank[kPer];
  #pragma unroll
      for (int k = 0; k < kPer; ++k) {
        const int p = tid + 256 * k;
        packed[k] = 0;
        if (p < count) packed[k] = CPLX ? aux[start + p].x : reinterpret_cast<const uint32_t *>(aux)[start + p];
      }
  #pragma unroll
      for (int k = 0; k < kPer; ++k) {
        rank[k] = 0;
        if (tid + 256 * k < count) rank[k] = atomicAdd(&colOff[1 + ((packed[k] >> 4) & 15)], 1);
      }
      __syncthreads();
      if (tid == 0) {
        int run = 0;
  #pragma unroll
        for (int v = 1; v <= Bo; ++v) {
          run += colOff[v];
          colOff[v] = run;
        }
      }
      __syncthreads();
  #pragma unroll
      for (int k = 0; k < kPer; ++k) {
        const int p = tid + 256 * k;
        if (p < count) order[colOff[(packed[k] >> 4) & 15] + rank[k]] = (uint32_t)p | (packed[k] << 16);
      }
    }
    __syncthreads();

    // ---- this wavefront's quarter of the sorted points ----
    const int per = ((count + 255) / 256) * 64;   // whole batches of 64
    const int wb = min(count, wave * per), we = min(count, wb + per);
    floatx4 acc[kT], acci[CPLX ? kT : 1];
  #pragma unroll
    for (int t = 0; t < kT; ++t) {
      acc[t] = floatx4{0.f, 0.f, 0.f, 0.f};
      if (CPLX) acci[CPLX ? t : 0] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
    // matrix-step reads: lane (i, g) takes point p + g's psi0 at cell i % H,
    // psi1 of its plane in every tile and psi2 at cell i
    const float *const rd = &rows[wave][g][0];
    const float *const rd0 = rd + (i & (H - 1)), *const rd2 = rd + R::k2 + i;
    const float *const rdEven = rd + R::k1 + (H == 8 ? 4 * (i >> 3) : 0);         // P, Q
    const float *const rdOdd = rd + R::k1 + (H == 8 ? (i >> 3 ? 0 : 8) : 0);      // R, P
    struct Step {
      float a, c;
      float4 b0, b1;   // psi1 by tile
      float2 y;
    };
    // steps points [p, end) of the wavefront's rows; their axis-1 origin is V
    auto run = [&](auto vc, int p, int end) {
      constexpr int V = decltype(vc)::value;
      constexpr bool odd = H == 8 && (V & 1);
      constexpr int t0 = V / kPlanes;
      constexpr int nt = H == 8 ? (odd ? (W + 2) / 2 : (W + 1) / 2) : W;   // tiles reached
      const float *const rd1 = odd ? rdOdd : rdEven;
      auto fetch = [&](int at) {
        Step s;
        s.a = rd0[at * kRow];
        s.c = rd2[at * kRow];
        s.b0 = *reinterpret_cast<const float4 *>(rd1 + at * kRow);
        if (nt > 4) s.b1 = *reinterpret_cast<const float4 *>(rd1 + 4 + at * kRow);
        if (CPLX) s.y = *reinterpret_cast<const float2 *>(rd + R::kY + at * kRow);
        return s;
      };
      auto step = [&](const Step &s, bool use) {   // use: this lane's point is one of [p, end)
        const float cr = use ? (CPLX ? s.c * s.y.x : s.c) : 0.f;
        const float ci = CPLX && use ? s.c * s.y.y : 0.f;
        const float b[8] = {s.b0.x, s.b0.y, s.b0.z, s.b0.w, s.b1.x, s.b1.y, s.b1.z, s.b1.w};
  #pragma unroll
        for (int t = 0; t < nt; ++t) {
          if (t0 + t >= kT) continue;
          const float ab = use ? s.a * b[t] : 0.f;
          acc[t0 + t] = __builtin_amdgcn_mfma_f32_16x16x4f32(ab, cr, acc[t0 + t], 0, 0, 0);
          if (CPLX)
            acci[CPLX ? t0 + t : 0] =
                __builtin_amdgcn_mfma_f32_16x16x4f32(ab, ci, acci[CPLX ? t0 + t : 0], 0, 0, 0);
        }
      };
      // Two steps a turn over two register sets: the next step's rows are read
      // while this one's matrix instructions run (vector and matrix
      // instructions of a SIMD's wavefronts hardly overlap, so moves and address
      // arithmetic in this loop cost what they take)
      Step x = fetch(p), z;
      for (; p + 8 <= end; p += 8) {
        z = fetch(p + 4);
        __builtin_amdgcn_sched_barrier(0);
        step(x, true);
        __builtin_amdgcn_sched_barrier(0);
        x = fetch(min(p + 8, 64));   // rows 64 .. 67 are zero
        __builtin_amdgcn_sched_barrier(0);
        step(z, true);
        __builtin_amdgcn_sched_barrier(0);
      }
      if (p < end) {
        z = fetch(min(p + 4, 64));
        step(x, p + g < end);
        if (p + 4 < end) step(z, p + 4 + g < end);
      }
    };

    uint32_t ent = 0u;
    float4 pv = make_float4(0.f, 0.f, 0.f, 0.f);
    float pyi = 0.f;
    auto load_batch = [&](int b0) {
      if (b0 + lane < we) {
        ent = order[b0 + lane];
        pv = pts[start + (ent & 0xffffu)];
        if (CPLX) pyi = __uint_as_float(aux[start + (ent & 0xffffu)].y);
      }
    };
    load_batch(wb);
    for (int b0 = wb; b0 < we; b0 += 64) {
      const int cnt = min(64, we - b0);
      const float4 v = pv;
      const float yi = pyi;
      const uint32_t en = ent;
      load_batch(b0 + 64);   // the next batch's points are on their way during this one
      __builtin_amdgcn_wave_barrier();
      {
        float *const row = rows[wave][lane];
        float4 *const row4 = reinterpret_cast<float4 *>(row);
        const float4 z = make_float4(0.f, 0.f, 0.f, 0.f);
  #pragma unroll
        for (int q = 0; q < H / 4; ++q) row4[q] = z;
  #pragma unroll
        for (int q = 0; q < 4; ++q) row4[R::k2 / 4 + q] = z;
        float w1[8] = {};
        if (lane < cnt) {
          float w0[W], t1[W], w2[W];
          es_weights<W>(v.y, beta, w0);
          es_weights<W>(v.z, beta, t1);
          es_weights<W>(v.w, beta, w2);
          const int o0 = (en >> 16) & 15, o2 = (en >> 24) & 15;
  #pragma unroll
          for (int a = 0; a < W; ++a) {
            row[o0 + a] = CPLX ? w0[a] : v.x * w0[a];
            row[R::k2 + o2 + a] = w2[a];
            w1[a] = t1[a];
          }
        }
        if (H == 8) {
          row4[R::k1 / 4] = make_float4(w1[0], w1[2], w1[4], w1[6]);
          row4[R::k1 / 4 + 1] = make_float4(w1[1], w1[3], w1[5], w1[7]);
          row4[R::k1 / 4 + 2] = make_float4(0.f, w1[1], w1[3], w1[5]);
        } else {
          row4[R::k1 / 4] = make_float4(w1[0], w1[1], w1[2], w1[3]);
          row4[R::k1 / 4 + 1] = make_float4(w1[4], w1[5], w1[6], w1[7]);
        }
        if (CPLX) *reinterpret_cast<float2 *>(row + R::kY) = make_float2(v.x, yi);
      }
      __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0): this wavefront's rows are written
      __builtin_amdgcn_wave_barrier();
      for (int p = 0; p < cnt;) {   // the batch's origins in turn
        const int o1 = (__builtin_amdgcn_readlane((int)en, p) >> 20) & 15;
        const int end = min(cnt, __builtin_amdgcn_readfirstlane(colOff[o1 + 1]) - b0);
        switch (o1) {
          case 0: run(std::integral_constant<int, 0>{}, p, end); break;
          case 1: run(std::integral_constant<int, 1>{}, p, end); break;
          case 2: run(std::integral_constant<int, 2>{}, p, end); break;
          case 3: run(std::integral_constant<int, 3>{}, p, end); break;
          case 4: run(std::integral_constant<int, 4>{}, p, end); break;
          case 5: run(std::integral_constant<int, 5>{}, p, end); break;
          case 6: run(std::integral_constant<int, 6>{}, p, end); break;
          case 7: run(std::integral_constant<int, 7>{}, p, end); break;
          case 8: run(std::integral_constant<int, 8>{}, p, end); break;
          case 9: run(std::integral_constant<int, (Bo > 9 ? 9 : 0)>{}, p, end); break;
          case 10: run(std::integral_constant<int, (Bo > 10 ? 10 : 0)>{}, p, end); break;
          case 11: run(std::integral_constant<int, (Bo > 11 ? 11 : 0)>{}, p, end); break;
          default: run(std::integral_constant<int, (Bo > 12 ? 12 : 0)>{}, p, end); break;
        }
        p = end;
      }
    }
    // Sum the four wavefronts' bricks in LDS (each its own copy, added in
    // order), then flush.  Result lane layout: lane (i, g) holds rows 4 g + r
    // of a tile (axis-0 cell row % H of plane row / H), column i (axis 2).
    __syncthreads();
    constexpr int kCells = H * 16 * 16, kRed = 4 * kStaged * kRow / kCells / kA;   // copies that fit
    static_assert(kRed >= 1, "reduction buffer");
    float *const red = &rows[0][0][0];
    for (int w0 = 0; w0 < 4; w0 += kRed) {
      if (wave >= w0 && wave < w0 + kRed) {
        float *const mine = red + (wave - w0) * kCells * kA;
  #pragma unroll
        for (int t = 0; t < kT; ++t)
  #pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int row = 4 * g + r;
            const int c = ((row & (H - 1)) * 16 + t * kPlanes + row / H) * 16 + i;
            // the first copy keeps the sum of the copies before it
            const bool add = w0 > 0 && wave == w0;
            mine[kA * c] = add ? mine[kA * c] + acc[t][r] : acc[t][r];
            if (CPLX)
              mine[kA * c + 1] = add ? mine[kA * c + 1] + acci[CPLX ? t : 0][r] : acci[CPLX ? t : 0][r];
          }
      }
      __syncthreads();
      if (w0 + kRed < 4) {   // more to come: the copies into the first
        for (int c = tid; c < kCells * kA; c += 256) {
          float v = red[c];
  #pragma unroll
          for (int k = 1; k < kRed; ++k) v += red[k * kCells * kA + c];
          red[c] = v;
        }
        __syncthreads();
      }
    }
    constexpr int kLast = 4 % kRed == 0 ? kRed : 4 % kRed;   // copies of the last round
    const int bb2 = bin % nb, bb1 = (bin / nb) % nb, bb0 = bin / (nb * nb);
    const int lo0 = bb0 * origins0(W), lo1 = bb1 * Bo, lo2 = bb2 * Bo;
    for (int c = tid; c < kCells; c += 256) {
      float vr = red[kA * c], vi = CPLX ? red[kA * c + 1] : 0.f;
  #pragma unroll
      for (int k = 1; k < kLast; ++k) {
        vr += red[k * kCells * kA + kA * c];
        if (CPLX) vi += red[k * kCells * kA + kA * c + 1];
      }
      if (vr == 0.f && vi == 0.f) continue;
      const int i2 = c & 15, i1 = (c >> 4) & 15, i0 = c >> 8;
      // lo < nf and i < 16: one subtraction wraps unless the grid is
      // smaller than a brick
      int g0 = lo0 + i0, g1 = lo1 + i1, g2 = lo2 + i2;
      if (g0 >= nf) g0 = nf >= kBrick ? g0 - nf : g0 % nf;
      if (g1 >= nf) g1 = nf >= kBrick ? g1 - nf : g1 % nf;
      if (g2 >= nf) g2 = nf >= kBrick ? g2 - nf : g2 % nf;
      const int64_t cell = ((int64_t)g0 * nf + g1) * nf + g2;
      if (CPLX) {
        if (vr != 0.f) unsafeAtomicAdd(grid + 2 * cell, vr);
        if (vi != 0.f) unsafeAtomicAdd(grid + 2 * cell + 1, vi);
      } else {
        unsafeAtomicAdd(grid + cell, vr);
      }
    }
    __syncthreads();   // LDS is free for the next subproblem
  }
}

size_t bin_count(int nf, int w) {
  const size_t nb0 = (nf + origins0(w) - 1) / origins0(w), nb = (nf + origins12(w) - 1) / origins12(w);
  return nb0 * nb * nb;
}

size_t bin_scan_blocks(int nf, int w) { return (bin_count(nf, w) + kScanBins - 1) / kScanBins; }

// Points per subproblem for a batch: whole subproblems of sub_cap points where
// the batch gives the chip a thousand of them, smaller ones down to 256 points
// otherwise.
static int batch_cap(bool cplx, int64_t points) {
  const int64_t even = (points / 1024 + 255) / 256 * 256;
  return (int)std::min<int64_t>(sub_cap(cplx), std::max<int64_t>(256, even));
}

size_t bin_max_subproblems(int nf, int w, bool cplx, int64_t points) {
  return (size_t)(points / batch_cap(cplx, points)) + bin_count(nf, w) + 1;
}

template <int W, bool CPLX>
static hipError_t spread_binned_wc(const Plan &pl, const float *quats, int64_t n_img, int64_t P,
                                   const void *values, const float *weights, hipStream_t s) {
  const int nf = pl.nf;
  const int nb = (nf + origins12(W) - 1) / origins12(W);
  const int nbins = (int)bin_count(nf, W);
  const int scans = (int)bin_scan_blocks(nf, W);
  const int tiles = (int)((P + kTile - 1) / kTile);
  // A single batch is binned and spread on the caller's stream.  With more,
  // batch b is binned on the plan's stream into buffer set b % 2 and spread
  // on the caller's stream from it, so the binning of batch b + 1 (memory
  // and atomics) runs beside the spread of batch b (matrix cores).  The
  // plan's stream starts after the caller's work so far; every spread waits
  // for its batch's binning, and the binning of batch b + 2 for the spread of
  // batch b, which also orders all of it before the caller's later work.
  const bool two = n_img > pl.bin_batch;
  hipStream_t bs = two ? pl.bin_stream : s;
  hipError_t e = hipSuccess;
  const bool recorded = capturing(s);
  if (recorded) pl.bin_zero = false;
  if (two) {
    e = hipEventRecord(pl.ev_bin_start, s);
    if (e == hipSuccess) e = hipStreamWaitEvent(bs, pl.ev_bin_start, 0);
    if (e != hipSuccess) return e;
  }
  int64_t b = 0;
  for (int64_t n0 = 0; n0 < n_img; n0 += pl.bin_batch, ++b) {
    const int k = (int)(b & 1);
    const int64_t nbat = std::min<int64_t>(pl.bin_batch, n_img - n0);
    const int64_t blocks = (nbat + kImages - 1) / kImages * tiles;
    const int cap = batch_cap(CPLX, nbat * P);
    if (b >= 2) {
      e = hipStreamWaitEvent(bs, pl.ev_spread[k], 0);
      if (e != hipSuccess) return e;
    }
    e = launch_rotations(quats + 4 * n0, nbat, (double)nf / (2.0 * M_PI), pl.rot, bs);
    if (e == hipSuccess && !pl.bin_zero) e = launch_fill_zero(pl.bin_cnt, (size_t)nbins * 4, bs);
    if (e != hipSuccess) return e;
    pl.bin_zero = false;
    hipLaunchKernelGGL((bin_count_kernel<W>), dim3((unsigned)blocks), dim3(kTile), 0, bs, pl.rot,
                       (int)nbat, pl.det_sorted, P, tiles, nf, nb, pl.bin_cnt);
    hipLaunchKernelGGL(bin_scan_kernel, dim3((unsigned)scans), dim3(kScanThreads), 0, bs, pl.bin_cnt,
                       nbins, cap, pl.bin_sums);
    hipLaunchKernelGGL(bin_offsets_kernel, dim3((unsigned)scans), dim3(kScanThreads), 0, bs, pl.bin_cnt,
                       nbins, cap, pl.bin_sums, pl.bin_cur, pl.bin_sub[k], pl.bin_nsub[k]);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    pl.bin_zero = true;
    hipLaunchKernelGGL((bin_scatter_kernel<W, CPLX>), dim3((unsigned)blocks), dim3(kTile), 0, bs,
                       pl.rot, (int)nbat, n0, pl.det_sorted, pl.det_perm, P, tiles, nf, nb, values,
                       weights, pl.bin_cur, pl.bin_pts[k], pl.bin_aux[k]);
    e = hipGetLastError();
    if (two) {
      if (e == hipSuccess) e = hipEventRecord(pl.ev_binned[k], bs);
      if (e == hipSuccess) e = hipStreamWaitEvent(s, pl.ev_binned[k], 0);
    }
    if (e != hipSuccess) return e;
    const int64_t grid = std::min<int64_t>((int64_t)bin_max_subproblems(nf, W, CPLX, nbat * P), kSpreadGrid);
    hipLaunchKernelGGL((spread_binned_kernel<W, CPLX>), dim3((unsigned)grid), dim3(256), 0, s,
                       static_cast<float *>(pl.acc), nf, (float)pl.beta, nb, pl.bin_pts[k],
                       pl.bin_aux[k], pl.bin_sub[k], pl.bin_nsub[k]);
    e = hipGetLastError();
    if (e == hipSuccess && two) e = hipEventRecord(pl.ev_spread[k], s);
    if (e != hipSuccess) return e;
  }
  if (recorded) pl.bin_zero = false;
  return hipSuccess;
}

template <int W>
static hipError_t spread_binned_w(const Plan &pl, const float *quats, int64_t n_img, int64_t P,
                                  const void *values, const float *weights, hipStream_t s) {
  return pl.domain == SPFEL_COMPLEX
             ? spread_binned_wc<W, true>(pl, quats, n_img, P, values, weights, s)
             : spread_binned_wc<W, false>(pl, quats, n_img, P, values, weights, s);
}

hipError_t launch_spread_binned(const Plan &pl, const float *quats, int64_t n_img, int64_t P,
                                const void *values, const float *weights, hipStream_t s) {
  switch (pl.w) {
    case 4: return spread_binned_w<4>(pl, quats, n_img, P, values, weights, s);
    case 5: return spread_binned_w<5>(pl, quats, n_img, P, values, weights, s);
    case 6: return spread_binned_w<6>(pl, quats, n_img, P, values, weights, s);
    case 7: return spread_binned_w<7>(pl, quats, n_img, P, values, weights, s);
    default: return spread_binned_w<8>(pl, quats, n_img, P, values, weights, s);
  }
}

}  // namespace spfel
