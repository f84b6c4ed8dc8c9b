// Orientation matching (section II-B): every image against every model
// image, D[m, n] = |s_m|^2 + |d_n|^2 - 2 s_m . d_n, nearest model wins.
//
// The cross term is a GEMM S (M x P) . D^T (P x n_img) on the matrix cores;
// the M x n_img distance matrix is never stored: each 128 x 128 tile reduces
// its columns in registers/LDS and publishes one result per image.
//   FP32: v_mfma_f32_32x32x2_f32, per-tile column argmin, then a 64-bit
//         atomicMin of (order-preserving distance key << 32 | model index),
//         so the lowest index wins ties across tiles and across calls.
//   BF16: v_mfma_f32_32x32x16_bf16 with float32 accumulation on centred,
//         rounded operands, per-tile column top-8 of the proxy distance; a
//         second kernel merges the tiles' candidates per image, rescores in
//         float32 those whose lower bound can beat the running best, and
//         certifies that no other model image can; images it cannot
//         certify are matched again against every model image in float32.
#include <algorithm>

#include "device_common.h"
#include "internal.h"

namespace spfel {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int kBM = 128;   // model images per tile
constexpr int kBN = 128;   // images per tile
constexpr int kGroup = 8;  // m-tiles per launch-order group

// Tile of a block: blocks are dealt round-robin to the 8 XCDs, so the block
// id is first remapped to make each XCD's blocks a contiguous range, and
// that range is walked m-fastest in groups of `group` m-tiles, so the blocks
// resident on one XCD share slabs of S and D in that XCD's L2.
template <int group = kGroup>
__device__ inline void tile_of_block(int tiles_m, int tiles_n, int splits, int &tm, int &tn,
                                     int &split) {
  const int G = gridDim.x, bid = blockIdx.x;
  const int xcd = bid & 7, slot = bid >> 3, per = G >> 3, rem = G & 7;
  int v = (xcd < rem ? xcd * (per + 1) : rem * (per + 1) + (xcd - rem) * per) + slot;
  const int tiles = tiles_m * tiles_n;
  split = v / tiles;
  v -= split * tiles;
  const int gsize = group * tiles_n;
  const int g = v / gsize;
  const int first = g * group;
  const int gm = min(tiles_m - first, group);
  const int w = v - g * gsize;
  tm = first + w % gm;
  tn = w / gm;
}

// ---------------------------------------------------------------- FP32 ----
constexpr int kBK = 32;         // floats of P per K step
constexpr int kLdF = kBK + 4;   // LDS row stride (floats)

// Four consecutive values p[0..3] of a row, zero from the n-th on (n may be
// negative).  Whole quads take one load at whatever alignment the row has (odd
// row lengths, such as a detector behind a beam stop: four single loads
// instead of one took 2.3 times as long on 512 x 256 x 4,095).
__device__ inline float4 load_quad(const float *__restrict__ p, int n) {
  float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
  if (n >= 4) {
    __builtin_memcpy(&v, p, 16);
    return v;
  }
  v.x = n > 0 ? p[0] : 0.f;
  v.y = n > 1 ? p[1] : 0.f;
  v.z = n > 2 ? p[2] : 0.f;
  return v;
}

// Split-K: block (split, tile) covers K range [split kchunk, (split+1)
// kchunk) and stores its partial tile, row-major; reduce_f32_kernel adds the
// partials in split order and runs the epilogue.
//
// Tiles of T x T outputs by 4 T threads, wavefronts as 2 (M) x T / 32 (N).
// T = 128: each wavefront owns a 64 x 32 quarter-column (two 32x32 MFMA
// accumulators plus two per-K-step partials), which keeps the register count
// low enough for four wavefronts per SIMD.  T = 64, for launches that would
// leave CUs idle: one 32 x 32 accumulator a wavefront, and with few
// wavefronts to hide them the loads run four K steps ahead.  The sums of an
// output run over K in the same order either way.
template <int T>
__global__ __launch_bounds__(4 * T) __attribute__((amdgpu_waves_per_eu(T == 128 ? 4 : 1, 4))) void match_f32_kernel(
    const float *__restrict__ S, const float *__restrict__ D, const float *__restrict__ sn,
    const float *__restrict__ dn, int64_t M, int64_t N, int64_t P, uint32_t m_offset,
    unsigned long long *__restrict__ keys, int tiles_m, int tiles_n, int splits, int64_t kchunk,
    float *__restrict__ partials) {
  constexpr int kThreads = 4 * T, kI = T / 64, kAhead = T == 128 ? 1 : 4;
  // double-buffered A/B stages: one barrier per K step
  __shared__ __attribute__((aligned(16))) float As[2][T * kLdF];
  __shared__ __attribute__((aligned(16))) float Bs[2][T * kLdF];
  __shared__ float sns[T], dns[T];
  __shared__ unsigned long long red[2][T];

  int tm, tn, split;
  tile_of_block(tiles_m, tiles_n, splits, tm, tn, split);
  const int64_t row0 = (int64_t)tm * T, col0 = (int64_t)tn * T;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / (T / 32), wn = wave % (T / 32), lr = lane & 31, lh = lane >> 5;
  const int64_t kbeg = (int64_t)split * kchunk;
  const int64_t kend = min(P, kbeg + kchunk);

  // Rows past the last read the last one (their outputs are not used), so that
  // whole K steps load without a branch: with one, each step waited for its
  // own loads.
  float4 ra[kAhead][2], rb[kAhead][2];
  const float *pa[2], *pb[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int id = tid + kThreads * i, r = id >> 3, c = (id & 7) * 4;
    pa[i] = S + min(row0 + r, M - 1) * P + c;
    pb[i] = D + min(col0 + r, N - 1) * P + c;
  }
  const int whole = kend > kbeg ? (int)((kend - kbeg) / kBK) : 0;   // whole K steps
  auto gload = [&](int step, int set) {   // steps past the last whole one load that
    const int64_t k = kbeg + (int64_t)min(step, whole - 1) * kBK;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      __builtin_memcpy(&ra[set][i], pa[i] + k, 16);
      __builtin_memcpy(&rb[set][i], pb[i] + k, 16);
    }
  };

  floatx16 acc[kI];
#pragma unroll
  for (int i = 0; i < kI; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;

  auto lstore = [&](int buf, int set) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int id = tid + kThreads * i, r = id >> 3, c = (id & 7) * 4;
      *reinterpret_cast<float4 *>(&As[buf][r * kLdF + c]) = ra[set][i];
      *reinterpret_cast<float4 *>(&Bs[buf][r * kLdF + c]) = rb[set][i];
    }
  };
  auto multiply = [&](int buf) {
    // Fresh partial sums per K step keep every accumulation chain short:
    // at most 2 kBK roundings inside the step plus one per step.
    floatx16 part[kI];
#pragma unroll
    for (int i = 0; i < kI; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) part[i][r] = 0.f;
    const float *A = As[buf], *B = Bs[buf];
    // raised priority for the MFMA section (the other wavefronts' loads and
    // stores are served between its MFMAs, not ahead of them)
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int kk = 0; kk < kBK / 8; ++kk) {
      float4 a[kI];
#pragma unroll
      for (int i = 0; i < kI; ++i)
        a[i] = *reinterpret_cast<const float4 *>(&A[(wm * 32 * kI + i * 32 + lr) * kLdF + kk * 8 + lh * 4]);
      const float4 b = *reinterpret_cast<const float4 *>(&B[(wn * 32 + lr) * kLdF + kk * 8 + lh * 4]);
      // Lane half lh supplies k = 4 lh + e for MFMA e: A and B use the same
      // permutation of the 8 k values, so the sum is unchanged.
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < kI; ++i)
          part[i] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i][e], b[e], part[i], 0, 0, 0);
    }
    __builtin_amdgcn_s_setprio(0);
#pragma unroll
    for (int i = 0; i < kI; ++i) acc[i] += part[i];
  };
  // step s: products from stage s % 2, step s + 1 stored to the other.  Several
  // sets: loads of step s + kAhead into the set that step s was stored from
  // first.  One set (T = 128): the loads of step s + 2 go out as it is stored, so
  // they are on their way through the barrier and the next products as well.  Two
  // blocks on a CU start together and keep in step, and issued after the barrier
  // the loads of both fell together too: 2,301 x 2,299 x 4,096 (324 tiles) 567 us,
  // 526 here; 3,837 x 3,835 x 4,096 1,106 and 1,034.
  constexpr bool kOneSet = kAhead == 1;
  auto step = [&](int s, int u) {
    if constexpr (!kOneSet) gload(s + kAhead, u % kAhead);
    multiply(u & 1);
    lstore((u + 1) & 1, (u + 1) % kAhead);
    if constexpr (kOneSet) gload(s + 2, 0);
    __syncthreads();
  };
  constexpr int kU = kAhead > 2 ? kAhead : 2;
  if (whole > 0) {
#pragma unroll
    for (int d = 0; d < kAhead; ++d) gload(d, d);
    lstore(0, 0);
    if constexpr (kOneSet) gload(1, 0);
    __syncthreads();
    int s = 0;
    for (; s + kU <= whole; s += kU) {
#pragma unroll
      for (int u = 0; u < kU; ++u) step(s + u, u);
    }
#pragma unroll
    for (int u = 0; u < kU - 1; ++u)
      if (s + u < whole) step(s + u, u);
  }
  const int64_t k0 = kbeg + (int64_t)whole * kBK;
  if (k0 < kend) {   // the ragged step
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int c = ((tid + kThreads * i) & 7) * 4;
      ra[0][i] = load_quad(pa[i] + k0, (int)(kend - k0) - c);
      rb[0][i] = load_quad(pb[i] + k0, (int)(kend - k0) - c);
    }
    lstore(whole & 1, 0);
    __syncthreads();
    multiply(whole & 1);
    __syncthreads();
  }

  if (splits > 1) {
    float *mine = partials + ((int64_t)(tm * tiles_n + tn) * splits + split) * (T * T);
#pragma unroll
    for (int i = 0; i < kI; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        mine[(wm * 32 * kI + i * 32 + (r >> 2) * 8 + lh * 4 + (r & 3)) * T + wn * 32 + lr] = acc[i][r];
    return;
  }
  if (tid < T) {
    sns[tid] = row0 + tid < M ? sn[row0 + tid] : 0.f;
  } else if (tid < 2 * T) {
    const int c = tid - T;
    dns[c] = col0 + c < N ? dn[col0 + c] : 0.f;
  }
  __syncthreads();
  {
    const int cl = wn * 32 + lr;
    unsigned long long best = ~0ull;
#pragma unroll
    for (int i = 0; i < kI; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        // 32x32 MFMA output layout: lane holds column lane % 32 and rows
        // 8 (r / 4) + 4 (lane / 32) + r % 4.
        const int rl = wm * 32 * kI + i * 32 + (r >> 2) * 8 + lh * 4 + (r & 3);
        if (row0 + rl < M) {
          const float d = fmaf(-2.0f, acc[i][r], sns[rl] + dns[cl]);
          const unsigned long long key =
              ((unsigned long long)float_key(d) << 32) | (uint32_t)(m_offset + (uint32_t)(row0 + rl));
          best = key < best ? key : best;
        }
      }
    const unsigned long long o = __shfl_xor(best, 32);
    best = o < best ? o : best;
    if (lh == 0) red[wm][cl] = best;
  }
  __syncthreads();
  if (tid < T) {
    const unsigned long long a = red[0][tid], b = red[1][tid];
    const unsigned long long k = a < b ? a : b;
    if (col0 + tid < N && k != ~0ull) atomicMin(keys + col0 + tid, k);
  }
}

// Sum of element (row, col) of a tile's partials in split order.
template <int T = kBM>
__device__ inline float split_sum(const float *__restrict__ part, int splits, int row, int col) {
  const float *p = part + row * T + col;
  float v = 0.f;
#pragma unroll 4
  for (int sp = 0; sp < splits; ++sp) v += p[(int64_t)sp * (T * T)];
  return v;
}

// Epilogue of a split launch: a block takes 32 columns of a tile, a thread 16
// (tiles of 64: 8) rows of one of them.
constexpr int kRedCols = 32;

template <int T>
__global__ __launch_bounds__(256) void reduce_f32_kernel(
    const float *__restrict__ partials, int splits, const float *__restrict__ sn,
    const float *__restrict__ dn, int64_t M, int64_t N, uint32_t m_offset, int tiles_n,
    unsigned long long *__restrict__ keys) {
  constexpr int kRows = T / (256 / kRedCols);
  __shared__ unsigned long long red[256];
  const int tile = blockIdx.x / (T / kRedCols), c0 = (blockIdx.x % (T / kRedCols)) * kRedCols;
  const int col = c0 + (threadIdx.x & (kRedCols - 1)), rg = threadIdx.x / kRedCols;
  const int64_t row0 = (int64_t)(tile / tiles_n) * T, n = (int64_t)(tile % tiles_n) * T + col;
  const float *part = partials + (int64_t)tile * splits * (T * T);
  unsigned long long best = ~0ull;
  if (n < N) {
    const float dnn = dn[n];
#pragma unroll 4
    for (int j = 0; j < kRows; ++j) {
      const int row = rg * kRows + j;
      if (row0 + row >= M) break;
      const float d = fmaf(-2.0f, split_sum<T>(part, splits, row, col), sn[row0 + row] + dnn);
      const unsigned long long key =
          ((unsigned long long)float_key(d) << 32) | (uint32_t)(m_offset + (uint32_t)(row0 + row));
      best = key < best ? key : best;
    }
  }
  red[threadIdx.x] = best;
  __syncthreads();
  if (threadIdx.x < kRedCols && n < N) {
#pragma unroll
    for (int k = 1; k < 256 / kRedCols; ++k) {
      const unsigned long long o = red[threadIdx.x + k * kRedCols];
      best = o < best ? o : best;
    }
    if (best != ~0ull) atomicMin(keys + n, best);
  }
}

__global__ void pack_keys_kernel(const int32_t *__restrict__ idx, const float *__restrict__ dist,
                                 unsigned long long *__restrict__ keys, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) keys[i] = ((unsigned long long)float_key(dist[i]) << 32) | (uint32_t)idx[i];
}

__global__ void unpack_keys_kernel(const unsigned long long *__restrict__ keys,
                                   int32_t *__restrict__ idx, float *__restrict__ dist, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) {
    const unsigned long long k = keys[i];
    idx[i] = (int32_t)(uint32_t)(k & 0xffffffffu);
    dist[i] = key_float((uint32_t)(k >> 32));
  }
}

hipError_t launch_pack_keys(const int32_t *idx, const float *dist, unsigned long long *keys,
                            int64_t n, hipStream_t s) {
  hipLaunchKernelGGL(pack_keys_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, idx,
                     dist, keys, n);
  return hipGetLastError();
}

hipError_t launch_unpack_keys(const unsigned long long *keys, int32_t *idx, float *dist, int64_t n,
                              hipStream_t s) {
  hipLaunchKernelGGL(unpack_keys_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, keys,
                     idx, dist, n);
  return hipGetLastError();
}

static bool al16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

// Resident blocks of match_f32_kernel and match_bf16_kernel on the whole
// chip (256 CUs x 2).
constexpr int kSlots = 512;

static int64_t tiles_of(int64_t M, int64_t N, int T) { return ((M + T - 1) / T) * ((N + T - 1) / T); }

// K splits of an FP32 launch: the count up to four that best fills the chip's
// resident blocks with 128 x 128 tiles, each split at least 1024 values of P
// long.  Only launches of under half a round of tiles are split: blocks are
// dispatched dynamically, so a partial last round costs less than the
// partial tiles' extra traffic (1,264 tiles of K = 16,384: unsplit 5.21 ms,
// two splits 5.23).  The distances are differences of
// nearly equal sums, so their rounding shows the order of those: more splits,
// down to 512 values, moved distances of Poisson images by up to 3e-5 of
// themselves.
static int f32_splits(int64_t M, int64_t N, int64_t P) {
  const int64_t tiles = tiles_of(M, N, kBM);
  if (2 * tiles >= kSlots) return 1;
  int best = 1;
  double best_eff = 0.0;
  for (int s = 1; s <= 4; ++s) {
    if (s > 1 && P / s < 1024) break;
    const int64_t units = tiles * s;
    const int64_t rounds = (units + kSlots - 1) / kSlots;
    const double eff = (double)units / (double)(rounds * kSlots);
    if (eff > best_eff + 0.02) {
      best_eff = eff;
      best = s;
    }
  }
  return best;
}

// Blocks of 128 x 128 outputs for fewer than three quarters of the CUs: tiles
// of a quarter, four times as many blocks of half the matrix instructions per
// K step and wavefront.  Whole calls, 128- and 64-tiles: one block of 128
// (128 x 64 x 4,096) 279 and 100 us; 64 (1,000 x 256 x 4,096) 89 and 41; 128
// (1,000 x 512 x 4,096) 89 and 56; 192 (1,500 x 512 x 4,096) 91 and 93; 240
// (1,920 x 512 x 4,096) 91 and 95; 480 (2,560 x 768 x 4,096) 153 and 173.
static bool f32_small(int64_t M, int64_t N, int64_t P) {
  return tiles_of(M, N, kBM) * f32_splits(M, N, P) < kSlots * 3 / 8;
}

// Packed keys first.  A launch that splits K has its partial tiles at the
// offset below.  The word per 128 x 128 tile between the two is not used: it
// keeps the size that spfel_match_workspace_bytes has always given, which
// callers may have stored (tiles of 64 never need more).
static size_t f32_partials_at(int64_t M, int64_t N) {
  const size_t keys = ((size_t)N * sizeof(unsigned long long) + 255) & ~(size_t)255;
  return keys + (((size_t)tiles_of(M, N, kBM) * sizeof(unsigned) + 255) & ~(size_t)255);
}

size_t match_f32_workspace_bytes(int64_t M, int64_t N, int64_t P) {
  const int s = f32_splits(M, N, P);
  if (s == 1) return ((size_t)N * sizeof(unsigned long long) + 255) & ~(size_t)255;
  return f32_partials_at(M, N) + (size_t)tiles_of(M, N, kBM) * s * kBM * kBN * sizeof(float);
}

template <int T>
static hipError_t match_f32_go(const float *S, const float *D, const float *sn, const float *dn,
                               int64_t M, int64_t N, int64_t P, int64_t m_offset, int splits,
                               unsigned long long *keys, float *partials, hipStream_t s) {
  const int tiles_m = (int)((M + T - 1) / T), tiles_n = (int)((N + T - 1) / T);
  const int64_t tiles = (int64_t)tiles_m * tiles_n, blocks = tiles * splits;
  if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
  // K chunk: a multiple of the K step
  int64_t kchunk = (P + splits - 1) / splits;
  kchunk = (kchunk + kBK - 1) / kBK * kBK;
  hipLaunchKernelGGL((match_f32_kernel<T>), dim3((unsigned)blocks), dim3(4 * T), 0, s, S, D, sn, dn, M, N,
                     P, (uint32_t)m_offset, keys, tiles_m, tiles_n, splits, kchunk, partials);
  if (splits > 1)
    hipLaunchKernelGGL((reduce_f32_kernel<T>), dim3((unsigned)(tiles * (T / kRedCols))), dim3(256), 0, s,
                       partials, splits, sn, dn, M, N, (uint32_t)m_offset, tiles_n, keys);
  return hipGetLastError();
}

hipError_t launch_match_f32(const float *S, const float *D, const float *sn, const float *dn,
                            int64_t M, int64_t N, int64_t P, int64_t m_offset, void *workspace,
                            hipStream_t s) {
  char *ws = static_cast<char *>(workspace);
  auto *keys = reinterpret_cast<unsigned long long *>(ws);
  float *partials = reinterpret_cast<float *>(ws + f32_partials_at(M, N));
  const int splits = f32_splits(M, N, P);
  return f32_small(M, N, P) ? match_f32_go<64>(S, D, sn, dn, M, N, P, m_offset, splits, keys, partials, s)
                            : match_f32_go<kBM>(S, D, sn, dn, M, N, P, m_offset, splits, keys, partials, s);
}

// ---------------------------------------------------------------- BF16 ----
constexpr int kBKH = 64;          // bf16 values of P per K step
constexpr int kLdH = kBKH + 8;    // LDS row stride (bf16 values)

// Eight consecutive values p[0..7] of a row, zero from the n-th on (n may be
// negative); whole groups in one load at whatever alignment the row has.
__device__ inline uint4 load_oct(const uint16_t *__restrict__ p, int n) {
  uint4 v;
  if (n >= 8) {
    __builtin_memcpy(&v, p, 16);
    return v;
  }
  uint32_t h[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) h[e] = e < n ? p[e] : 0u;
  return make_uint4(h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), h[6] | (h[7] << 16));
}

// Sorted (ascending) insertion into a register top-8; branch free.
__device__ inline void insert8(uint32_t (&top)[8], uint32_t x) {
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    const uint32_t lo = min(top[s], x);
    x = max(top[s], x);
    top[s] = lo;
  }
}
__device__ inline void insert8(unsigned long long (&top)[8], unsigned long long x) {
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    const unsigned long long lo = top[s] < x ? top[s] : x;
    x = top[s] < x ? x : top[s];
    top[s] = lo;
  }
}

// The large-tile kernel needs rows of whole 64-wide K steps and 16-byte aligned
// operands; otherwise 128 x 128 tiles.  Its blocks run in rounds of 256 of equal
// length, of which a last one that is hardly filled is lost, and what its long
// prologue and epilogue cost weighs more the shorter the rows are.  Measured
// (whole calls, large tiles : 128 x 128):
//   several rounds, by the share of their blocks that is used:
//     P =    256  0.98  140 : 133 us (756 tiles)
//     P =  1,024  0.88  245 : 239 (900)    0.98  198 : 203 (756)
//     P =  1,600  0.78  239 : 226 (600)    0.85  241 : 242 (650)  0.95  244 : 259 (729)
//     P =  2,304  0.75  292 : 267 (576)    0.82  380 : 377 (840)  0.85  297 : 309 (650)
//     P =  4,096  0.75  438 : 416 (576)    0.78  441 : 449 (600)  0.85  444 : 485 (650)
//     P =  6,400  0.74  435 : 436 (380)    0.75  634 : 618 (576)  0.78  638 : 666 (600)
//     P = 16,384  0.60  1,018 : 987 (306)  0.67  1,040 : 1,082 (342)  0.69  1,557 : 1,615 (528)
//   one round:
//     144 tiles   P = 256 77 : 72   1,600 104 : 99   3,136 142 : 141   6,400 225 : 230
//     196 tiles   P = 256 78 : 81   1,600 104 : 117
int match_bf16_tile_rows(int64_t M, int64_t N, int64_t P, const void *S, const void *D) {
  if (P <= 0 || P % 64 != 0 || !al16(S) || !al16(D)) return 128;   // (their first K step is loaded unasked)
  const int64_t big = ((M + 255) / 256) * ((N + 255) / 256), rounds = (big + 255) / 256;
  if (rounds == 1) return big > (P >= 3072 ? 136 : 191) ? 256 : 128;
  const double used = (double)big / (256.0 * (double)rounds);
  return used >= (P >= 8192 ? 2.0 / 3.0 : 0.72 + 230.0 / (double)P) ? 256 : 128;
}

// Candidate buffer for the 128-row tiling, the larger of the two.
size_t match_bf16_candidate_bytes(int64_t M, int64_t N) {
  const int64_t tiles_m = (M + 127) / 128;
  return (size_t)tiles_m * (size_t)N * 8 * sizeof(uint32_t);
}

// Candidate word: proxy-distance key with its 7 low bits replaced by the
// row within the tile (a relative perturbation below 2^-15 of the proxy;
// clearing or setting those bits bounds the proxy from below or above).
//
// Tiles of 128 rows by BN images, four wavefronts: 2 x 2 of 64 x 64 (BN =
// 128), or 4 x 1 of 32 x 32 (BN = 32) for launches that would leave CUs idle,
// which have few wavefronts to hide their loads and run them four K steps
// ahead.
template <int BN>
__global__ __launch_bounds__(256, 2) void match_bf16_kernel(
    const uint16_t *__restrict__ S, const uint16_t *__restrict__ D, const float *__restrict__ sn,
    const float *__restrict__ dn, int64_t M, int64_t N, int64_t P, uint32_t *__restrict__ cand,
    int tiles_m, int tiles_n) {
  constexpr int kSeg = kBKH / 8;                                       // 16-byte segments per row and step
  constexpr int kA = kBM * kSeg / 256, kB = BN * kSeg / 256;           // segments per thread
  constexpr int kWaveN = BN == 128 ? 2 : 1, kWaveM = 4 / kWaveN;       // wavefronts of a tile
  constexpr int kI = kBM / kWaveM / 32, kJ = BN / kWaveN / 32;         // accumulators of a wavefront
  constexpr int kAhead = BN == 128 ? 1 : 4;
  __shared__ __attribute__((aligned(16))) uint16_t As[kBM * kLdH];
  __shared__ __attribute__((aligned(16))) uint16_t Bs[BN * kLdH];
  __shared__ float sns[kBM], dns[BN];
  __shared__ uint32_t red[kWaveM][BN][8];

  int tm, tn, split;
  tile_of_block(tiles_m, tiles_n, 1, tm, tn, split);
  const int64_t row0 = (int64_t)tm * kBM, col0 = (int64_t)tn * BN;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / kWaveN, wn = wave % kWaveN, lr = lane & 31, lh = lane >> 5;

  // rows past the last read the last one: their outputs are not used
  uint4 ra[kAhead][kA], rb[kAhead][kB];
  const uint16_t *pa[kA], *pb[kB];
  const int c = (tid % kSeg) * 8;
#pragma unroll
  for (int i = 0; i < kA; ++i) pa[i] = S + min(row0 + (tid + 256 * i) / kSeg, M - 1) * P + c;
#pragma unroll
  for (int i = 0; i < kB; ++i) pb[i] = D + min(col0 + (tid + 256 * i) / kSeg, N - 1) * P + c;
  const int whole = (int)(P / kBKH);   // whole K steps
  auto gload = [&](int step, int set) {   // steps past the last whole one load that
    const int64_t k = (int64_t)min(step, whole - 1) * kBKH;
#pragma unroll
    for (int i = 0; i < kA; ++i) __builtin_memcpy(&ra[set][i], pa[i] + k, 16);
#pragma unroll
    for (int i = 0; i < kB; ++i) __builtin_memcpy(&rb[set][i], pb[i] + k, 16);
  };
  auto lstore = [&](int set) {
#pragma unroll
    for (int i = 0; i < kA; ++i) *reinterpret_cast<uint4 *>(&As[(tid + 256 * i) / kSeg * kLdH + c]) = ra[set][i];
#pragma unroll
    for (int i = 0; i < kB; ++i) *reinterpret_cast<uint4 *>(&Bs[(tid + 256 * i) / kSeg * kLdH + c]) = rb[set][i];
  };

  floatx16 acc[kI][kJ];
#pragma unroll
  for (int i = 0; i < kI; ++i)
#pragma unroll
    for (int j = 0; j < kJ; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  auto multiply = [&]() {
#pragma unroll
    for (int kk = 0; kk < kBKH / 16; ++kk) {
      bf16x8 a[kI], b[kJ];
#pragma unroll
      for (int i = 0; i < kI; ++i)
        a[i] = *reinterpret_cast<const bf16x8 *>(&As[((wm * kI + i) * 32 + lr) * kLdH + kk * 16 + lh * 8]);
#pragma unroll
      for (int j = 0; j < kJ; ++j)
        b[j] = *reinterpret_cast<const bf16x8 *>(&Bs[((wn * kJ + j) * 32 + lr) * kLdH + kk * 16 + lh * 8]);
#pragma unroll
      for (int i = 0; i < kI; ++i)
#pragma unroll
        for (int j = 0; j < kJ; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
    }
  };
  auto step = [&](int s, int set) {
    __syncthreads();
    lstore(set);
    gload(s + kAhead, set);
    __syncthreads();
    multiply();
  };
  if (whole > 0) {
#pragma unroll
    for (int d = 0; d < kAhead; ++d) gload(d, d);
    int s = 0;
    for (; s + kAhead <= whole; s += kAhead) {
#pragma unroll
      for (int u = 0; u < kAhead; ++u) step(s + u, u);
    }
#pragma unroll
    for (int u = 0; u < kAhead - 1; ++u)
      if (s + u < whole) step(s + u, u);
  }
  if (P % kBKH) {   // the ragged step
    const int k0 = whole * kBKH, left = (int)(P - k0) - c;
#pragma unroll
    for (int i = 0; i < kA; ++i) ra[0][i] = load_oct(pa[i] + k0, left);
#pragma unroll
    for (int i = 0; i < kB; ++i) rb[0][i] = load_oct(pb[i] + k0, left);
    __syncthreads();
    lstore(0);
    __syncthreads();
    multiply();
  }

  if (tid < kBM) {
    sns[tid] = row0 + tid < M ? sn[row0 + tid] : 0.f;
  } else if (tid < kBM + BN) {
    const int cl = tid - kBM;
    dns[cl] = col0 + cl < N ? dn[col0 + cl] : 0.f;
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kJ; ++j) {
    const int cl = (wn * kJ + j) * 32 + lr;
    uint32_t top[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) top[s] = ~0u;
#pragma unroll
    for (int i = 0; i < kI; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int rl = (wm * kI + i) * 32 + (r >> 2) * 8 + lh * 4 + (r & 3);
        if (row0 + rl < M) {
          const float b = fmaf(-2.0f, acc[i][j][r], sns[rl] + dns[cl]);
          insert8(top, (float_key(b) & ~127u) | (uint32_t)rl);
        }
      }
    uint32_t other[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) other[s] = __shfl_xor(top[s], 32);
#pragma unroll
    for (int s = 0; s < 8; ++s) insert8(top, other[s]);
    if (lh == 0) {
#pragma unroll
      for (int s = 0; s < 8; ++s) red[wm][cl][s] = top[s];
    }
  }
  __syncthreads();
  if (tid < BN && col0 + tid < N) {
    uint32_t top[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) top[s] = red[0][tid][s];
#pragma unroll
    for (int w = 1; w < kWaveM; ++w)
#pragma unroll
      for (int s = 0; s < 8; ++s) insert8(top, red[w][tid][s]);
    uint4 *dst = reinterpret_cast<uint4 *>(cand + ((int64_t)tm * N + col0 + tid) * 8);
    dst[0] = make_uint4(top[0], top[1], top[2], top[3]);
    dst[1] = make_uint4(top[4], top[5], top[6], top[7]);
  }
}

// Large-tile form for launches with many tiles: 256 x 256 tiles, each of
// 8 wavefronts (two per SIMD) owning a 128 x 64 block (8 MFMA accumulators:
// 6 fragment reads per 8 MFMAs).  A and B stream from global memory straight
// into a double-buffered LDS ring (global_load_lds_dwordx4: each lane's 16
// bytes land at the instruction's LDS base + 16 x lane), one barrier per K
// step.  Rows are 128 bytes (64 bf16) without padding; the 16-byte chunk c
// of row r is stored at chunk c ^ f(r), f(r) = (r & 7) ^ ((r >> 3) & 1), so
// the 16 consecutive rows one fragment read touches fall in distinct bank
// groups.  Fragments are double-buffered in registers: the reads for the
// next 16-wide K slice are issued before the current slice's MFMAs.
// Requires P % 64 == 0 and 16-byte aligned rows; rows and columns past the
// matrix edge read the last row (their results are discarded).
constexpr int kBM2 = 256, kBN2 = 256, kBK2 = 64;
constexpr int kStage2 = (kBM2 + kBN2) * kBK2;   // bf16 values per LDS stage

__device__ inline int chunk_swizzle(int r) { return (r & 7) ^ ((r >> 3) & 1); }

// Tile of a block of the large-tile kernel.  When the tile grid is a whole
// number of 16 x 16 squares, each round of 256 resident blocks (one per CU)
// covers one square: XCD x takes an 8 x 4 part of it (x % 2 selects the 8
// m-tiles, x / 2 the 4 n-tiles), so a round reads 32 distinct tiles of S and
// D instead of 40, each m-tile shared by four XCDs and each n-tile by two.
// Other grids use the grouped order.
__device__ inline void big_tile_of_block(int tiles_m, int tiles_n, int &tm, int &tn) {
  if ((tiles_m & 15) == 0 && (tiles_n & 15) == 0) {
    const int bid = blockIdx.x, x = bid & 7, s = bid >> 3;
    const int r = s >> 5, w = s & 31;
    const int sq_m = tiles_m >> 4;
    const int rm = r % sq_m, rn = r / sq_m;
    tm = rm * 16 + (x & 1) * 8 + (w & 7);
    tn = rn * 16 + (x >> 1) * 4 + (w >> 3);
  } else {
    int split;
    tile_of_block(tiles_m, tiles_n, 1, tm, tn, split);
  }
}

__global__ __launch_bounds__(512, 1) void match_bf16_big_kernel(
    const uint16_t *__restrict__ S, const uint16_t *__restrict__ D, const float *__restrict__ sn,
    const float *__restrict__ dn, int64_t M, int64_t N, int64_t P, uint32_t *__restrict__ cand,
    int tiles_m, int tiles_n) {
  __shared__ __attribute__((aligned(16))) uint16_t smem[2 * kStage2];

  int tm, tn;
  big_tile_of_block(tiles_m, tiles_n, tm, tn);
  const int64_t row0 = (int64_t)tm * kBM2, col0 = (int64_t)tn * kBN2;
  // 8 wavefronts as 2 (M) x 4 (N), each owning a 128 x 64 block of the tile
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 2, wn = wave & 3, lr = lane & 31, lh = lane >> 5;

  // Loader: each wavefront moves 4 blocks of 8 rows of A and of B per K
  // step; block q's lane l carries row 8 q + l / 8, stored chunk l % 8,
  // which holds logical chunk (l % 8) ^ f(row).
  const uint16_t *srcA[4], *srcB[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int q = wave * 4 + i, r = q * 8 + (lane >> 3);
    const int lc = (lane & 7) ^ chunk_swizzle(r);
    const int64_t ga = min(row0 + r, M - 1), gb = min(col0 + r, N - 1);
    srcA[i] = S + ga * P + lc * 8;
    srcB[i] = D + gb * P + lc * 8;
  }
  auto issue = [&](int64_t k0, int buf) {
    uint16_t *As = smem + buf * kStage2;
    uint16_t *Bs = As + kBM2 * kBK2;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int q = wave * 4 + i;
      __builtin_amdgcn_global_load_lds(srcA[i] + k0, (__attribute__((address_space(3))) void *)(As + q * 512), 16, 0, 0);
      __builtin_amdgcn_global_load_lds(srcB[i] + k0, (__attribute__((address_space(3))) void *)(Bs + q * 512), 16, 0, 0);
    }
  };

  floatx16 acc[4][2];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  // fragment rows share lr's swizzle: logical chunk 2 kk + lh sits at
  // 2 (kk ^ (f >> 1)) + ((lh ^ f) & 1)
  const int fl = chunk_swizzle(lr), fhi = fl >> 1, flo = (lh ^ fl) & 1;
  const int arow = (wm * 128 + lr) * kBK2, brow = (wn * 64 + lr) * kBK2;
  bf16x8 fa[2][4], fb[2][2];
  auto frags = [&](const uint16_t *As, const uint16_t *Bs, int kk, int slot) {
    const int c = (2 * (kk ^ fhi) + flo) * 8;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      fa[slot][i] = *reinterpret_cast<const bf16x8 *>(&As[arow + i * 32 * kBK2 + c]);
#pragma unroll
    for (int j = 0; j < 2; ++j)
      fb[slot][j] = *reinterpret_cast<const bf16x8 *>(&Bs[brow + j * 32 * kBK2 + c]);
  };

  const int64_t steps = P / kBK2;
  auto multiply = [&](int slot) {
    // raised priority while issuing the MFMAs: the SIMD's other wavefront
    // is then served between them, not ahead of them
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[slot][i], fb[slot][j], acc[i][j], 0, 0, 0);
    __builtin_amdgcn_s_setprio(0);
    __builtin_amdgcn_sched_barrier(0);
  };
  issue(0, 0);
  __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): this wavefront's loads are in LDS
  __syncthreads();
  if (steps > 1) issue(kBK2, 1);
  frags(smem, smem + kBM2 * kBK2, 0, 0);
  __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0)
  for (int64_t st = 0; st < steps; ++st) {
    const uint16_t *As = smem + (st & 1) * kStage2;
    const uint16_t *Bs = As + kBM2 * kBK2;
#pragma unroll
    for (int kk = 0; kk < 3; ++kk) {
      // the scheduling barriers keep the next slice's reads ahead of this
      // slice's MFMAs (the compiler would otherwise sink them to save
      // registers and stall every MFMA group on a fresh LDS read)
      frags(As, Bs, kk + 1, (kk + 1) & 1);
      // LDS reads complete in order: this slice's 6 are in once at most
      // the next slice's 6 are outstanding
      __builtin_amdgcn_s_waitcnt(0xC67F);   // lgkmcnt(6), vmcnt/expcnt not waited
      multiply(kk & 1);
    }
    // This stage's last fragments are in registers and the next stage is in
    // LDS (vmcnt(0), lgkmcnt(0)) before the barrier; after it, the stage's
    // buffer is free for the step after next, and the next step's first
    // fragments are read ahead of this step's last MFMAs.
    __builtin_amdgcn_s_waitcnt(0x0070);
    __syncthreads();
    if (st + 2 < steps) issue((st + 2) * kBK2, (int)(st & 1));
    if (st + 1 < steps) {
      const uint16_t *An = smem + ((st + 1) & 1) * kStage2;
      frags(An, An + kBM2 * kBK2, 0, 0);
    }
    multiply(1);
  }
  __syncthreads();

  // Epilogue (LDS reused): norms of the tile's rows and columns, then each
  // column's 8 smallest proxies; candidate words carry the row in 8 bits.
  float *sns = reinterpret_cast<float *>(smem);
  float *dns = sns + kBM2;
  uint32_t *red = reinterpret_cast<uint32_t *>(dns + kBN2);   // [2][kBN2][8]
  if (tid < kBM2) sns[tid] = row0 + tid < M ? sn[row0 + tid] : 0.f;
  else dns[tid - kBM2] = col0 + tid - kBM2 < N ? dn[col0 + tid - kBM2] : 0.f;
  __syncthreads();
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int cl = wn * 64 + j * 32 + lr;
    uint32_t top[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) top[q] = ~0u;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int rl = wm * 128 + i * 32 + (r >> 2) * 8 + lh * 4 + (r & 3);
        if (row0 + rl < M) {
          const float b = fmaf(-2.0f, acc[i][j][r], sns[rl] + dns[cl]);
          insert8(top, (float_key(b) & ~255u) | (uint32_t)rl);
        }
      }
    uint32_t other[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) other[q] = __shfl_xor(top[q], 32);
#pragma unroll
    for (int q = 0; q < 8; ++q) insert8(top, other[q]);
    if (lh == 0) {
#pragma unroll
      for (int q = 0; q < 8; ++q) red[(wm * kBN2 + cl) * 8 + q] = top[q];
    }
  }
  __syncthreads();
  if (tid < kBN2 && col0 + tid < N) {
    uint32_t top[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) top[q] = red[tid * 8 + q];
#pragma unroll
    for (int q = 0; q < 8; ++q) insert8(top, red[(kBN2 + tid) * 8 + q]);
    uint4 *dst = reinterpret_cast<uint4 *>(cand + ((int64_t)tm * N + col0 + tid) * 8);
    dst[0] = make_uint4(top[0], top[1], top[2], top[3]);
    dst[1] = make_uint4(top[4], top[5], top[6], top[7]);
  }
}

// Tiles of 32 images instead of 128 up to this many 128 x 128 tiles (half a
// tile per CU).  Whole calls, 128 and 32 images: 1 tile (100 x 32 x 4,096) 92
// and 61 us; 2 (200 x 64 x 25,600) 329 and 176; 16 (1,000 x 256 x 4,096) 98
// and 66; 32 (1,000 x 512 x 10,089) 197 and 129; 128 (2,000 x 1,000 x 4,096)
// 100 and 86; 144 (1,500 x 1,500 x 4,096) 107 and 110; 240 (2,048 x 1,900 x
// 3,000) 98 and 125.
constexpr int64_t kNarrowTiles = 128;

template <int BN>
static hipError_t match_bf16_go(const uint16_t *S, const uint16_t *D, const float *sn, const float *dn,
                                int64_t M, int64_t N, int64_t P, uint32_t *cand, hipStream_t s) {
  const int tiles_m = (int)((M + kBM - 1) / kBM), tiles_n = (int)((N + BN - 1) / BN);
  const int64_t blocks = (int64_t)tiles_m * tiles_n;
  if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
  hipLaunchKernelGGL((match_bf16_kernel<BN>), dim3((unsigned)blocks), dim3(256), 0, s, S, D, sn, dn, M,
                     N, P, cand, tiles_m, tiles_n);
  return hipGetLastError();
}

hipError_t launch_match_bf16(const uint16_t *S, const uint16_t *D, const float *sn,
                             const float *dn, int64_t M, int64_t N, int64_t P, uint32_t *cand,
                             hipStream_t s) {
  if (match_bf16_tile_rows(M, N, P, S, D) == 256) {
    const int tiles_m = (int)((M + kBM2 - 1) / kBM2), tiles_n = (int)((N + kBN2 - 1) / kBN2);
    const int64_t blocks = (int64_t)tiles_m * tiles_n;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    hipLaunchKernelGGL(match_bf16_big_kernel, dim3((unsigned)blocks), dim3(512), 0, s, S, D, sn,
                       dn, M, N, P, cand, tiles_m, tiles_n);
    return hipGetLastError();
  }
  return tiles_of(M, N, kBM) <= kNarrowTiles ? match_bf16_go<32>(S, D, sn, dn, M, N, P, cand, s)
                                             : match_bf16_go<kBN>(S, D, sn, dn, M, N, P, cand, s);
}

// Bounds of the certified rescore (float32 arithmetic; every bound carries
// a relative margin of 2^-16, far above the few roundings in its formula).
//   proxy b~ = |s^|^2 + |d^|^2 - 2 s^.d^ with the dot product accumulated
//     on the matrix cores: each v_mfma_f32_32x32x16_bf16 is taken as a tree
//     of its 16 exact products plus the add to the accumulator, every
//     rounding at most 2^-23 relative (truncation allowed), so a product
//     meets at most P/16 + 8 roundings:
//       |s^.d^ computed - s^.d^| <= g_acc sum_p |s^_p d^_p| <= g_acc |s^| |d^|,
//     g_acc = gamma_{P/16+8} at u = 2^-23 (a probe of the instruction on
//     random, wide-exponent and cancelling inputs measured at most
//     3.2 x 2^-24 (|C| + sum |p|) per instruction).  The norms (float32
//     sums of P/256 + 8 roundings) and the epilogue's two roundings add at
//     most g_n (|s^| + |d^|)^2, g_n = gamma_{P/256+24} at u = 2^-24:
//       A = 2 g_acc |s^| |d^| + g_n (|s^| + |d^|)^2 >= |b~ - |s^ - d^|^2|;
//   true distance D = |s - d|^2:  |sqrt(D) - |s^ - d^|| <= e_m + f_n;
//   float32 rescore D~ of D (direct sum of (s - d)^2, chains of at most
//     P/64 + 16 roundings):  |D~ - D| <= g_run D.
struct CertBounds {
  float g_acc, g_n, g_run;
};
__device__ inline float proxy_slack(const CertBounds &cb, float ns, float nd) {
  return 2.0f * cb.g_acc * ns * nd + cb.g_n * (ns + nd) * (ns + nd);
}
constexpr float kLo = 1.0f - 0x1p-16f, kHi = 1.0f + 0x1p-16f;

__device__ inline float lower_sqrt_dist(float b_lo, float A, float ef) {
  return sqrtf(fmaxf(b_lo - A, 0.f)) * kLo - ef * kHi;
}
__device__ inline float upper_sqrt_dist(float b_hi, float A, float ef) {
  return sqrtf(fmaxf(b_hi, 0.f) + A) * kHi + ef * kHi;
}
// sqrt of the largest exact distance a float32 rescored value d can stand for
__device__ inline float upper_sqrt_rescored(float d, float g_run) {
  return sqrtf(d * (1.0f + 2.0f * g_run)) * kHi;
}

// Sum over p of (s_p - d_p)^2 for one lane's share of a row (float32): whole
// quads at whatever alignment the rows have, then the last P % 4 values.
__device__ inline float direct_part(const float *__restrict__ srow, const float *__restrict__ drow,
                                    int64_t P, int lane) {
  float acc = 0.f;
#pragma unroll 2
  for (int64_t q = lane; q < P / 4; q += 64) {
    float4 a, b;
    __builtin_memcpy(&a, srow + 4 * q, 16);
    __builtin_memcpy(&b, drow + 4 * q, 16);
    float t;
    t = a.x - b.x; acc = fmaf(t, t, acc);
    t = a.y - b.y; acc = fmaf(t, t, acc);
    t = a.z - b.z; acc = fmaf(t, t, acc);
    t = a.w - b.w; acc = fmaf(t, t, acc);
  }
  const int64_t p = (P & ~(int64_t)3) + lane;
  if (p < P) {
    const float t = srow[p] - drow[p];
    acc = fmaf(t, t, acc);
  }
  return acc;
}

__device__ inline float wave_sum(float v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  return v;
}

// Chunk maxima the certificate needs: max_m |s^_m| and max_m e_m; clears the
// fallback count.
__global__ __launch_bounds__(1024) void chunk_stats_kernel(const float *__restrict__ sn,
                                                           const float *__restrict__ se, int64_t M,
                                                           float *__restrict__ stats,
                                                           unsigned *__restrict__ count) {
  __shared__ float sh[2][1024];
  float a = 0.f, b = 0.f;
  for (int64_t m = threadIdx.x; m < M; m += 1024) {
    a = fmaxf(a, sqrtf(fmaxf(sn[m], 0.f)));
    b = fmaxf(b, se[m]);
  }
  sh[0][threadIdx.x] = a;
  sh[1][threadIdx.x] = b;
  __syncthreads();
  for (int st = 512; st > 0; st >>= 1) {
    if ((int)threadIdx.x < st) {
      sh[0][threadIdx.x] = fmaxf(sh[0][threadIdx.x], sh[0][threadIdx.x + st]);
      sh[1][threadIdx.x] = fmaxf(sh[1][threadIdx.x], sh[1][threadIdx.x + st]);
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    stats[0] = sh[0][0];
    stats[1] = sh[1][0];
    *count = 0u;
  }
}

// One wavefront per image:
//  1. merge every tile's 8 candidates into the image's 8 smallest proxies
//     (ties: lowest model index);
//  2. bound each candidate's true distance from below and above;
//  3. rescore in float32 (direct sum of squared differences) exactly the
//     candidates whose lower bound does not exceed both the running best
//     and the smallest upper bound among the 8 (no other candidate can be
//     the minimiser), and fold the best into (best_dist, best_idx);
//  4. certify the image: every model image outside the 8 has a true
//     distance at least the 8th proxy's lower bound (with the chunk's
//     largest norm and rounding error); if that bound does not exceed the
//     running best, the image goes on the fallback list (and flags[n] |= 1)
//     with its running best as the fallback's starting key.
__global__ __launch_bounds__(256) void rescore_kernel(
    const uint32_t *__restrict__ cand, int tiles_m, int tile_rows, int64_t M, int64_t N, int64_t P,
    uint32_t m_offset, const float *__restrict__ S32, const float *__restrict__ D32,
    const float *__restrict__ sn, const float *__restrict__ dn, const float *__restrict__ se,
    const float *__restrict__ de, const float *__restrict__ stats, CertBounds cb,
    int32_t *__restrict__ best_idx, float *__restrict__ best_dist, int32_t *__restrict__ flags,
    unsigned *__restrict__ fb_count, int32_t *__restrict__ fb_list,
    unsigned long long *__restrict__ fb_keys) {
  const int lane = threadIdx.x & 63;
  const int64_t n = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (n >= N) return;
  const uint32_t low = (uint32_t)tile_rows - 1u;
  unsigned long long top[8];
#pragma unroll
  for (int s = 0; s < 8; ++s) top[s] = ~0ull;
  const int total = tiles_m * 8;
  for (int c = lane; c < total; c += 64) {
    const int t = c >> 3, s = c & 7;
    const uint32_t k = cand[((int64_t)t * N + n) * 8 + s];
    if (k != ~0u) {
      const uint32_t m = (uint32_t)t * (uint32_t)tile_rows + (k & low);
      insert8(top, ((unsigned long long)(k & ~low) << 32) | m);
    }
  }
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    unsigned long long other[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) other[s] = __shfl_xor(top[s], off);
#pragma unroll
    for (int s = 0; s < 8; ++s) insert8(top, other[s]);
  }
  const float nd = sqrtf(fmaxf(dn[n], 0.f)), fd = de[n];
  int mi[8];
  bool valid[8];
  float lb[8];
  float ub_min = __builtin_inff();
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    valid[s] = top[s] != ~0ull;
    mi[s] = valid[s] ? (int)(uint32_t)(top[s] & 0xffffffffu) : 0;
    const uint32_t key = (uint32_t)(top[s] >> 32);
    const float ns = sqrtf(fmaxf(sn[mi[s]], 0.f));
    const float A = proxy_slack(cb, ns, nd);
    const float ef = se[mi[s]] + fd;
    lb[s] = lower_sqrt_dist(key_float(key), A, ef);
    if (valid[s]) ub_min = fminf(ub_min, upper_sqrt_dist(key_float(key | low), A, ef));
  }
  const float run = best_dist[n];
  const int32_t run_i = best_idx[n];
  const float thr = fminf(ub_min, upper_sqrt_rescored(run, cb.g_run));
  bool take[8];
  bool any = false;
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    take[s] = valid[s] && lb[s] <= thr;
    any = any || take[s];
  }
  unsigned long long best = ~0ull;
  if (any) {
    const float *drow = D32 + n * P;
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      if (take[s]) {   // wavefront-uniform
        const float d = wave_sum(direct_part(S32 + (int64_t)mi[s] * P, drow, P, lane));
        const unsigned long long key =
            ((unsigned long long)float_key(d) << 32) | (uint32_t)(m_offset + (uint32_t)mi[s]);
        best = key < best ? key : best;
      }
    }
  }
  const unsigned long long run_key = ((unsigned long long)float_key(run) << 32) | (uint32_t)run_i;
  const unsigned long long now = best < run_key ? best : run_key;
  // certificate: only needed when model images lie outside the 8
  bool cert = true;
  if (M > 8) {
    const float A8 = proxy_slack(cb, stats[0], nd);
    const float lb8 = lower_sqrt_dist(key_float((uint32_t)(top[7] >> 32)), A8, stats[1] + fd);
    cert = lb8 > upper_sqrt_rescored(key_float((uint32_t)(now >> 32)), cb.g_run);
  }
  if (lane == 0) {
    if (now != run_key) {
      best_idx[n] = (int32_t)(uint32_t)(now & 0xffffffffu);
      best_dist[n] = key_float((uint32_t)(now >> 32));
    }
    if (!cert) {
      if (flags) flags[n] |= 1;
      const unsigned pos = atomicAdd(fb_count, 1u);
      fb_list[pos] = (int32_t)n;
      fb_keys[pos] = now;
    }
  }
}

// Fallback for uncertified images: each work item is (listed image, slab of
// 64 model images); the block's four wavefronts rescore 16 rows each in
// float32 (direct sums, as in the rescore) and fold their minimum into the
// image's key with a 64-bit atomicMin (lowest index on ties).  The number
// of listed images is read on the device; every block leaves the loop when
// the work items run out (none when every image was certified).
__global__ __launch_bounds__(256) void fallback_kernel(
    const float *__restrict__ S32, const float *__restrict__ D32, int64_t M, int64_t P,
    uint32_t m_offset, const unsigned *__restrict__ fb_count, const int32_t *__restrict__ fb_list,
    unsigned long long *__restrict__ fb_keys) {
  __shared__ unsigned long long red[4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t slabs = (M + 63) / 64;
  const int64_t items = (int64_t)(*fb_count) * slabs;
  for (int64_t w = blockIdx.x; w < items; w += gridDim.x) {
    const int64_t pos = w / slabs, slab = w - pos * slabs;
    const int64_t n = fb_list[pos];
    const float *drow = D32 + n * P;
    unsigned long long best = ~0ull;
    for (int r = 0; r < 16; ++r) {
      const int64_t m = slab * 64 + wave * 16 + r;
      if (m >= M) break;   // wavefront-uniform
      const float d = wave_sum(direct_part(S32 + m * P, drow, P, lane));
      const unsigned long long key =
          ((unsigned long long)float_key(d) << 32) | (uint32_t)(m_offset + (uint32_t)m);
      best = key < best ? key : best;
    }
    if (lane == 0) red[wave] = best;
    __syncthreads();
    if (threadIdx.x == 0) {
      unsigned long long k = red[0];
#pragma unroll
      for (int i = 1; i < 4; ++i) k = red[i] < k ? red[i] : k;
      if (k != ~0ull) atomicMin(fb_keys + pos, k);
    }
    __syncthreads();
  }
}

__global__ __launch_bounds__(256) void fallback_unpack_kernel(
    const unsigned *__restrict__ fb_count, const int32_t *__restrict__ fb_list,
    const unsigned long long *__restrict__ fb_keys, int32_t *__restrict__ best_idx,
    float *__restrict__ best_dist) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (int64_t)(*fb_count)) return;
  const int32_t n = fb_list[i];
  const unsigned long long k = fb_keys[i];
  best_idx[n] = (int32_t)(uint32_t)(k & 0xffffffffu);
  best_dist[n] = key_float((uint32_t)(k >> 32));
}

static double gamma_of(double L, double u) { return L * u / (1.0 - L * u); }

size_t match_rescore_bytes(int64_t N) {
  // stats (2 floats) and the fallback count, then the list and the keys
  return 256 + (((size_t)N * 4 + 255) & ~(size_t)255) + (size_t)N * 8;
}

hipError_t launch_rescore(const uint32_t *cand, int tile_rows, int64_t M, int64_t N, int64_t P,
                          int64_t m_offset, const float *S32, const float *D32, const float *sn,
                          const float *dn, const float *se, const float *de, int32_t *best_idx,
                          float *best_dist, int32_t *flags, void *scratch, hipStream_t s) {
  const int tr = tile_rows;
  const int tiles_m = (int)((M + tr - 1) / tr);
  char *w = static_cast<char *>(scratch);
  float *stats = reinterpret_cast<float *>(w);
  unsigned *count = reinterpret_cast<unsigned *>(w + 16);
  int32_t *list = reinterpret_cast<int32_t *>(w + 256);
  auto *keys = reinterpret_cast<unsigned long long *>(w + 256 + (((size_t)N * 4 + 255) & ~(size_t)255));
  CertBounds cb;
  cb.g_acc = (float)gamma_of((double)(P / 16) + 8.0, 0x1p-23);
  cb.g_n = (float)gamma_of((double)(P / 256) + 24.0, 0x1p-24);
  cb.g_run = (float)gamma_of((double)(P / 64) + 16.0, 0x1p-24);
  hipLaunchKernelGGL(chunk_stats_kernel, dim3(1), dim3(1024), 0, s, sn, se, M, stats, count);
  hipLaunchKernelGGL(rescore_kernel, dim3((unsigned)((N + 3) / 4)), dim3(256), 0, s, cand, tiles_m,
                     tr, M, N, P, (uint32_t)m_offset, S32, D32, sn, dn, se, de, stats, cb, best_idx,
                     best_dist, flags, count, list, keys);
  hipLaunchKernelGGL(fallback_kernel, dim3(1024), dim3(256), 0, s, S32, D32, M, P,
                     (uint32_t)m_offset, count, list, keys);
  hipLaunchKernelGGL(fallback_unpack_kernel, dim3((unsigned)((N + 255) / 256)), dim3(256), 0, s,
                     count, list, keys, best_idx, best_dist);
  return hipGetLastError();
}

}  // namespace spfel
