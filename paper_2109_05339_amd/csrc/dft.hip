// Line transforms of the separable 3D DFTs: one axis of a 3D transform,
// every line of the array at once, as real matrix products on the matrix
// cores.
//
// A complex DFT of a line by its full table costs four real multiply-adds
// per (input, output) pair.  Cosine and sine have definite parity, so the
// inputs are first folded into sums E and differences O of the elements x_p
// and x_-p, and the outputs y_q and y_-q unfolded from one cosine sum and one
// sine sum:
//   C_q = sum_p E_p cos(q p),  S_q = sum_p O_p sin(q p),  y_+-q = C_q +- i S_q
// (a quarter of the multiply-adds, for any length, prime ones among them).
// Between 2H grid cells and modes (H odd) a second folding, of the cells l
// and H - l, splits the sums by the parity of the mode and halves them
// again.  What is real, what is Hermitian and what is only needed in its
// real part carries one real product instead of two.
//
// One block takes 16 lines (columns): it reads every element of its lines
// once, folds them into LDS, and each wavefront forms row tiles of 16 outputs
// with v_mfma_f32_16x16x4f32, the table read in operand order (one 8-byte
// load per lane and step, shared by all blocks through L2).  The folded
// products leave the passes bound by the traffic of the lines themselves,
// so neighbouring passes are fused where a block already holds whole lines:
// the middle (axis 0) pass of a convolution runs forward transform, product
// and inverse transform on lines that never leave the CU.
//
// Measured on an application of the normal equations (N = 129, L = 258, 8
// REAL systems): 7.1 ms by full complex tables (42% of the FP32 matrix rate
// on eleven times the products), 0.74 ms here: axis-0 pass 325 us, axis 1
// 108 and 110 us (415 MB each, 3.8 TB/s), axis 2 92 us (73 before it read the
// opposite lines too) and 101 us.  One error reduction at N = 129: 329 us by
// full tables and full spectra, 70 us here (axis-0 pass with the projection 26
// us, the others 11 to 13 us each, half of it matrix instructions).  The merge's
// transform at N = 129: 515 us plus a 17 us clear of the accumulator by full
// tables, 79 us here.
//
// Lane layout of the instruction: lane t supplies A[t % 16][t / 16] and
// B[t / 16][t % 16] and receives D[4 (t / 16) + j][t % 16], j = 0..3.
#include <algorithm>
#include <cmath>
#include <vector>

#include "device_common.h"
#include "internal.h"

namespace spfel {

typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int kCol = 16;            // lines per block
constexpr int kPitch = kCol + 1;    // LDS row pitch (vectors): lanes along a line or across lines
                                    // both fall in distinct banks
constexpr int kMaxWaves = 8;
constexpr size_t kLdsMax = 160 * 1024;
// A fused pass keeps its prefetched inputs in registers: at most kMaxItems
// slots per thread (slots <= 16 tiles + 8, 64 threads per tile).
constexpr int kMaxItems = 5;

struct Geo {   // what a kernel needs of a table
  const float2 *t;
  int h, H, even_slots, slots, even_tiles, tiles;
};
static Geo geo_of(const DftTable &tab) {
  return {tab.t, tab.h, tab.H, tab.even_slots, tab.slots, tab.even_tiles, tab.tiles};
}

// ------------------------------------------------------------ folding ----
// LDS vectors: complex forms hold (Re E, Im E, Re O, Im O); the real forms
// (kRH, kCRe, kHR) hold the one real number of E and of O that their sums
// need.
template <bool CPLX>
struct Vec;
template <>
struct Vec<true> {
  typedef float4 T;
};
template <>
struct Vec<false> {
  typedef float2 T;
};

// One input pair (x, y): E = x + y and O = x - y in the form's parts.  An
// input that is its own partner comes with y = 0: E = x, and its O meets a
// zero of the sine table.
template <int IO>
__device__ inline typename Vec<IO == kCC>::T fold(float2 x, float2 y) {
  if constexpr (IO == kCC) {
    return make_float4(x.x + y.x, x.y + y.y, x.x - y.x, x.y - y.y);
  } else if constexpr (IO == kRH) {
    return make_float2(x.x + y.x, x.x - y.x);
  } else {   // kCRe: the sums of the real output's parts
    return make_float2(x.x + y.x, x.y - y.y);
  }
}
// A Hermitian pair (x, conj x): E = 2 Re x, O = 2 i Im x (its imaginary
// part); by itself E = Re x.
__device__ inline float2 fold_half(float2 x, bool self) {
  return make_float2(self ? x.x : 2.f * x.x, 2.f * x.y);
}

__device__ inline float4 vadd(float4 a, float4 b, float so) {   // E + E', O + so O'
  return make_float4(a.x + b.x, a.y + b.y, fmaf(so, b.z, a.z), fmaf(so, b.w, a.w));
}
__device__ inline float2 vadd(float2 a, float2 b, float so) { return make_float2(a.x + b.x, fmaf(so, b.y, a.y)); }
__device__ inline float4 vsub(float4 a, float4 b, float so) {   // E - E', O + so O'
  return make_float4(a.x - b.x, a.y - b.y, fmaf(so, b.z, a.z), fmaf(so, b.w, a.w));
}
__device__ inline float2 vsub(float2 a, float2 b, float so) { return make_float2(a.x - b.x, fmaf(so, b.y, a.y)); }

// Element offsets are 32-bit (the launchers refuse larger arrays).
template <int IO>
__device__ inline float2 load_at(const void *in, uint32_t o) {
  if constexpr (IO == kRH)
    return make_float2(static_cast<const float *>(in)[o], 0.f);
  else
    return static_cast<const float2 *>(in)[o];
}

// The elements of one input slot as loaded: kToGrid and kCyclic x_p, x_-p;
// kToModes cells l, H - l, L - l, H + l.
template <int KIND>
struct Raw {
  float2 x[KIND == kToModes ? 4 : 2];
};

// Loads slot `slot` of the line at `in` + base (elements `st` apart).  Slots
// past the line's last pair, and lines that are not `ok` (their base is that
// of some line), give zeros: the addresses are clamped and the values
// selected, so that the loads of several slots go out together.
template <int KIND, int IO>
__device__ inline Raw<KIND> load_slot(const Geo &g, const void *in, uint32_t base, uint32_t st, int slot,
                                      bool ok) {
  Raw<KIND> r;
  auto get = [&](int e, bool keep) {
    const float2 v = load_at<IO>(in, base + (uint32_t)e * st);
    return make_float2(keep ? v.x : 0.f, keep ? v.y : 0.f);
  };
  if constexpr (KIND == kToGrid) {
    const int k0 = slot < g.even_slots ? 2 * slot : 2 * (slot - g.even_slots) + 1;
    const int k = min(k0, g.h);
    const bool in_line = ok && k0 <= g.h;
    r.x[0] = get(g.h + k, in_line);
    r.x[1] = get(g.h - k, in_line && k > 0);
  } else if constexpr (KIND == kToModes) {
    const int H = g.H, l = min(slot, H / 2);
    const bool in_line = ok && 2 * slot <= H;
    r.x[0] = get(l, in_line);
    r.x[1] = get(H - l, in_line);
    if constexpr (IO == kHR) {
      r.x[2] = r.x[3] = make_float2(0.f, 0.f);
    } else {
      r.x[2] = get(l > 0 ? 2 * H - l : 0, in_line && l > 0);
      r.x[3] = get(H + l, in_line && l > 0);
    }
  } else {
    const int n = g.H, p = min(slot, n / 2);
    const bool in_line = ok && 2 * slot <= n;
    r.x[0] = get(p, in_line);
    if constexpr (IO == kHR)
      r.x[1] = make_float2(0.f, 0.f);
    else
      r.x[1] = get(p > 0 ? n - p : 0, in_line && p > 0 && 2 * p < n);
  }
  return r;
}

// The same slot of the even part of a real 3D array (kToGrid, axis 2): `mirror`
// is where the line of the opposite modes of the other axes starts.  Halved
// sums of opposite elements, formed before anything is rounded: an odd array
// gives zeros.
__device__ inline Raw<kToGrid> load_even_slot(const Geo &g, const void *in, uint32_t base, uint32_t mirror,
                                              int slot, bool ok) {
  const Raw<kToGrid> a = load_slot<kToGrid, kRH>(g, in, base, 1, slot, ok);
  const Raw<kToGrid> b = load_slot<kToGrid, kRH>(g, in, mirror, 1, slot, ok);
  const bool zero = slot == 0;   // mode 0 is its own opposite: b.x[1] is not loaded
  Raw<kToGrid> r;
  r.x[0] = make_float2(0.5f * (a.x[0].x + (zero ? b.x[0].x : b.x[1].x)), 0.f);
  r.x[1] = make_float2(zero ? 0.f : 0.5f * (a.x[1].x + b.x[0].x), 0.f);
  return r;
}

// Folds a loaded slot into its vector(s) of V.
template <int KIND, int IO>
__device__ inline void fold_slot(const Geo &g, const Raw<KIND> &r, int slot, int col,
                                 typename Vec<IO == kCC>::T *V) {
  typedef typename Vec<IO == kCC>::T T;
  if constexpr (KIND == kToModes) {
    T p, q;
    if constexpr (IO == kHR) {
      p = fold_half(r.x[0], slot == 0);
      q = fold_half(r.x[1], slot == 0);
    } else {
      p = fold<IO>(r.x[0], r.x[2]);
      q = fold<IO>(r.x[1], r.x[3]);
    }
    V[slot * kPitch + col] = vadd(p, q, -1.f);   // cell H - l: cos (-1)^k, sin -(-1)^k of cell l's
    V[(g.slots + slot) * kPitch + col] = vsub(p, q, 1.f);
  } else if constexpr (IO == kHR) {
    V[slot * kPitch + col] = fold_half(r.x[0], slot == 0 || 2 * slot == g.H);
  } else {
    V[slot * kPitch + col] = fold<IO>(r.x[0], r.x[1]);
  }
}

// Where a column's elements start.
__device__ inline uint32_t col_base(uint32_t c, uint32_t B, int len) {
  const uint32_t a = c / B;
  return a * (uint32_t)len * B + (c - a * B);
}

// ----------------------------------------------------------- products ----
template <bool CPLX, bool SWAP>
__device__ inline void product(float2 cs, typename Vec<CPLX>::T x, floatx4 (&acc)[CPLX ? 4 : 2]) {
  auto mm = [](float tab, float v, floatx4 c) {
    return SWAP ? __builtin_amdgcn_mfma_f32_16x16x4f32(v, tab, c, 0, 0, 0)
                : __builtin_amdgcn_mfma_f32_16x16x4f32(tab, v, c, 0, 0, 0);
  };
  if constexpr (CPLX) {
    acc[0] = mm(cs.x, x.x, acc[0]);
    acc[1] = mm(cs.x, x.y, acc[1]);
    acc[2] = mm(cs.y, x.z, acc[2]);
    acc[3] = mm(cs.y, x.w, acc[3]);
  } else {
    acc[0] = mm(cs.x, x.x, acc[0]);
    acc[1] = mm(cs.y, x.y, acc[1]);
  }
}

template <int N>
__device__ inline void clear(floatx4 (&acc)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) acc[i] = floatx4{0.f, 0.f, 0.f, 0.f};
}

// acc += table rows x folded slots over n steps of 4 slots: t is the row
// tile's entries at this lane, v the vectors at this lane's slot and column.
// Four steps at a time, their table entries loaded while the four before are
// multiplied (steps past the end load the last entry and are skipped).
template <bool CPLX, bool SWAP>
__device__ inline void products(const float2 *__restrict__ t, const typename Vec<CPLX>::T *v, int n,
                                floatx4 (&acc)[CPLX ? 4 : 2]) {
  constexpr int kU = 4;
  float2 cs[kU];
#pragma unroll
  for (int u = 0; u < kU; ++u) cs[u] = t[min(u, n - 1) * 64];
  for (int k = 0; k < n; k += kU) {
    float2 next[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) next[u] = t[min(k + kU + u, n - 1) * 64];
    typename Vec<CPLX>::T x[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) x[u] = v[min(k + u, n - 1) * 4 * kPitch];
#pragma unroll
    for (int u = 0; u < kU; ++u)
      if (k + u < n) product<CPLX, SWAP>(cs[u], x[u], acc);   // wavefront-uniform
#pragma unroll
    for (int u = 0; u < kU; ++u) cs[u] = next[u];
  }
}

// The sums of row tile `rt`: acc over all slots (kToGrid: acc over the even
// modes' slots, odd over the rest).  SWAP exchanges the instruction's
// operands, so that consecutive lanes hold consecutive outputs of one line
// instead of one output of consecutive columns.
template <int KIND, bool CPLX, bool SWAP>
__device__ inline void tile_sums(const Geo &g, int rt, const typename Vec<CPLX>::T *V,
                                 floatx4 (&acc)[CPLX ? 4 : 2], floatx4 (&odd)[CPLX ? 4 : 2]) {
  const int lane = threadIdx.x & 63;
  const int steps = g.slots / 4, es = KIND == kToGrid ? g.even_slots / 4 : steps;
  const typename Vec<CPLX>::T *v = V + (lane >> 4) * kPitch + (lane & 15);
  if (KIND == kToModes && rt >= g.even_tiles) v += g.slots * kPitch;
  const float2 *t = g.t + (int64_t)rt * steps * 64 + lane;
  clear(acc);
  products<CPLX, SWAP>(t, v, es, acc);
  if constexpr (KIND == kToGrid) {
    clear(odd);
    products<CPLX, SWAP>(t + es * 64, v + g.even_slots * kPitch, steps - es, odd);
  }
}

// The cosine and sine sums of one output pair, in the form's parts:
// complex (cr, ci, sr, si), real forms (c, s).
template <bool CPLX>
struct Sums;
template <>
struct Sums<true> {
  float cr, ci, sr, si;
  __device__ float2 plus() const { return make_float2(cr - si, ci + sr); }
  __device__ float2 minus() const { return make_float2(cr + si, ci - sr); }
};
template <>
struct Sums<false> {
  float c, s;
};
template <bool CPLX>
__device__ inline Sums<CPLX> sums_of(const floatx4 (&a)[CPLX ? 4 : 2], int j) {
  if constexpr (CPLX)
    return {a[0][j], a[1][j], a[2][j], a[3][j]};
  else
    return {a[0][j], a[1][j]};
}
// Grid rows from the even (e) and odd (o) modes' sums: cell l and cell H - l.
__device__ inline Sums<true> row_l(const Sums<true> &e, const Sums<true> &o) {
  return {e.cr + o.cr, e.ci + o.ci, e.sr + o.sr, e.si + o.si};
}
__device__ inline Sums<true> row_Hl(const Sums<true> &e, const Sums<true> &o) {
  return {e.cr - o.cr, e.ci - o.ci, o.sr - e.sr, o.si - e.si};
}
__device__ inline Sums<false> row_l(const Sums<false> &e, const Sums<false> &o) { return {e.c + o.c, e.s + o.s}; }
__device__ inline Sums<false> row_Hl(const Sums<false> &e, const Sums<false> &o) { return {e.c - o.c, o.s - e.s}; }

// Output row of a tile's row r (0..15): grid cell, mode or frequency; -1
// past the last.  Row 0 is left out of the tiles (zero_row): 64 rows of a
// transform of 129 then make four whole tiles, one per wavefront of a block
// of four, instead of five.
template <int KIND>
__device__ inline int row_of(const Geo &g, int rt, int r) {
  if constexpr (KIND == kToModes) {
    const int odd = rt >= g.even_tiles ? 1 : 0;
    const int q = 2 * ((rt - (odd ? g.even_tiles : 0)) * 16 + r) + 2 - odd;
    return q <= g.h ? q : -1;
  } else {
    const int q = 1 + rt * 16 + r;
    return 2 * q <= g.H ? q : -1;
  }
}

// Calls f(q, col, j, sums, sums of the row H - q (kToGrid)) for this lane's
// four outputs of row tile rt: rows j of one column, or (SWAP) one row of
// columns j.
template <int KIND, bool CPLX, bool SWAP, class F>
__device__ inline void tile_rows(const Geo &g, int rt, const typename Vec<CPLX>::T *V, F f) {
  floatx4 acc[CPLX ? 4 : 2], odd[CPLX ? 4 : 2];
  tile_sums<KIND, CPLX, SWAP>(g, rt, V, acc, odd);
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int q = row_of<KIND>(g, rt, SWAP ? lane & 15 : 4 * (lane >> 4) + j);
    if (q < 0) continue;
    const int col = SWAP ? 4 * (lane >> 4) + j : lane & 15;
    const Sums<CPLX> a = sums_of<CPLX>(acc, j);
    if constexpr (KIND == kToGrid) {
      const Sums<CPLX> o = sums_of<CPLX>(odd, j);
      f(q, col, j, row_l(a, o), row_Hl(a, o));
    } else {
      f(q, col, j, a, a);
    }
  }
}

// Row 0 (cosine 1, sine 0): the weighted sums of E, by one wavefront; calls
// f(0, col, -1, sums, sums of row H) in the lanes of column col = lane < 16.
template <int KIND, bool CPLX, class F>
__device__ inline void zero_row(const Geo &g, const typename Vec<CPLX>::T *V, F f) {
  const int lane = threadIdx.x & 63, steps = g.slots / 4;
  const int es = KIND == kToGrid ? g.even_slots / 4 : steps;
  const float *w = reinterpret_cast<const float *>(g.t + (int64_t)g.tiles * steps * 64) + (lane >> 4);
  const typename Vec<CPLX>::T *v = V + (lane >> 4) * kPitch + (lane & 15);
  float e[2] = {0.f, 0.f}, o[2] = {0.f, 0.f};
  for (int k = 0; k < steps; ++k) {
    const float c = w[4 * k];
    const auto x = v[k * 4 * kPitch];
    float *acc = KIND == kToGrid && k >= es ? o : e;
    acc[0] = fmaf(c, x.x, acc[0]);
    if constexpr (CPLX) acc[1] = fmaf(c, x.y, acc[1]);
  }
#pragma unroll
  for (int off = 16; off < 64; off <<= 1) {
#pragma unroll
    for (int i = 0; i < (CPLX ? 2 : 1); ++i) {
      e[i] += __shfl_xor(e[i], off);
      if (KIND == kToGrid) o[i] += __shfl_xor(o[i], off);
    }
  }
  if (lane >= kCol) return;
  Sums<CPLX> a{}, b{};
  if constexpr (CPLX) {
    a.cr = e[0];
    a.ci = e[1];
    b.cr = o[0];
    b.ci = o[1];
  } else {
    a.c = e[0];
    b.c = o[0];
  }
  if constexpr (KIND == kToGrid)
    f(0, lane, -1, row_l(a, b), row_Hl(a, b));
  else
    f(0, lane, -1, a, a);
}

// ------------------------------------------------------------- kernel ----
constexpr int kMaxLambdas = 16;
struct Tail {
  bool accumulate, clear_in;
  uint32_t even_lines;
  int mirror1, mirror2, half;
  const void *lam_v;
  float lambda[kMaxLambdas];
  uint32_t per;   // columns per system
  const uint8_t *support;
  int positivity;
  const float *err_part;
  int err_n;
  float *err;
};

// *err = (sum of part[0 .. n)) / (sum of part[n .. 2n)), in a fixed order, by
// one block.
__device__ inline void reduce_error(const float *__restrict__ part, int n, float *err) {
  __shared__ float sh[2][kMaxWaves];
  float e = 0.f, a = 0.f;
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    e += part[i];
    a += part[n + i];
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    e += __shfl_xor(e, off);
    a += __shfl_xor(a, off);
  }
  if ((threadIdx.x & 63) == 0) {
    sh[0][threadIdx.x >> 6] = e;
    sh[1][threadIdx.x >> 6] = a;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < (int)(blockDim.x >> 6); ++w) {
      e += sh[0][w];
      a += sh[1][w];
    }
    *err = a > 0.f ? e / a : 0.f;
  }
}

// Blocks take neighbouring column tiles at about the same time (the tiles of
// one XCD are contiguous): strided tiles share cache lines at their edges,
// and a block that walked over several tiles, with its table in registers,
// wrote a third more bytes and took longer (183 against 146 us for a pass of
// 138 MB -> 277 MB) for lack of wavefronts to hide its latencies.
template <int KIND, int IO, bool LINES>
__global__ __launch_bounds__(64 * kMaxWaves) void dft_kernel(Geo g, const void *in, void *out_,
                                                             uint32_t cols, uint32_t B, int len_in,
                                                             int len_out, Tail tail) {
  constexpr bool C = IO == kCC;
  typedef typename Vec<C>::T T;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  T *V = reinterpret_cast<T *>(smem);
  const int lane = threadIdx.x & 63, nw = blockDim.x >> 6;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t st = LINES ? 1 : B;
  const uint32_t c0 = (uint32_t)xcd_contiguous_block() * kCol;
  if constexpr (KIND == kCyclic && IO == kCC) {
    if (tail.err && blockIdx.x == 0) reduce_error(tail.err_part, tail.err_n, tail.err);
  }
  if constexpr (LINES) {   // lanes along a line
    for (int sl = lane; sl < g.slots; sl += 64)
      for (int col0 = wave; col0 < kCol; col0 += 4 * nw) {
        Raw<KIND> raw[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int col = col0 + u * nw;
          const bool ok = col < kCol && c0 + col < cols;
          const uint32_t base = ok ? (c0 + col) * (uint32_t)len_in : 0;
          if constexpr (KIND == kToGrid && IO == kRH) {
            if (tail.even_lines) {   // lines per array, in the order of the other axes' modes
              const uint32_t c = ok ? c0 + col : 0, r = c % tail.even_lines;
              raw[u] = load_even_slot(g, in, base, (c - r + tail.even_lines - 1 - r) * (uint32_t)len_in, sl, ok);
              continue;
            }
          }
          raw[u] = load_slot<KIND, IO>(g, in, base, 1, sl, ok);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (col0 + u * nw < kCol) fold_slot<KIND, IO>(g, raw[u], sl, col0 + u * nw, V);
      }
  } else {                 // lanes across the columns
    const int col = threadIdx.x & (kCol - 1);
    const bool ok = c0 + col < cols;
    const uint32_t base = ok ? col_base(c0 + col, B, len_in) : 0;
    const int step = blockDim.x / kCol;
    for (int s0 = threadIdx.x / kCol; s0 < g.slots; s0 += 4 * step) {
      Raw<KIND> raw[4];   // slots past the end load as zeros
#pragma unroll
      for (int u = 0; u < 4; ++u) raw[u] = load_slot<KIND, IO>(g, in, base, st, s0 + u * step, ok);
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (s0 + u * step < g.slots) fold_slot<KIND, IO>(g, raw[u], s0 + u * step, col, V);
    }
  }
  __syncthreads();
  if constexpr (KIND == kToModes && LINES && IO != kHR) {
    if (tail.clear_in) {   // the block's lines are read: one range of the input
      const uint32_t words = IO == kRH ? 1 : 2;
      const uint32_t lo = c0 * (uint32_t)len_in * words;
      const uint32_t hi = min(c0 + kCol, cols) * (uint32_t)len_in * words;
      float *z = const_cast<float *>(static_cast<const float *>(in));
      for (uint32_t o = lo + threadIdx.x; o < hi; o += blockDim.x) z[o] = 0.f;
    }
  }
  const uint32_t c_lane = c0 + (lane & 15);
  const uint32_t b_lane = LINES || c_lane >= cols ? 0 : col_base(c_lane, B, len_out);
  auto store = [&](int q, int col, int, const Sums<C> &a, const Sums<C> &b) {
    const uint32_t c = LINES ? c0 + col : c_lane;
    if (c >= cols) return;
    const uint32_t base = LINES ? c * (uint32_t)len_out : b_lane;
    const int H = g.H, h = g.h;
    if constexpr (IO == kCC) {
      float2 *out = static_cast<float2 *>(out_);
      auto put = [&](int e, float2 y) {
        const uint32_t o = base + (uint32_t)e * st;
        if (KIND == kToModes) {
          if (tail.accumulate) {
            const float2 z = out[o];
            y.x += z.x;
            y.y += z.y;
          }
          if (tail.lam_v) {
            const float lam = tail.lambda[c / tail.per];
            const float2 z = static_cast<const float2 *>(tail.lam_v)[o];
            y.x = fmaf(lam, z.x, y.x);
            y.y = fmaf(lam, z.y, y.y);
          }
        }
        out[o] = y;
      };
      if constexpr (KIND == kToGrid) {
        put(q, a.plus());
        put(H - q, b.plus());
        if (q > 0) {
          put(2 * H - q, a.minus());
          put(H + q, b.minus());
        }
      } else if constexpr (KIND == kToModes) {
        put(h + q, a.plus());
        if (q > 0) put(h - q, a.minus());
      } else {
        put(q, a.plus());
        if (q > 0 && 2 * q < H) put(H - q, a.minus());
      }
    } else if constexpr (IO == kRH) {
      float2 *out = static_cast<float2 *>(out_);
      out[base + q * st] = make_float2(a.c, a.s);
      if constexpr (KIND == kToGrid) out[base + (H - q) * st] = make_float2(b.c, b.s);
    } else if constexpr (IO == kCRe) {
      // real part at (e, i1, i2) and its mirror image
      float *out = static_cast<float *>(out_);
      const int i1 = (int)(c / (uint32_t)tail.half), i2 = (int)(c - (uint32_t)i1 * tail.half);
      const int m1 = tail.mirror1, m2 = tail.mirror2;
      auto put1 = [&](uint32_t o, float y) {
        if (tail.accumulate) y += out[o];
        out[o] = y;
      };
      auto put = [&](int e, float y) {
        put1(((uint32_t)e * m1 + i1) * m2 + h + i2, y);
        if (i2 != 0) put1(((uint32_t)(2 * h - e) * m1 + (m1 - 1 - i1)) * m2 + h - i2, y);
      };
      put(h + q, a.c - a.s);
      if (q > 0) put(h - q, a.c + a.s);
    } else {   // kHR
      float *out = static_cast<float *>(out_);
      auto put = [&](int e, float y) {
        const uint32_t o = base + (uint32_t)e * st;
        if constexpr (KIND == kCyclic) {
          if (tail.support) {   // the real-space step of error reduction
            const bool holds = tail.support[o] && (!tail.positivity || y >= 0.f);
            y = holds ? y : 0.f;
          }
        } else {
          if (tail.lam_v)
            y = fmaf(tail.lambda[c / tail.per], static_cast<const float *>(tail.lam_v)[o], y);
        }
        out[o] = y;
      };
      if constexpr (KIND == kToModes) {
        put(h + q, a.c - a.s);
        if (q > 0) put(h - q, a.c + a.s);
      } else {
        put(q, a.c - a.s);
        if (q > 0 && 2 * q < H) put(H - q, a.c + a.s);
      }
    }
  };
  for (int rt = wave; rt < g.tiles; rt += nw) tile_rows<KIND, C, LINES>(g, rt, V, store);
  if (wave == nw - 1) zero_row<KIND, C>(g, V, store);
}

// ------------------------------------------------- fused middle passes ----
// Normal equations, axis 0: the columns of X are taken to the grid, the grid
// values multiplied by the kernel's transform, and taken back, all within
// the block.  CPLX = false: the grid values are those of an even real vector,
// hence real; what rounding leaves in their imaginary parts is dropped, so the
// forward sums are the real form's.  The block walks over the n systems of its column tile,
// the kernel's transform at its cells in registers (PRE: one row tile per
// wavefront) and the next system's inputs on their way.
template <bool CPLX, bool PRE>
__global__ __launch_bounds__(64 * kMaxWaves) void dft_normal_kernel(Geo f, Geo b, float2 *X,
                                                                    const float2 *__restrict__ That,
                                                                    int n, uint32_t cols) {
  constexpr int IO = CPLX ? kCC : kCRe;
  typedef typename Vec<CPLX>::T T;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  T *V1 = reinterpret_cast<T *>(smem);
  float4 *V2 = reinterpret_cast<float4 *>(smem + ((size_t)f.slots * kPitch * sizeof(T) + 15) / 16 * 16);
  const uint32_t c0 = (uint32_t)xcd_contiguous_block() * kCol;
  const int tid = threadIdx.x, lane = tid & 63, nw = blockDim.x >> 6;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int H = f.H, N = 2 * f.h + 1;
  const uint32_t st = cols, sys = (uint32_t)N * cols;
  const uint32_t c = c0 + (lane & 15);
  const bool ok = c < cols;
  const uint32_t cc = ok ? c : 0;
  // the kernel's transform at cells l, H - l, L - l, H + l of the lane's rows
  float2 th[4][4];
  auto load_that = [&](int rt) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int l = row_of<kToGrid>(f, rt, 4 * (lane >> 4) + j);
      // clamped addresses: rows and columns past the end are not used
      const int lc = max(l, 0);
      const uint32_t up = lc * st, mid = (uint32_t)H * st;
      th[j][0] = That[cc + up];
      th[j][1] = That[cc + mid - up];
      th[j][2] = That[cc + (lc > 0 ? 2 * mid - up : 0)];
      th[j][3] = That[cc + mid + up];
    }
  };
  // this thread's column of the inputs and its first slot
  const int icol = tid & (kCol - 1), islot = tid / kCol, istep = blockDim.x / kCol;
  const bool iok = c0 + icol < cols;
  const uint32_t ibase = iok ? c0 + icol : 0;
  constexpr int kItems = PRE ? kMaxItems : 1;
  Raw<kToGrid> raw[kItems];
  auto load_system = [&](int s) {
#pragma unroll
    for (int k = 0; k < kItems; ++k)
      raw[k] = load_slot<kToGrid, IO>(f, X, s * sys + ibase, st, islot + k * istep, iok);
  };
  float2 th0[2] = {};   // cells 0 and H (row 0, the last wavefront's)
  if (wave == nw - 1) {
    th0[0] = That[cc];
    th0[1] = That[cc + (uint32_t)H * st];
  }
  if constexpr (PRE) load_system(0);
  if (PRE && wave < f.tiles) load_that(wave);
  // slots of the second transform past the last grid pair
  for (int e = tid; e < b.slots * kCol; e += blockDim.x)
    if (2 * (e / kCol) > H)
      V2[(e / kCol) * kPitch + (e & 15)] = V2[(b.slots + e / kCol) * kPitch + (e & 15)] =
          make_float4(0.f, 0.f, 0.f, 0.f);
  for (int s = 0; s < n; ++s) {
    if constexpr (PRE) {
#pragma unroll
      for (int k = 0; k < kItems; ++k)
        if (islot + k * istep < f.slots) fold_slot<kToGrid, IO>(f, raw[k], islot + k * istep, icol, V1);
    } else {
      for (int sl = islot; sl < f.slots; sl += istep)
        fold_slot<kToGrid, IO>(f, load_slot<kToGrid, IO>(f, X, s * sys + ibase, st, sl, iok), sl, icol, V1);
    }
    __syncthreads();   // V1 is written; V2's readers of the system before are done
    if (PRE && s + 1 < n) load_system(s + 1);
    auto times = [](float2 t, float2 x) {
      if constexpr (CPLX)
        return make_float2(x.x * t.x - x.y * t.y, x.x * t.y + x.y * t.x);
      else
        return make_float2(x.x * t.x, x.x * t.y);
    };
    auto multiply = [&](int l, int col, int j, const Sums<CPLX> &u, const Sums<CPLX> &v) {
      float2 ga, gb, gc, gd;   // cells l, L - l, H - l, H + l
      const float2 ta = j < 0 ? th0[0] : th[j & 3][0], tc = j < 0 ? th0[1] : th[j & 3][1];
      if constexpr (CPLX) {
        ga = times(ta, u.plus());
        gc = times(tc, v.plus());
        gb = times(th[j & 3][2], u.minus());
        gd = times(th[j & 3][3], v.minus());
      } else {
        ga = times(ta, make_float2(u.c - u.s, 0.f));
        gc = times(tc, make_float2(v.c - v.s, 0.f));
        gb = times(th[j & 3][2], make_float2(u.c + u.s, 0.f));
        gd = times(th[j & 3][3], make_float2(v.c + v.s, 0.f));
      }
      if (j < 0) gb = gd = make_float2(0.f, 0.f);
      const float4 p = fold<kCC>(ga, gb), q = fold<kCC>(gc, gd);
      V2[l * kPitch + col] = vadd(p, q, -1.f);
      V2[(b.slots + l) * kPitch + col] = vsub(p, q, 1.f);
    };
    for (int rt = wave; rt < f.tiles; rt += nw) {
      if (!PRE) load_that(rt);
      tile_rows<kToGrid, CPLX, false>(f, rt, V1, multiply);
    }
    if (wave == nw - 1) zero_row<kToGrid, CPLX>(f, V1, multiply);
    __syncthreads();   // V2 is written; V1's readers are done
    const uint32_t x0 = s * sys + c + (uint32_t)b.h * st;
    auto store = [&](int k, int, int, const Sums<true> &u, const Sums<true> &) {
      if (!ok) return;
      const uint32_t d = (uint32_t)k * st;
      X[x0 + d] = u.plus();
      if (k > 0) X[x0 - d] = u.minus();
    };
    for (int rt = wave; rt < b.tiles; rt += nw) tile_rows<kToModes, true, false>(b, rt, V2, store);
    if (wave == 0) zero_row<kToModes, true>(b, V2, store);
  }
}

// Amplitude projection of one coefficient f = F[k] of the half spectrum of a
// real density and, with it, of F[-k] = conj f.  The next density is the real
// part of the inverse transform, that is the inverse transform of the
// Hermitian part (G[k] + conj G[-k]) / 2 of the projected spectrum: with
// G[+-k] = amp[+-k] f / |f| where measured (amp where f is 0 or not finite)
// and f elsewhere; an f that neither side keeps is replaced, whatever it is.
// k2_self: the mirror image lies in the half spectrum itself and counts its
// own error.
struct Amps {
  float a, am;        // amp[k], amp[-k]
  bool seen, seen_m;  // measured
};
__device__ inline float2 project(float2 f, const Amps &m, bool k2_self, float &e, float &a2) {
  const float mag = sqrtf(fmaf(f.x, f.x, f.y * f.y));
  float2 u = mag > 0.f ? make_float2(f.x / mag, f.y / mag) : make_float2(1.f, 0.f);
  if (u.x != u.x || u.y != u.y) u = make_float2(1.f, 0.f);   // infinite f
  float w = 0.f, keep = 2.f;
  if (m.seen) {
    const float d = mag - m.a;
    e = fmaf(d, d, e);
    a2 = fmaf(m.a, m.a, a2);
    w += m.a;
    keep -= 1.f;
  }
  if (m.seen_m) {
    if (!k2_self) {
      const float d = mag - m.am;
      e = fmaf(d, d, e);
      a2 = fmaf(m.am, m.am, a2);
    }
    w += m.am;
    keep -= 1.f;
  }
  const float2 kept = keep > 0.f ? make_float2(keep * f.x, keep * f.y) : make_float2(0.f, 0.f);
  return make_float2(0.5f * fmaf(w, u.x, kept.x), 0.5f * fmaf(w, u.y, kept.y));
}

// The amplitudes at (k0, k1, k2) and at its mirror image, axes of n.
__device__ inline Amps load_amps(const float *__restrict__ amp, const uint8_t *__restrict__ measured,
                                 uint32_t n, uint32_t k0, uint32_t k1, uint32_t k2) {
  const uint32_t m0 = k0 ? n - k0 : 0, m1 = k1 ? n - k1 : 0, m2 = k2 ? n - k2 : 0;
  const uint32_t o = (k0 * n + k1) * n + k2, om = (m0 * n + m1) * n + m2;
  return {amp[o], amp[om], !measured || measured[o] != 0, !measured || measured[om] != 0};
}

// Sums e and a2 over the block (a fixed order) into part[block] and
// part[gridDim + block].
__device__ inline void store_error(float e, float a2, float *__restrict__ part) {
  __shared__ float sh[2][kMaxWaves];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    e += __shfl_xor(e, off);
    a2 += __shfl_xor(a2, off);
  }
  if ((threadIdx.x & 63) == 0) {
    sh[0][threadIdx.x >> 6] = e;
    sh[1][threadIdx.x >> 6] = a2;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < (int)(blockDim.x >> 6); ++w) {
      e += sh[0][w];
      a2 += sh[1][w];
    }
    part[blockIdx.x] = e;
    part[gridDim.x + blockIdx.x] = a2;
  }
}

// Phasing, axis 0: the columns of the half spectrum are transformed,
// projected and transformed back within the block.
__global__ __launch_bounds__(64 * kMaxWaves) void dft_phase_kernel(Geo f, Geo b, float2 *X,
                                                                   const float *__restrict__ amp,
                                                                   const uint8_t *__restrict__ measured,
                                                                   uint32_t cols,
                                                                   float *__restrict__ part) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  float4 *V1 = reinterpret_cast<float4 *>(smem);
  float4 *V2 = V1 + f.slots * kPitch;
  const uint32_t c0 = (uint32_t)xcd_contiguous_block() * kCol;
  const int tid = threadIdx.x, lane = tid & 63, nw = blockDim.x >> 6;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t n = f.H, half = n / 2 + 1, st = cols;
  const uint32_t c = c0 + (lane & 15);
  const bool ok = c < cols;
  const uint32_t k1 = ok ? c / half : 0, k2 = ok ? c - k1 * half : 0;
  const bool k2_self = k2 == 0 || 2 * k2 == n;
  {
    const int icol = tid & (kCol - 1), step = blockDim.x / kCol;
    const bool iok = c0 + icol < cols;
    const uint32_t base = iok ? c0 + icol : 0;
    for (int s0 = tid / kCol; s0 < f.slots; s0 += 4 * step) {
      Raw<kCyclic> raw[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) raw[u] = load_slot<kCyclic, kCC>(f, X, base, st, s0 + u * step, iok);
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (s0 + u * step < f.slots) fold_slot<kCyclic, kCC>(f, raw[u], s0 + u * step, icol, V1);
    }
    for (int e = tid; e < b.slots * kCol; e += blockDim.x)
      if (2 * (e / kCol) > (int)n) V2[(e / kCol) * kPitch + (e & 15)] = make_float4(0.f, 0.f, 0.f, 0.f);
  }
  float e = 0.f, a2 = 0.f;
  Amps am[4][2];   // rows q and n - q of the lane
  auto load_rows = [&](int rt) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t q = max(row_of<kCyclic>(f, rt, 4 * (lane >> 4) + j), 0);   // clamped: not used
      am[j][0] = load_amps(amp, measured, n, q, k1, k2);
      am[j][1] = load_amps(amp, measured, n, q ? n - q : 0, k1, k2);
    }
  };
  if (wave < f.tiles) load_rows(wave);
  __syncthreads();
  auto fold2 = [&](int q, int col, const Sums<true> &a, const Amps &mp, const Amps &mm) {
    if (!ok) {   // columns past the end: any finite values
      V2[q * kPitch + col] = make_float4(0.f, 0.f, 0.f, 0.f);
      return;
    }
    const float2 g = project(a.plus(), mp, k2_self, e, a2);
    float2 h = make_float2(0.f, 0.f);
    if (q > 0 && 2 * q < (int)n) h = project(a.minus(), mm, k2_self, e, a2);
    V2[q * kPitch + col] = fold<kCC>(g, h);
  };
  for (int rt = wave; rt < f.tiles; rt += nw) {
    if (rt != wave) load_rows(rt);
    tile_rows<kCyclic, true, false>(f, rt, V1, [&](int q, int col, int j, const Sums<true> &a, const Sums<true> &) {
      fold2(q, col, a, am[j][0], am[j][1]);
    });
  }
  if (wave == nw - 1) {
    const Amps a0 = load_amps(amp, measured, n, 0, k1, k2);
    zero_row<kCyclic, true>(f, V1, [&](int q, int col, int, const Sums<true> &a, const Sums<true> &) {
      fold2(q, col, a, a0, a0);
    });
  }
  __syncthreads();
  auto store = [&](int q, int, int, const Sums<true> &a, const Sums<true> &) {
    if (!ok) return;
    X[c + (uint32_t)q * st] = a.plus();
    if (q > 0 && 2 * q < (int)n) X[c + (n - (uint32_t)q) * st] = a.minus();
  };
  for (int rt = wave; rt < b.tiles; rt += nw) tile_rows<kCyclic, true, false>(b, rt, V2, store);
  if (wave == 0) zero_row<kCyclic, true>(b, V2, store);
  store_error(e, a2, part);
}

// The projection alone (sizes whose fused pass does not fit the LDS).
__global__ __launch_bounds__(256) void phase_projection_kernel(float2 *__restrict__ F,
                                                               const float *__restrict__ amp,
                                                               const uint8_t *__restrict__ measured,
                                                               uint32_t n, uint32_t cols,
                                                               float *__restrict__ part) {
  const uint32_t half = n / 2 + 1;
  const int64_t total = (int64_t)n * cols, stride = (int64_t)gridDim.x * 256;
  float e = 0.f, a2 = 0.f;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < total; i += stride) {
    const uint32_t k0 = (uint32_t)(i / cols), c = (uint32_t)(i - (int64_t)k0 * cols);
    const uint32_t k1 = c / half, k2 = c - k1 * half;
    F[i] = project(F[i], load_amps(amp, measured, n, k0, k1, k2), k2 == 0 || 2 * k2 == n, e, a2);
  }
  store_error(e, a2, part);
}

// --------------------------------------------------------------- host ----
static int up(int v, int m) { return (v + m - 1) / m * m; }

static size_t table_bytes(const DftTable &tab) {
  return (size_t)tab.tiles * (tab.slots / 4) * 64 * sizeof(float2) + tab.slots * sizeof(float);
}

size_t dft_table_sizes(DftTable &tab, int kind, int h, int H) {
  tab.kind = kind;
  tab.h = h;
  tab.H = H;
  const int pairs = H / 2 + 1;   // grid cells 0..H/2 (kCyclic: frequencies 0..n/2)
  tab.even_slots = tab.even_tiles = 0;
  tab.slots = up(pairs, 4);
  tab.tiles = up(pairs - 1, 16) / 16;   // row 0 apart
  if (kind == kToGrid) {
    tab.even_slots = up(h / 2 + 1, 4);
    tab.slots = tab.even_slots + up((h + 1) / 2, 4);
  } else if (kind == kToModes) {
    tab.even_tiles = up(h / 2, 16) / 16;
    tab.tiles = tab.even_tiles + up((h + 1) / 2, 16) / 16;
  }
  return table_bytes(tab);
}

void dft_table_values(const DftTable &tab, int sign, const std::function<double(int)> &weight,
                      float2 *t) {
  const int steps = tab.slots / 4;
  const long n = tab.kind == kCyclic ? tab.H : 2L * tab.H;
  const size_t tiled = (size_t)tab.tiles * steps * 64;
  std::fill(t, t + tiled + tab.slots / 2, make_float2(0.f, 0.f));
  float *row0 = reinterpret_cast<float *>(t + tiled);
  // phases reduced modulo the length exactly, float64, rounded once
  std::vector<double> co(n), si(n);
  for (long j = 0; j < n; ++j) {
    co[j] = std::cos(2.0 * M_PI * (double)j / (double)n);
    si[j] = 2 * j == n ? 0.0 : std::sin(2.0 * M_PI * (double)j / (double)n) * sign;
  }
  // the (cell, mode) pair of a slot and an output row; for kCyclic the cell
  // is the input's index, the mode the output's
  auto mode_of_slot = [&](int slot) {
    return slot < tab.even_slots ? 2 * slot : 2 * (slot - tab.even_slots) + 1;
  };
  auto put = [&](long cell, long mode, float2 &v) {
    if (2 * cell > tab.H || (tab.kind == kCyclic ? 2 * mode > tab.H : mode > tab.h)) return;
    const double w = weight((int)mode);
    const long ph = (cell * mode) % n;
    v = make_float2((float)(co[ph] * w), (float)(si[ph] * w));
  };
  for (int rt = 0; rt < tab.tiles; ++rt)
    for (int st = 0; st < steps; ++st)
      for (int lane = 0; lane < 64; ++lane) {
        const int r = lane & 15, slot = 4 * st + (lane >> 4);
        float2 &v = t[((size_t)rt * steps + st) * 64 + lane];
        if (tab.kind == kToGrid)
          put(1 + rt * 16 + r, mode_of_slot(slot), v);
        else if (tab.kind == kToModes)
          put(slot, rt < tab.even_tiles ? 2 * (rt * 16 + r) + 2 : 2 * ((rt - tab.even_tiles) * 16 + r) + 1, v);
        else
          put(slot, 1 + rt * 16 + r, v);
      }
  for (int slot = 0; slot < tab.slots; ++slot) {
    float2 v = make_float2(0.f, 0.f);
    if (tab.kind == kToGrid)
      put(0, mode_of_slot(slot), v);
    else
      put(slot, 0, v);
    row0[slot] = v.x;
  }
}

hipError_t dft_table_fill(DftTable &tab, int sign, const std::function<double(int)> &weight) {
  std::vector<float2> t(table_bytes(tab) / sizeof(float2));
  dft_table_values(tab, sign, weight, t.data());
  return hipMemcpy(tab.t, t.data(), table_bytes(tab), hipMemcpyHostToDevice);
}

// Wavefronts per block: one per row tile up to eight, rounded to 2, 4 or 8.
// A CU places a block's wavefronts over its four SIMDs: five of them (a
// block of five row tiles) left one resident block per CU, its SIMDs uneven.
static int waves_of(int tiles) { return tiles <= 2 ? 2 : tiles <= 4 ? 4 : 8; }

static size_t fold_bytes(const DftTable &t, bool cplx) {
  return (size_t)t.slots * kPitch * (cplx ? 16 : 8) * (t.kind == kToModes ? 2 : 1);
}

template <int KIND, int IO, bool LINES>
static hipError_t dft_go2(const DftTable &tab, const DftLines &ln, const void *in, void *out,
                          const Tail &tail, hipStream_t s) {
  const int64_t blocks = (ln.cols + kCol - 1) / kCol;
  if (blocks * kCol * std::max(ln.len_in, ln.len_out) > 0x7fffffffLL) return hipErrorInvalidValue;
  const size_t lds = fold_bytes(tab, IO == kCC);
  if (lds > kLdsMax) return hipErrorInvalidValue;
  hipLaunchKernelGGL((dft_kernel<KIND, IO, LINES>), dim3((unsigned)blocks),
                     dim3(64 * waves_of(tab.tiles)), lds, s, geo_of(tab), in, out,
                     (uint32_t)ln.cols, (uint32_t)ln.B, ln.len_in, ln.len_out, tail);
  return hipGetLastError();
}

template <int KIND, int IO>
static hipError_t dft_go(const DftTable &tab, const DftLines &ln, const void *in, void *out,
                         const Tail &tail, hipStream_t s) {
  // real sides are axis 2 (contiguous lines), real parts axis 0
  constexpr bool kLinesOnly = IO == kRH || IO == kHR;
  if (kLinesOnly ? ln.B != 1 : IO == kCRe && ln.B == 1) return hipErrorInvalidValue;
  return ln.B == 1 ? dft_go2<KIND, IO, IO != kCRe>(tab, ln, in, out, tail, s)
                   : dft_go2<KIND, IO, kLinesOnly>(tab, ln, in, out, tail, s);
}

hipError_t launch_dft(const DftTable &tab, int io, const DftLines &ln, const void *in, void *out,
                      const DftEpilogue &ep, hipStream_t s) {
  if (ln.cols <= 0) return hipSuccess;
  Tail t{};
  t.accumulate = ep.accumulate;
  t.clear_in = ep.clear_in;
  t.even_lines = (uint32_t)ep.even_lines;
  t.mirror1 = ep.mirror1;
  t.mirror2 = ep.mirror2;
  t.half = ep.mirror1 > 0 ? (int)(ln.cols / ep.mirror1) : 1;
  t.lam_v = ep.lam_v;
  for (int i = 0; i < ep.systems && i < kMaxLambdas; ++i) t.lambda[i] = ep.lambda[i];
  t.per = ep.cols_per_system > 0 ? ep.cols_per_system : 1;
  t.support = ep.support;
  t.positivity = ep.positivity;
  t.err_part = ep.err_part;
  t.err_n = ep.err_n;
  t.err = ep.err;
  switch (tab.kind * 4 + io) {
    case kToGrid * 4 + kCC: return dft_go<kToGrid, kCC>(tab, ln, in, out, t, s);
    case kToGrid * 4 + kRH: return dft_go<kToGrid, kRH>(tab, ln, in, out, t, s);
    case kToModes * 4 + kCC: return dft_go<kToModes, kCC>(tab, ln, in, out, t, s);
    case kToModes * 4 + kRH: return dft_go<kToModes, kRH>(tab, ln, in, out, t, s);
    case kToModes * 4 + kCRe: return dft_go<kToModes, kCRe>(tab, ln, in, out, t, s);
    case kToModes * 4 + kHR: return dft_go<kToModes, kHR>(tab, ln, in, out, t, s);
    case kCyclic * 4 + kCC: return dft_go<kCyclic, kCC>(tab, ln, in, out, t, s);
    case kCyclic * 4 + kRH: return dft_go<kCyclic, kRH>(tab, ln, in, out, t, s);
    case kCyclic * 4 + kHR: return dft_go<kCyclic, kHR>(tab, ln, in, out, t, s);
    default: return hipErrorInvalidValue;
  }
}

static size_t normal_lds(const DftTable &f, const DftTable &b, bool cplx) {
  return (fold_bytes(f, cplx) + 15) / 16 * 16 + fold_bytes(b, true);
}

bool dft_normal_fits(const DftTable &to_grid, const DftTable &to_modes, bool cplx) {
  return normal_lds(to_grid, to_modes, cplx) <= kLdsMax;
}

hipError_t launch_dft_normal(const DftTable &f, const DftTable &b, bool cplx, float2 *X,
                             const float2 *That, int n, int64_t cols, hipStream_t s) {
  const int64_t blocks = (cols + kCol - 1) / kCol;
  if (blocks * kCol * 2 * f.H > 0x7fffffffLL || (int64_t)n * (2 * f.h + 1) * cols > 0x7fffffffLL)
    return hipErrorInvalidValue;
  const int waves = waves_of(std::max(f.tiles, b.tiles));
  const bool pre = f.tiles <= waves && (f.slots * kCol + 64 * waves - 1) / (64 * waves) <= kMaxItems;
  const dim3 grid((unsigned)blocks), block(64 * waves);
  const size_t lds = normal_lds(f, b, cplx);
#define SPFEL_DFTN(C, P)                                                                         \
  hipLaunchKernelGGL((dft_normal_kernel<C, P>), grid, block, lds, s, geo_of(f), geo_of(b), X,    \
                     That, n, (uint32_t)cols)
  if (cplx && pre)
    SPFEL_DFTN(true, true);
  else if (cplx)
    SPFEL_DFTN(true, false);
  else if (pre)
    SPFEL_DFTN(false, true);
  else
    SPFEL_DFTN(false, false);
#undef SPFEL_DFTN
  return hipGetLastError();
}

static int64_t phase_cols(int n) { return (int64_t)n * (n / 2 + 1); }

int64_t dft_phase_parts(int n) { return (phase_cols(n) + kCol - 1) / kCol; }

bool dft_phase_fits(const DftTable &tab) { return 2 * fold_bytes(tab, true) <= kLdsMax - 256; }

hipError_t launch_dft_phase(const DftTable &fwd, const DftTable &inv, float2 *X, const float *amp,
                            const uint8_t *measured, float *part, hipStream_t s) {
  const int n = fwd.H;
  hipLaunchKernelGGL(dft_phase_kernel, dim3((unsigned)dft_phase_parts(n)), dim3(64 * waves_of(fwd.tiles)),
                     2 * fold_bytes(fwd, true), s, geo_of(fwd), geo_of(inv), X, amp, measured,
                     (uint32_t)phase_cols(n), part);
  return hipGetLastError();
}

hipError_t launch_phase_projection(int n, float2 *F, const float *amp, const uint8_t *measured,
                                   float *part, hipStream_t s) {
  hipLaunchKernelGGL(phase_projection_kernel, dim3((unsigned)dft_phase_parts(n)), dim3(256), 0, s, F,
                     amp, measured, (uint32_t)n, (uint32_t)phase_cols(n), part);
  return hipGetLastError();
}

}  // namespace spfel
