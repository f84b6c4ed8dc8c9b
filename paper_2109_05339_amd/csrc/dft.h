// Line transforms of the separable 3D DFTs (dft.hip): tables, shapes and
// launchers shared by the merge's transform, the normal equations and
// phasing.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <functional>

namespace spfel {

// What a line transform maps.  L = 2 H is the grid length (H odd), h the
// largest mode; modes are stored centred (mode k at index k + h).
//   kToGrid   modes -h..h -> grid cells 0..L-1
//   kToModes  grid cells 0..L-1 -> modes -h..h
//   kCyclic   n cells -> n frequencies, both in standard order (H = n)
enum DftKind { kToGrid = 0, kToModes = 1, kCyclic = 2 };

// Values on each side of a line.
//   kCC  complex -> complex
//   kRH  real -> complex, the nonnegative half of the output alone
//        (grid 0..H, modes 0..h, frequencies 0..n/2)
//   kCRe complex -> the real part, written at the output and at its mirror
//        image through the origin of the 3D output (kToModes)
//   kHR  the nonnegative half of a Hermitian line -> real
enum DftIo { kCC = 0, kRH = 1, kCRe = 2, kHR = 3 };

// A line transform's table on the device, in matrix-operand order: entry
// (tile, step, lane) holds the cosine and sine terms of output row
// 16 tile + lane % 16 and input slot 4 step + lane / 16.
struct DftTable {
  int kind = kCyclic, h = 0, H = 0;
  int even_slots = 0, slots = 0;   // input slots (multiples of 4); kToGrid: even modes first
  int even_tiles = 0, tiles = 0;   // output row tiles; kToModes: even modes first
  float2 *t = nullptr;
};

// Host part of a table: its sizes (returns its bytes, a multiple of 16), its
// values (t: that many bytes of host memory), and the values sent to the device.
// weight(k) multiplies mode (or output frequency) k; sign is that of the exponent.
size_t dft_table_sizes(DftTable &tab, int kind, int h, int H);
void dft_table_values(const DftTable &tab, int sign, const std::function<double(int)> &weight,
                      float2 *t);
hipError_t dft_table_fill(DftTable &tab, int sign, const std::function<double(int)> &weight);

// Lines of one launch: element e of column c = (a, b), b < B, is at
// (a len + e) B + b on either side, with that side's len.
struct DftLines {
  int64_t cols = 0;   // A * B
  int B = 1;
  int len_in = 0, len_out = 0;
};

// One line transform.  accumulate: kToModes outputs are added to `out`.
// kCRe: `mirror1` and `mirror2` are the lengths of the two other axes of the
// mirrored output (axis 1 full, axis 2 full), B = mirror1 * (half of axis 2).
// lambda / lam_v (kToModes, kHR or kCC): adds lambda[a / per] * lam_v to the
// output, element for element.
struct DftEpilogue {
  bool accumulate = false;
  bool clear_in = false;   // zeros the lines once read (kToModes on contiguous lines)
  int64_t even_lines = 0;  // kToGrid, kRH: transforms the even part of 3D arrays of this many lines each
  int mirror1 = 0, mirror2 = 0;
  const void *lam_v = nullptr;
  const float *lambda = nullptr;   // host values, one per system
  int systems = 0;
  int64_t cols_per_system = 0;
  // real-space step of error reduction (kCyclic, kHR): out is rho
  const uint8_t *support = nullptr;
  int positivity = 0;
  // error of a phasing iteration (kCyclic, kCC): *err = sum of the first
  // err_n partial sums over the sum of the next err_n, by the first block
  const float *err_part = nullptr;
  int err_n = 0;
  float *err = nullptr;
};
hipError_t launch_dft(const DftTable &tab, int io, const DftLines &ln, const void *in, void *out,
                      const DftEpilogue &ep, hipStream_t s);

// Whether the fused middle passes below fit the LDS for this table.
bool dft_normal_fits(const DftTable &to_grid, const DftTable &to_modes, bool cplx);
bool dft_phase_fits(const DftTable &tab);

// Axis-0 pass of the normal equations in place on X (n systems of [N][cols]
// complex columns): to the grid, times That ([L][cols]), back to the modes.
// cplx = false: the columns come from an even real vector, whose grid values
// are real; what rounding leaves in their imaginary parts is dropped.
hipError_t launch_dft_normal(const DftTable &to_grid, const DftTable &to_modes, bool cplx,
                             float2 *X, const float2 *That, int n, int64_t cols, hipStream_t s);

// Axis-0 pass of phasing in place on X ([n][cols] complex columns, cols =
// n * (n/2 + 1): the nonnegative half of axis 2): forward transform, the
// amplitude projection of the full spectrum and inverse transform.  part
// receives dft_phase_parts(n) partial sums of (|F| - amp)^2 over the measured
// coefficients, then as many of amp^2.
int64_t dft_phase_parts(int n);
hipError_t launch_dft_phase(const DftTable &fwd, const DftTable &inv, float2 *X, const float *amp,
                            const uint8_t *measured, float *part, hipStream_t s);
// The projection alone, in place on F (the same half spectrum [n][cols]).
hipError_t launch_phase_projection(int n, float2 *F, const float *amp, const uint8_t *measured,
                                   float *part, hipStream_t s);

}  // namespace spfel
