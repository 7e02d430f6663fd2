// Kernels and launcher of the line pass along one axis; line_row.hip and line_col.hip instantiate them.
//
// A real-time step in one sweep.  The k-space propagator of Eqs. (H1), (H4) (Eq. TEOp) factors exactly:
// K(h) = X(h) Y(h), with X = F_x^-1 M'(k_x) F_x (k_x^2 / 2, the spin-momentum term and the uniform Raman
// coupling, a 2x2 matrix per k_x) along rows and Y = F_y^-1 P(k_y) F_y (k_y^2 / 2, a scalar) along columns,
// and X and Y commute.  So K(dt) between two real-space steps can be applied in either order, and with
// the order alternating a run of Strang steps reads
//     X(dt/2) | Y(dt/2) R Y(dt) | X(dt) R X(dt) | Y(dt) R Y(dt) | ... | Z(dt) R Z(dt/2) | W(dt/2)
// where every | is one trip of the state through memory: a step takes one sweep that holds a line along
// one axis through two 1-D convolutions and R, instead of a row and a column sweep.  The transforms per
// step are the same four.  (Imaginary time cannot do this: the norm of K(dt/2) R K(dt/2) psi is needed
// before the next R, and it is not known from data along one axis.)
//
// Bound: two passes' worth of VALU work per launch (about 2700 wave instructions at 1024 points and 16
// per lane) over one exchange of the state between the XCDs.  Measured per step, two sweeps -> one: 12.0
// -> 7.8 us at 512^2, 25.2 -> 16.2 us at 1024^2, 9.8 -> 6.5 us at 64^2 in complex128 (with the transforms
// of fft_device.hpp; calls of 50 to 200 steps on a caller's buffer).  Tiles and points per lane are the schedule's.
#pragma once

#include "line_body.hpp"

namespace sgpe {

// threads of a workgroup: column tiles may be wide (wide_cols, api.cpp) where the pass holds its registers
// at four waves per SIMD, which it does with the diagonal real-space exponential (but for 2 to 4 values
// that spill); with a spatial coupling a wide tile is taken in halves (line_cols, api.cpp)
constexpr int line_threads(int n, bool col, bool full) { return col && !full && n >= 2048 ? 1024 : 512; }

template <int N, bool COL, bool FULL, bool NLN, int P>
__global__ void __launch_bounds__(line_threads(N, COL, FULL)) line_kernel(LineArgs a) {
  line_body<N, COL, FULL, NLN, P, true>(a, blockIdx.x, gridDim.x);
}

template <int N, bool COL, bool FULL, int P>
__global__ void __launch_bounds__(line_threads(N, COL, FULL)) line_kernel_batch(const LineArgs* __restrict__ tab) {
  const int2 w = batch_item();
  line_body<N, COL, FULL, false, P, false>(tab[w.x], w.y, gridDim.x);
}

// complex128: 16 (or, for lines up to kMaxNSmallP, 8) points per lane, groups of at most 256 threads
// except where one line needs 512
template <int N, bool COL, bool FULL, int P>
__global__ void __launch_bounds__(2 * N / P > 256 ? 512 : 256) line_kernel_c128(LineArgsT<double> a) {
  line_body<N, COL, FULL, false, P, false>(a, blockIdx.x, gridDim.x);
}

template <int N, bool COL, bool FULL, bool NLN>
static hipError_t line_launch_t(const LineArgs& a, const LineArgs* tab, int count, int n_lines, int points,
                                hipStream_t s) {
  const dim3 block(2 * a.lines * (N / points));
  const dim3 grid(n_lines / a.lines, tab ? count : 1);
  const size_t lds = row_lds_bytes(N, a.lines);
  if (tab) {
    if constexpr (NLN) {
      return hipErrorInvalidValue;   // batches run the default split only
    } else {
      if (points == 16) hipLaunchKernelGGL((line_kernel_batch<N, COL, FULL, 16>), grid, block, lds, s, tab);
      else if constexpr (N <= kMaxNSmallP) {
        if (points == 8) hipLaunchKernelGGL((line_kernel_batch<N, COL, FULL, 8>), grid, block, lds, s, tab);
        else hipLaunchKernelGGL((line_kernel_batch<N, COL, FULL, 4>), grid, block, lds, s, tab);
      }
    }
  } else if (points == 16) {
    hipLaunchKernelGGL((line_kernel<N, COL, FULL, NLN, 16>), grid, block, lds, s, a);
  } else if constexpr (N <= kMaxNSmallP) {
    if (points == 8) hipLaunchKernelGGL((line_kernel<N, COL, FULL, NLN, 8>), grid, block, lds, s, a);
    else hipLaunchKernelGGL((line_kernel<N, COL, FULL, NLN, 4>), grid, block, lds, s, a);
  }
  return hipGetLastError();
}

template <int N, bool COL>
static hipError_t line_launch_n(const LineArgs& a, const LineArgs* tab, int count, int n_lines, bool full, bool nln,
                                int points, hipStream_t s) {
  // with a diagonal linear part the three factors of N L N are phases, which commute and leave both
  // densities as they are: their product is the frozen form's one phase
  if (!full) return line_launch_t<N, COL, false, false>(a, tab, count, n_lines, points, s);
  return nln ? line_launch_t<N, COL, true, true>(a, tab, count, n_lines, points, s)
             : line_launch_t<N, COL, true, false>(a, tab, count, n_lines, points, s);
}

template <bool COL>
static hipError_t line_dispatch(const LineArgs& a, const LineArgs* tab, int count, int n, int n_lines, bool full,
                                bool nln, int points, hipStream_t s) {
  if (!(COL && !full ? col_launch_supported : schedule_supported)(n, a.lines, 1, points) || n_lines % a.lines != 0)
    return hipErrorInvalidValue;
  if (tab && (count < 1 || count > 65535)) return hipErrorInvalidValue;
  switch (n) {
    case 16: return line_launch_n<16, COL>(a, tab, count, n_lines, full, nln, points, s);
    case 32: return line_launch_n<32, COL>(a, tab, count, n_lines, full, nln, points, s);
    case 64: return line_launch_n<64, COL>(a, tab, count, n_lines, full, nln, points, s);
    case 128: return line_launch_n<128, COL>(a, tab, count, n_lines, full, nln, points, s);
    case 256: return line_launch_n<256, COL>(a, tab, count, n_lines, full, nln, points, s);
    case 512: return line_launch_n<512, COL>(a, tab, count, n_lines, full, nln, points, s);
    case 1024: return line_launch_n<1024, COL>(a, tab, count, n_lines, full, nln, points, s);
    case 2048: return line_launch_n<2048, COL>(a, tab, count, n_lines, full, nln, points, s);
    case 4096: return line_launch_n<4096, COL>(a, tab, count, n_lines, full, nln, points, s);
    default: return hipErrorInvalidValue;
  }
}

template <int N, bool COL, bool FULL>
static hipError_t line_launch_c128(const LineArgsT<double>& a, int n_lines, int points, hipStream_t s) {
  const dim3 block(2 * a.lines * (N / points));
  const dim3 grid(n_lines / a.lines);
  if (block.x > (2 * N / points > 256 ? 512u : 256u)) return hipErrorInvalidValue;
  const size_t lds = 2 * row_lds_bytes(N, a.lines);   // double2 slots
  if (points == 16) {
    hipLaunchKernelGGL((line_kernel_c128<N, COL, FULL, 16>), grid, block, lds, s, a);
  } else if constexpr (N <= kMaxNSmallP) {
    hipLaunchKernelGGL((line_kernel_c128<N, COL, FULL, 8>), grid, block, lds, s, a);
  }
  return hipGetLastError();
}

template <int N, bool COL>
static hipError_t line_launch_c128_n(const LineArgsT<double>& a, int n_lines, bool full, int points, hipStream_t s) {
  return full ? line_launch_c128<N, COL, true>(a, n_lines, points, s)
              : line_launch_c128<N, COL, false>(a, n_lines, points, s);
}

template <bool COL>
static hipError_t line_dispatch_c128(const LineArgsT<double>& a, int n, int n_lines, bool full, int points,
                                     hipStream_t s) {
  if ((points != 16 && points != 8) || !schedule_supported(n, a.lines, 1, points) || n_lines % a.lines != 0)
    return hipErrorInvalidValue;
  switch (n) {
    case 16: return line_launch_c128_n<16, COL>(a, n_lines, full, points, s);
    case 32: return line_launch_c128_n<32, COL>(a, n_lines, full, points, s);
    case 64: return line_launch_c128_n<64, COL>(a, n_lines, full, points, s);
    case 128: return line_launch_c128_n<128, COL>(a, n_lines, full, points, s);
    case 256: return line_launch_c128_n<256, COL>(a, n_lines, full, points, s);
    case 512: return line_launch_c128_n<512, COL>(a, n_lines, full, points, s);
    case 1024: return line_launch_c128_n<1024, COL>(a, n_lines, full, points, s);
    case 2048: return line_launch_c128_n<2048, COL>(a, n_lines, full, points, s);
    case 4096: return line_launch_c128_n<4096, COL>(a, n_lines, full, points, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace sgpe
