// HIP kernels of the split-step solver for gfx950: energy and norm reductions, and the
// workgroup geometry shared by all passes.
#include <algorithm>
#include <type_traits>

#include "col_body.hpp"
#include "fft_device.hpp"
#include "sgpe_internal.hpp"

namespace sgpe {

// -------------------------------------------------------------------------------------------
// Geometry
// -------------------------------------------------------------------------------------------
// Step kernels: lane pairs (two components) x T = n/points lanes per line; a slot of the LDS
// exchange holds both components (16 bytes); lds_line places the lines.
size_t row_lds_bytes(int nx, int rows) { return size_t(rows) * size_t(nx + nx / 16) * 16 + kLdsSkew; }

// column pass: the transforms' exchange slots, then the k_y operator row (one float per k_y)
size_t col_lds_bytes(int ny, int cols) { return row_lds_bytes(ny, cols) + size_t(ny) * 4; }

// complex128 column pass: double2 slots, and the k_y row (one double per k_y) where the kernel
// stages it in LDS (16 points per lane, below 4096 points)
size_t col_lds_bytes_c128(int ny, int cols, int points) {
  return 2 * row_lds_bytes(ny, cols) + (points != 16 || ny >= 4096 ? 0 : size_t(ny) * 8);
}

int row_rows_per_block(int nx, int ny, int points, size_t max_lds) {
  int rows = 128 * points / nx;  // 256 threads
  if (rows < 1) rows = 1;
  if (rows > ny) rows = ny;
  while (rows > 1 && row_lds_bytes(nx, rows) > max_lds) rows >>= 1;
  return rows;
}

bool col_tile_supported(int nx, int ny, int cols, int iters, int points, size_t max_lds) {
  if (!col_launch_supported(ny, cols, iters, points)) return false;
  if (cols > nx || nx % (cols * iters) != 0) return false;
  return col_lds_bytes(ny, cols) <= max_lds;
}

bool col_cols_supported(int nx, int ny, int cols, int iters, int points, size_t max_lds) {
  return schedule_supported(ny, cols, iters, points) && col_tile_supported(nx, ny, cols, iters, points, max_lds);
}

int col_default_cols(int nx, int ny, int points, size_t max_lds) {
  int c = 128 * points / ny;  // 256 threads
  if (c < 1) c = 1;
  // prefer 64-byte row segments (4 columns) on grids of 2^20 points and with 16 points per lane,
  // 32-byte ones (2 columns) on small grids, while threads and LDS allow it (measured; 4096 x 512 at 8
  // points per lane: 40.7 us per step with 4 columns, 46.2 with 2)
  int want = points == 16 || size_t(nx) * size_t(ny) >= (size_t(1) << 20) ? 4 : 2;
  while (want > c && !col_cols_supported(nx, ny, want, 1, points, max_lds)) want >>= 1;
  if (want > c) c = want;
  while (c > 1 && !col_cols_supported(nx, ny, c, 1, points, max_lds)) c >>= 1;
  return c;
}

// Energy kernels (fp64, register-resident transforms): T = N / points lanes per component of a line, two
// components per lane pair.  16 points per lane from 1024 points on, where a line still fills two waves
// and, at 1024, two lines fit 256 threads and a column block reads 32-byte row segments (us per call with
// 16 and 8: 1024^2 27 and 35, 2048^2 74 and 77, 2048 x 512 35.6 and 36.4); 8 below, for more and shorter
// waves (512^2 19.5 and 18.3).  Lines per workgroup: up to 128 / T (a workgroup of at most 256 threads, 512
// at 4096 points), but no more than keeps ~256 workgroups on the grid (small grids are latency-bound: more
// workgroups, each shorter).
__host__ __device__ constexpr int energy_points(int n) { return n >= 1024 ? 16 : 8; }

size_t energy_lds_bytes(int n, int lines) { return 2 * row_lds_bytes(n, lines); }

static int energy_lines_per_block(int n, int count) {
  const int t = n / energy_points(n);
  return std::max(1, std::min(128 / t, count / 256));
}

int energy_rows_per_block(int nx, int ny) { return energy_lines_per_block(nx, ny); }

int energy_cols_per_block(int nx, int ny, size_t max_lds) {
  int c = energy_lines_per_block(ny, nx);
  while (c > 1 && energy_lds_bytes(ny, c) > max_lds) c >>= 1;
  return c;
}

bool energy_fits(int nx, int ny, size_t max_lds) {
  return energy_lds_bytes(nx, energy_rows_per_block(nx, ny)) <= max_lds &&
         energy_lds_bytes(ny, energy_cols_per_block(nx, ny, max_lds)) <= max_lds;
}

int norm_blocks() { return 256; }

// -------------------------------------------------------------------------------------------
// Energy, in fp64 throughout (it is evaluated on demand, not per step).  The k-space quadratic
// form sum_k psi^(k)^+ H_K(k) psi^(k) of the energy splits, by Parseval's theorem along one axis at
// a time, into 1-D pieces of the state as it is, so no 2-D transform is formed:
//   * the k_x terms (k_x^2 / 2 on both components, k_l k_x sigma_z): for every row, the x-DFT
//     u~(k_x) of the row, sum over k_x; over the whole grid the sum of |u^|^2 f(k_x) is ny times the
//     sum over rows of |u~|^2 f(k_x);
//   * the k_y term (k_y^2 / 2): the same with the y-DFT of every column, times nx;
//   * the uniform Raman term Omega Re(u^* d^) of H_K: N times its real-space sum, so it joins the
//     spatial Raman term Omega(r) Re(u* d) of the real-space energy.
// Row kernel: the real-space terms, the norm and the rows' k_x terms; column kernel: the columns'
// k_y terms.  The DFTs are the step kernels' register-resident forward transform (fwd_pass: radix-P
// stages exchanged through LDS, positions as real_pos and spec_pos give them) instantiated in fp64 on the
// state widened to fp64 as it is loaded, so the energy of a complex64 state carries no transform error of
// its own.  Each lane holds one component of one line.  The
// partials are scaled so that their combination reads E = (w / N ek + w er) / norm
// + w ei norm0 / norm^2 (w = dx dy, N = nx ny), as for a 2-D sum.
// -------------------------------------------------------------------------------------------
extern __shared__ __align__(16) unsigned char energy_lds[];
using EnergyRed = double[kEnergyRedDoubles];
static_assert(sizeof(EnergyRed) <= kStaticLds);

// A result of a reduction, to device memory or to pinned host memory that the host reads once the stream
// is done.
__device__ __forceinline__ void store_partial(double* p, double v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// One component of a state point (Q: float4 for a complex64 state, double4 for complex128).
template <class Q>
using Half = std::conditional_t<sizeof(Q) == sizeof(double4), double2, float2>;

// The lane's component of state point i.
template <class Q>
__device__ __forceinline__ Half<Q> energy_load(const EnergyArgs& a, size_t i, int comp) {
  if constexpr (sizeof(Q) == sizeof(double4)) {
    return reinterpret_cast<const double2*>(a.psi64)[2 * i + comp];
  } else {
    return reinterpret_cast<const float2*>(a.psi)[2 * i + comp];
  }
}

__device__ __forceinline__ int energy_freq(int j, int n) { return j < n / 2 ? j : j - n; }

// Point i of the state.
template <class Q>
__device__ __forceinline__ Q energy_point(const EnergyArgs& a, size_t i) {
  if constexpr (sizeof(Q) == sizeof(double4)) return a.psi64[i];
  else return a.psi[i];
}

// block_sum of four values at once (each in the same order): v is the sums for thread 0; red must hold
// kEnergyRedDoubles.
__device__ __forceinline__ void block_sums(double (&v)[4], double* red) {
  const int n = blockDim.x;
  const bool waves = (n & 63) == 0;   // else a workgroup smaller than one wave (small grids)
  const int parts = waves ? n >> 6 : n, part = waves ? threadIdx.x >> 6 : threadIdx.x;
  if (waves) {
#pragma unroll
    for (double& x : v) x = wave_sum(x);
  }
  if (!waves || (threadIdx.x & 63) == 0) {
#pragma unroll
    for (int k = 0; k < 4; ++k) red[4 * part + k] = v[k];
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
#pragma unroll
  for (double& x : v) x = 0.0;
  for (int p = 0; p < parts; ++p) {
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] += red[4 * p + k];
  }
}

// Rows block*rows .. block*rows + rows - 1 of the state a describes.
template <int N, class Q>
__device__ __forceinline__ void energy_row_body(const EnergyArgs& a, int block, double* red) {
  constexpr int P = energy_points(N);
  constexpr int T = N / P;
  const int tid = threadIdx.x, comp = tid & 1, pair = tid >> 1;
  const int t = pair & (T - 1), r = pair / T;
  const int row = block * a.rows + r;
  const size_t row0 = size_t(row) * N;
  // The real-space terms and the norm: P/2 points per thread with both components in one load, four
  // loads in flight.  At 8 points per lane the transform's loads, which find the row in the L2, go out
  // with them (16 points would hold 250 VGPRs instead of 166).  The roots wait until the sums have given
  // their registers back.  With the four sums in one round of barriers, per energy call: 512^2 20.6 ->
  // 19.6 us, 64^2 17.5 -> 16.9.
  const double y = a.ymin + a.dy * row;
  const double om_row = a.om_y ? a.om_y[row] : 0.0;
  double er = 0.0, ei = 0.0, nr = 0.0;
  const LanePos<T> rp = real_pos<N, P>(t);
  Half<Q> w[P];
  auto load = [&] {
#pragma unroll
    for (int m = 0; m < P; ++m) w[m] = energy_load<Q>(a, row0 + rp.at(m), comp);
  };
#pragma unroll 1
  for (int j0 = tid & (2 * T - 1); j0 < N; j0 += 8 * T) {
    Q q[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) q[i] = energy_point<Q>(a, row0 + j0 + 2 * T * i);
    if constexpr (P == 8) load();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int j = j0 + 2 * T * i;
      const double ux = q[i].x, uy = q[i].y, dx = q[i].z, dy = q[i].w;
      const double x = a.xmin + a.dx * j;
      const double V = a.wx2h * x * x + a.wy2h * y * y;
      const double nu = ux * ux + uy * uy, nd = dx * dx + dy * dy;
      // spatial Raman coupling Omega(r) and the uniform one Omega (its k-space sum, by Parseval)
      const double om = (a.om_x ? a.om_x[j] + om_row : 0.0) + a.omega;
      er += V * (nu + nd) + 0.5 * a.delta * (nu - nd) + om * (ux * dx + uy * dy);
      ei += 0.5 * a.g_uu * nu * nu + 0.5 * a.g_dd * nd * nd + a.g_ud * nu * nd;
      nr += nu + nd;
    }
  }
  int tt = t;
  asm volatile("" : "+v"(tt), "+v"(er), "+v"(ei), "+v"(nr)::"memory");
  if constexpr (P != 8) load();
  double2 v[P];
#pragma unroll
  for (int m = 0; m < P; ++m) v[m] = make_double2(w[m].x, w[m].y);
  TwPlain<N, P, double> tr;
  load_twiddles<N>(tr, tt, a.twx);
  const LdsView<double2> lds = lds_line<N, double2>(energy_lds, r, a.rows, comp);
  fwd_pass<N>(v, lds, tt, tr);
  const LanePos<T> sp = spec_pos<N, P>(tt);
  const double kl = comp == 0 ? a.k_l : -a.k_l;
  double ex = 0.0;   // the rows' k_x terms
#pragma unroll
  for (int m = 0; m < P; ++m) {
    const double kx = energy_freq(sp.at(m), N) * a.dkx;
    ex += (0.5 * kx * kx + kl * kx) * (v[m].x * v[m].x + v[m].y * v[m].y);
  }
  double s[4] = {er, ex, ei, nr};
  block_sums(s, red);
  if (tid == 0) {
    // w / N * (ny * sum) = w * sum / nx: the k_x terms join the real-space linear ones
    a.row_partials[kEnergyRowParts * block] = s[0] + s[1] / double(N);
    a.row_partials[kEnergyRowParts * block + 1] = s[2];
    a.row_partials[kEnergyRowParts * block + 2] = s[3];
  }
}

// Columns of column block `block` (of a.nx / a.cols; the blocks spread over the XCDs as the column
// pass spreads its tiles).
template <int N, class Q>
__device__ __forceinline__ void energy_col_body(const EnergyArgs& a, int block, double* red) {
  constexpr int P = energy_points(N);
  constexpr int T = N / P;
  const int C = a.cols;
  const int tid = threadIdx.x, comp = tid & 1, pair = tid >> 1;
  const int cc = pair & (C - 1), t = pair / C;
  const int x = col_group(block, a.nx / C) * C + cc;
  const LanePos<T> rp = real_pos<N, P>(t), sp = spec_pos<N, P>(t);
  double2 v[P];
#pragma unroll
  for (int m = 0; m < P; ++m) {
    const Half<Q> w = energy_load<Q>(a, size_t(rp.at(m)) * a.nx + x, comp);
    v[m] = make_double2(w.x, w.y);
  }
  TwPlain<N, P, double> tr;
  load_twiddles<N>(tr, t, a.twy);
  const LdsView<double2> lds = lds_line<N, double2>(energy_lds, cc, C, comp);
  fwd_pass<N>(v, lds, t, tr);
  double acc = 0.0;
#pragma unroll
  for (int m = 0; m < P; ++m) {
    const double ky = energy_freq(sp.at(m), N) * a.dky;
    acc += 0.5 * ky * ky * (v[m].x * v[m].x + v[m].y * v[m].y);
  }
  const double s = block_sum(acc, red);
  if (tid == 0) a.col_partials[block] = double(a.nx) * s;   // nx times the columns' sum
}

template <int N, class Q>
__global__ void __launch_bounds__(512) energy_row_kernel(EnergyArgs a) {
  __shared__ EnergyRed red;
  energy_row_body<N, Q>(a, blockIdx.x, red);
}

template <int N, class Q>
__global__ void __launch_bounds__(512) energy_col_kernel(EnergyArgs a) {
  __shared__ double red[kRedDoubles];
  energy_col_body<N, Q>(a, blockIdx.x, red);
}

// Square grids: the row blocks and the column blocks are independent and of one shape, so one launch
// holds both (the first `row_blocks` blocks are the rows').
template <int N, class Q>
__global__ void __launch_bounds__(512) energy_square_kernel(EnergyArgs a, int row_blocks) {
  __shared__ EnergyRed red;
  if (static_cast<int>(blockIdx.x) < row_blocks) energy_row_body<N, Q>(a, blockIdx.x, red);
  else energy_col_body<N, Q>(a, blockIdx.x - row_blocks, red);
}

// Batched: grid y = the members of a batch class, each with its own arguments.
template <int N, class Q>
__global__ void __launch_bounds__(512) energy_row_kernel_batch(const EnergyArgs* __restrict__ tab) {
  __shared__ EnergyRed red;
  const EnergyArgs a = tab[blockIdx.y];
  energy_row_body<N, Q>(a, blockIdx.x, red);
}

template <int N, class Q>
__global__ void __launch_bounds__(512) energy_col_kernel_batch(const EnergyArgs* __restrict__ tab) {
  __shared__ double red[kRedDoubles];
  const EnergyArgs a = tab[blockIdx.y];
  energy_col_body<N, Q>(a, blockIdx.x, red);
}

// The grid's threads over the n points of psi in turn, eight loads of a thread in flight at a time (the
// norm of a 2048^2 grid, 64 MiB in complex64: 22 -> 11 us).  f sees the points in the order of a plain loop.
template <class Q, class F>
__device__ __forceinline__ void for_each_point(const Q* __restrict__ psi, long long n, F f) {
  const long long stride = 256LL * gridDim.x;
  long long i = blockIdx.x * 256LL + threadIdx.x;
  for (; i + 7 * stride < n; i += 8 * stride) {
    Q w[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) w[k] = psi[i + k * stride];
#pragma unroll
    for (int k = 0; k < 8; ++k) f(w[k]);
  }
  for (; i < n; i += stride) f(psi[i]);
}

// -------------------------------------------------------------------------------------------
// Norm: sum |psi|^2 with a fixed grid (deterministic), fp64.
// -------------------------------------------------------------------------------------------
template <class Q>
__global__ void __launch_bounds__(256) norm_kernel(const Q* __restrict__ psi, long long n,
                                                   double* __restrict__ partials) {
  __shared__ double red[kRedDoubles];
  double acc = 0.0;
  for_each_point(psi, n, [&](const Q& w) {
    const double ur = w.x, ui = w.y, dr = w.z, di = w.w;
    acc += ur * ur + ui * ui + dr * dr + di * di;
  });
  const double s = block_sum(acc, red);
  if (threadIdx.x == 0) store_partial(partials + blockIdx.x, s);
}

// One workgroup combines the energy kernels' partials on the device: each kind summed in a fixed
// order (thread-strided, then block_sum's fixed tree), then the energy per particle of the state
// rescaled to norm0, E = (w / N ek + w er) / norm + w ei norm0 / norm^2 with norm = w nr.
__device__ __forceinline__ void energy_finish_body(const EnergyArgs& a, double* out) {
  __shared__ double red[kRedDoubles];
  const int nrows = a.ny / a.rows, ncols = a.nx / a.cols;
  double er = 0.0, ei = 0.0, nr = 0.0, ek = 0.0;
#pragma unroll 4
  for (int b = threadIdx.x; b < nrows; b += blockDim.x) {
    er += a.row_partials[kEnergyRowParts * b];
    ei += a.row_partials[kEnergyRowParts * b + 1];
    nr += a.row_partials[kEnergyRowParts * b + 2];
  }
#pragma unroll 4
  for (int b = threadIdx.x; b < ncols; b += blockDim.x) ek += a.col_partials[b];
  er = block_sum(er, red);
  ei = block_sum(ei, red);
  nr = block_sum(nr, red);
  ek = block_sum(ek, red);
  if (threadIdx.x == 0) {
    const double w = a.dx * a.dy;
    const double nrm = w * nr;
    store_partial(out, (w / (double(a.nx) * double(a.ny)) * ek + w * er) / nrm + w * ei * a.norm0 / (nrm * nrm));
  }
}

__global__ void __launch_bounds__(256) energy_finish_kernel(EnergyArgs a, double* __restrict__ out) {
  energy_finish_body(a, out);
}

__global__ void __launch_bounds__(256) energy_finish_kernel_batch(const EnergyArgs* __restrict__ tab) {
  const EnergyArgs a = tab[blockIdx.x];
  energy_finish_body(a, a.result);
}

hipError_t launch_energy_finish(const EnergyArgs& a, double* out, hipStream_t s) {
  hipLaunchKernelGGL(energy_finish_kernel, dim3(1), dim3(256), 0, s, a, out);
  return hipGetLastError();
}

template <int N>
hipError_t launch_energy_row(const EnergyArgs& a, hipStream_t s) {
  constexpr int T = N / energy_points(N);
  const dim3 grid(a.ny / a.rows), block(2 * T * a.rows);
  const size_t lds = energy_lds_bytes(N, a.rows);
  if (a.psi64) hipLaunchKernelGGL((energy_row_kernel<N, double4>), grid, block, lds, s, a);
  else hipLaunchKernelGGL((energy_row_kernel<N, float4>), grid, block, lds, s, a);
  return hipGetLastError();
}

template <int N>
hipError_t launch_energy_col(const EnergyArgs& a, hipStream_t s) {
  constexpr int T = N / energy_points(N);
  const dim3 grid(a.nx / a.cols), block(2 * T * a.cols);
  const size_t lds = energy_lds_bytes(N, a.cols);
  if (a.psi64) hipLaunchKernelGGL((energy_col_kernel<N, double4>), grid, block, lds, s, a);
  else hipLaunchKernelGGL((energy_col_kernel<N, float4>), grid, block, lds, s, a);
  return hipGetLastError();
}

template <int N>
hipError_t launch_energy_square(const EnergyArgs& a, hipStream_t s) {
  constexpr int T = N / energy_points(N);
  const int rows = N / a.rows;
  const dim3 grid(rows + N / a.cols), block(2 * T * a.rows);
  const size_t lds = energy_lds_bytes(N, a.rows);
  if (a.psi64) hipLaunchKernelGGL((energy_square_kernel<N, double4>), grid, block, lds, s, a, rows);
  else hipLaunchKernelGGL((energy_square_kernel<N, float4>), grid, block, lds, s, a, rows);
  return hipGetLastError();
}

hipError_t launch_energy(const EnergyArgs& a, hipStream_t s) {
  // one launch instead of two (22.6 -> 18.5 us per call at 256^2, 38 -> 32 at 1024^2); 4096^2 keeps two
  // (its rows and columns fill the device many times over)
  if (a.nx == a.ny && a.rows == a.cols) {
    switch (a.nx) {
      case 16: return launch_energy_square<16>(a, s);
      case 32: return launch_energy_square<32>(a, s);
      case 64: return launch_energy_square<64>(a, s);
      case 128: return launch_energy_square<128>(a, s);
      case 256: return launch_energy_square<256>(a, s);
      case 512: return launch_energy_square<512>(a, s);
      case 1024: return launch_energy_square<1024>(a, s);
      case 2048: return launch_energy_square<2048>(a, s);
      default: break;
    }
  }
  hipError_t e = hipErrorInvalidValue;
  switch (a.nx) {
    case 16: e = launch_energy_row<16>(a, s); break;
    case 32: e = launch_energy_row<32>(a, s); break;
    case 64: e = launch_energy_row<64>(a, s); break;
    case 128: e = launch_energy_row<128>(a, s); break;
    case 256: e = launch_energy_row<256>(a, s); break;
    case 512: e = launch_energy_row<512>(a, s); break;
    case 1024: e = launch_energy_row<1024>(a, s); break;
    case 2048: e = launch_energy_row<2048>(a, s); break;
    case 4096: e = launch_energy_row<4096>(a, s); break;
    default: break;
  }
  if (e != hipSuccess) return e;
  switch (a.ny) {
    case 16: return launch_energy_col<16>(a, s);
    case 32: return launch_energy_col<32>(a, s);
    case 64: return launch_energy_col<64>(a, s);
    case 128: return launch_energy_col<128>(a, s);
    case 256: return launch_energy_col<256>(a, s);
    case 512: return launch_energy_col<512>(a, s);
    case 1024: return launch_energy_col<1024>(a, s);
    case 2048: return launch_energy_col<2048>(a, s);
    case 4096: return launch_energy_col<4096>(a, s);
    default: return hipErrorInvalidValue;
  }
}

template <int N>
hipError_t launch_energy_row_batch(const EnergyArgs* tab, int count, int ny, int rows, hipStream_t s) {
  constexpr int T = N / energy_points(N);
  hipLaunchKernelGGL((energy_row_kernel_batch<N, float4>), dim3(ny / rows, count), dim3(2 * T * rows),
                     energy_lds_bytes(N, rows), s, tab);
  return hipGetLastError();
}

template <int N>
hipError_t launch_energy_col_batch(const EnergyArgs* tab, int count, int nx, int cols, hipStream_t s) {
  constexpr int T = N / energy_points(N);
  hipLaunchKernelGGL((energy_col_kernel_batch<N, float4>), dim3(nx / cols, count), dim3(2 * T * cols),
                     energy_lds_bytes(N, cols), s, tab);
  return hipGetLastError();
}

hipError_t launch_energy_batch(const EnergyArgs* tab, int count, int nx, int ny, int rows, int cols, hipStream_t s) {
  hipError_t e = hipErrorInvalidValue;
  switch (nx) {
    case 16: e = launch_energy_row_batch<16>(tab, count, ny, rows, s); break;
    case 32: e = launch_energy_row_batch<32>(tab, count, ny, rows, s); break;
    case 64: e = launch_energy_row_batch<64>(tab, count, ny, rows, s); break;
    case 128: e = launch_energy_row_batch<128>(tab, count, ny, rows, s); break;
    case 256: e = launch_energy_row_batch<256>(tab, count, ny, rows, s); break;
    case 512: e = launch_energy_row_batch<512>(tab, count, ny, rows, s); break;
    case 1024: e = launch_energy_row_batch<1024>(tab, count, ny, rows, s); break;
    case 2048: e = launch_energy_row_batch<2048>(tab, count, ny, rows, s); break;
    case 4096: e = launch_energy_row_batch<4096>(tab, count, ny, rows, s); break;
    default: break;
  }
  if (e != hipSuccess) return e;
  switch (ny) {
    case 16: e = launch_energy_col_batch<16>(tab, count, nx, cols, s); break;
    case 32: e = launch_energy_col_batch<32>(tab, count, nx, cols, s); break;
    case 64: e = launch_energy_col_batch<64>(tab, count, nx, cols, s); break;
    case 128: e = launch_energy_col_batch<128>(tab, count, nx, cols, s); break;
    case 256: e = launch_energy_col_batch<256>(tab, count, nx, cols, s); break;
    case 512: e = launch_energy_col_batch<512>(tab, count, nx, cols, s); break;
    case 1024: e = launch_energy_col_batch<1024>(tab, count, nx, cols, s); break;
    case 2048: e = launch_energy_col_batch<2048>(tab, count, nx, cols, s); break;
    case 4096: e = launch_energy_col_batch<4096>(tab, count, nx, cols, s); break;
    default: e = hipErrorInvalidValue; break;
  }
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(energy_finish_kernel_batch, dim3(count), dim3(256), 0, s, tab);
  return hipGetLastError();
}

// Count of non-finite values per workgroup (as doubles, in the norm's partial buffer): the check of a
// state handed over in device memory.
template <class Q>
__global__ void __launch_bounds__(256) nonfinite_kernel(const Q* __restrict__ psi, long long n,
                                                        double* __restrict__ partials) {
  __shared__ double red[kRedDoubles];
  double bad = 0.0;
  for_each_point(psi, n, [&](const Q& w) {
    bad += (isfinite(w.x) && isfinite(w.y) && isfinite(w.z) && isfinite(w.w)) ? 0.0 : 1.0;
  });
  const double s = block_sum(bad, red);
  if (threadIdx.x == 0) store_partial(partials + blockIdx.x, s);
}

hipError_t launch_nonfinite(const float4* psi, long long npts, double* partials, int nblocks, hipStream_t s) {
  hipLaunchKernelGGL(nonfinite_kernel<float4>, dim3(nblocks), dim3(256), 0, s, psi, npts, partials);
  return hipGetLastError();
}

hipError_t launch_nonfinite(const double4* psi, long long npts, double* partials, int nblocks, hipStream_t s) {
  hipLaunchKernelGGL(nonfinite_kernel<double4>, dim3(nblocks), dim3(256), 0, s, psi, npts, partials);
  return hipGetLastError();
}

hipError_t launch_norm(const float4* psi, long long npts, double* partials, int nblocks, hipStream_t s) {
  hipLaunchKernelGGL(norm_kernel<float4>, dim3(nblocks), dim3(256), 0, s, psi, npts, partials);
  return hipGetLastError();
}

hipError_t launch_norm(const double4* psi, long long npts, double* partials, int nblocks, hipStream_t s) {
  hipLaunchKernelGGL(norm_kernel<double4>, dim3(nblocks), dim3(256), 0, s, psi, npts, partials);
  return hipGetLastError();
}

}  // namespace sgpe
