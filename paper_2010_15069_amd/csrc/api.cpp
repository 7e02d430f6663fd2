// Host side of the split-step solver: parameter validation, fp64 construction of the operator
// and twiddle tables, the fused step schedule, and the C ABI declared in include/sgpe.h.
#include "sgpe.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <type_traits>
#include <cstring>
#include <new>
#include <vector>

#include "host_internal.hpp"
#include "sgpe_internal.hpp"

using sgpe::ColArgs;
using sgpe::EnergyArgs;
using sgpe::RowArgs;

namespace {

constexpr int kMinN = 16;
constexpr int kMaxN = 4096;

bool is_pow2(int32_t n) { return n > 0 && (n & (n - 1)) == 0; }
bool is_finite(double v) { return std::isfinite(v); }

}  // namespace


namespace sgpe_host {

inline float4 mk4(double a, double b, double c, double d, float) { return make_float4(float(a), float(b), float(c), float(d)); }
inline double4 mk4(double a, double b, double c, double d, double) { return make_double4(a, b, c, d); }
inline float2 mk2h(double a, double b, float) { return make_float2(float(a), float(b)); }
inline double2 mk2h(double a, double b, double) { return make_double2(a, b); }

sgpe_status dev_alloc(sgpe_ctx* c, void** ptr, size_t bytes) {
  *ptr = nullptr;
  if (hipMalloc(ptr, bytes) != hipSuccess) {
    (void)hipGetLastError();
    *ptr = nullptr;
    return SGPE_ENOMEM;
  }
  c->allocations.push_back(*ptr);
  return SGPE_OK;
}

template <class T>
sgpe_status upload(sgpe_ctx* c, T** dst, const std::vector<T>& host) {
  void* p = nullptr;
  sgpe_status st = dev_alloc(c, &p, host.size() * sizeof(T));
  if (st != SGPE_OK) return st;
  if (hipMemcpy(p, host.data(), host.size() * sizeof(T), hipMemcpyHostToDevice) != hipSuccess) {
    (void)hipGetLastError();
    return SGPE_EDEVICE;
  }
  *dst = static_cast<T*>(p);
  return SGPE_OK;
}

// Tables of the spatial Raman coupling Omega_x(x_j) + Omega_y(y_i) (Eq. (H4) with Omega(r)): the
// step kernels' half-angles dt Omega / 2 in fp32 and the energy kernel's Omega in fp64.  NULL
// stands for a zero profile.  Allocated on first use, overwritten in place afterwards.
sgpe_status raman_tables(sgpe_ctx* c, const double* om_x, const double* om_y) {
  const sgpe_params& p = c->p;
  sgpe_status st;
  void* ptr = nullptr;
  if (c->prec == SGPE_C128 && !c->hbx64) {
    if ((st = dev_alloc(c, &ptr, size_t(p.nx) * sizeof(double))) != SGPE_OK) return st;
    c->hbx64 = static_cast<double*>(ptr);
    if ((st = dev_alloc(c, &ptr, size_t(p.ny) * sizeof(double))) != SGPE_OK) return st;
    c->hby64 = static_cast<double*>(ptr);
  }
  if (!c->hbx) {
    if ((st = dev_alloc(c, &ptr, size_t(p.nx) * sizeof(float))) != SGPE_OK) return st;
    c->hbx = static_cast<float*>(ptr);
    if ((st = dev_alloc(c, &ptr, size_t(p.ny) * sizeof(float))) != SGPE_OK) return st;
    c->hby = static_cast<float*>(ptr);
    if ((st = dev_alloc(c, &ptr, size_t(p.nx) * sizeof(double))) != SGPE_OK) return st;
    c->omx = static_cast<double*>(ptr);
    if ((st = dev_alloc(c, &ptr, size_t(p.ny) * sizeof(double))) != SGPE_OK) return st;
    c->omy = static_cast<double*>(ptr);
  }
  std::vector<double> ox(p.nx, 0.0), oy(p.ny, 0.0);
  if (om_x) ox.assign(om_x, om_x + p.nx);
  if (om_y) oy.assign(om_y, om_y + p.ny);
  std::vector<float> hx(p.nx), hy(p.ny);
  std::vector<double> hx64(p.nx), hy64(p.ny);
  for (int j = 0; j < p.nx; ++j) hx64[j] = 0.5 * p.dt * ox[j], hx[j] = float(hx64[j]);
  for (int i = 0; i < p.ny; ++i) hy64[i] = 0.5 * p.dt * oy[i], hy[i] = float(hy64[i]);
  if (c->prec == SGPE_C128 &&
      (hipStreamSynchronize(c->stream) != hipSuccess ||
       hipMemcpy(c->hbx64, hx64.data(), hx64.size() * sizeof(double), hipMemcpyHostToDevice) != hipSuccess ||
       hipMemcpy(c->hby64, hy64.data(), hy64.size() * sizeof(double), hipMemcpyHostToDevice) != hipSuccess)) {
    (void)hipGetLastError();
    return SGPE_EDEVICE;
  }
  // the stream's queued steps may still read the old tables
  if (hipStreamSynchronize(c->stream) != hipSuccess ||
      hipMemcpy(c->hbx, hx.data(), hx.size() * sizeof(float), hipMemcpyHostToDevice) != hipSuccess ||
      hipMemcpy(c->hby, hy.data(), hy.size() * sizeof(float), hipMemcpyHostToDevice) != hipSuccess ||
      hipMemcpy(c->omx, ox.data(), ox.size() * sizeof(double), hipMemcpyHostToDevice) != hipSuccess ||
      hipMemcpy(c->omy, oy.data(), oy.size() * sizeof(double), hipMemcpyHostToDevice) != hipSuccess) {
    (void)hipGetLastError();
    return SGPE_EDEVICE;
  }
  return SGPE_OK;
}

// Root table of a transform of length n: (tan(phi / 2), sin(phi)) of phi = 2 pi j / n at entry j + n/4,
// |j| <= n/4 -- the shears of a rotation by phi (see "Step-kernel transforms" in fft_device.hpp), each
// rounded once to T.
template <class T = float>
std::vector<sgpe::cplx_t<T>> root_table(int n) {
  std::vector<sgpe::cplx_t<T>> t(n / 2 + 1);
  for (int j = -n / 4; j <= n / 4; ++j) {
    const double a = 2.0 * M_PI * double(j) / double(n);
    t[j + n / 4] = mk2h(std::tan(0.5 * a), std::sin(a), T());
  }
  return t;
}

// FFT-ordered angular wave numbers: 2 pi fftfreq(n, d).
double kval(int j, int n, double d) {
  const int m = j < n / 2 ? j : j - n;
  return 2.0 * M_PI * double(m) / (double(n) * d);
}

// k-space 2x2 propagator factored as P(k_y) M'(k_x) with
//   M'(k_x) = e^{-h kx^2/2 (i)} [ c 1 - s (b . sigma) ],  b = (omega/2, k_l k_x),
//   P(k_y)  = e^{-h ky^2/2 (i)};
// stored as M' - 1 (per component its row, {own, other}) and P - 1, to relative accuracy.  Real time:
// complex entries, times the 1/nx and 1/ny of the line passes' inverse transforms (powers of two).
template <class T = float>
void k_tables_real(const sgpe_params& p, double h, std::vector<sgpe::point_t<T>>& kx_out,
                   std::vector<sgpe::cplx_t<T>>& ky_out) {
  const double dx = 2.0 * p.xmax / p.nx, dy = 2.0 * p.ymax / p.ny;
  kx_out.assign(2 * size_t(p.nx), mk4(0, 0, 0, 0, T()));
  ky_out.assign(size_t(p.ny), mk2h(0, 0, T()));
  for (int j = 0; j < p.nx; ++j) {
    const double kx = kval(j, p.nx, dx);
    const double bx = 0.5 * p.omega, bz = p.k_l * kx;
    const double bm = std::hypot(bx, bz);
    const double al = 0.5 * h * kx * kx;
    const double c = std::cos(h * bm);
    const double s = bm > 0.0 ? std::sin(h * bm) / bm : h;
    const double pr = std::cos(al), pi = -std::sin(al);
    // pref * (c - i s bz), pref * (-i s bx), pref * (c + i s bz)
    const double m11r = pr * c + pi * s * bz, m11i = pi * c - pr * s * bz;
    const double m12r = pi * s * bx, m12i = -pr * s * bx;
    const double m22r = pr * c - pi * s * bz, m22i = pi * c + pr * s * bz;
    // per component: {d_own, d_other} of its row of M' - 1 (up: d11, d12; down: d22, d21)
    const double w = 1.0 / p.nx;
    kx_out[2 * size_t(j)] = mk4(w * (m11r - 1.0), w * m11i, w * m12r, w * m12i, T());
    kx_out[2 * size_t(j) + 1] = mk4(w * (m22r - 1.0), w * m22i, w * m12r, w * m12i, T());
  }
  for (int i = 0; i < p.ny; ++i) {
    const double ky = kval(i, p.ny, dy);
    const double be = 0.5 * h * ky * ky;
    const double sh = std::sin(0.5 * be);
    const double w = 1.0 / p.ny;
    ky_out[i] = mk2h(-2.0 * w * sh * sh, -w * std::sin(be), T());
  }
}

// Imaginary time: the same with hyperbolic functions, all entries real.
template <class T = float>
void k_tables_imag(const sgpe_params& p, double h, std::vector<sgpe::cplx_t<T>>& kx_out, std::vector<T>& ky_out) {
  const double dx = 2.0 * p.xmax / p.nx, dy = 2.0 * p.ymax / p.ny;
  kx_out.assign(2 * size_t(p.nx), mk2h(0, 0, T()));
  ky_out.assign(size_t(p.ny), T(0));
  for (int j = 0; j < p.nx; ++j) {
    const double kx = kval(j, p.nx, dx);
    const double bx = 0.5 * p.omega, bz = p.k_l * kx;
    const double bm = std::hypot(bx, bz);
    const double ch = std::cosh(h * bm);
    const double sh = bm > 0.0 ? std::sinh(h * bm) / bm : h;
    const double pr = std::exp(-0.5 * h * kx * kx);
    kx_out[2 * size_t(j)] = mk2h(pr * (ch - sh * bz) - 1.0, -pr * sh * bx, T());
    kx_out[2 * size_t(j) + 1] = mk2h(pr * (ch + sh * bz) - 1.0, -pr * sh * bx, T());
  }
  for (int i = 0; i < p.ny; ++i) {
    const double ky = kval(i, p.ny, dy);
    ky_out[i] = T(std::expm1(-0.5 * h * ky * ky));
  }
}

// Default points per lane for lines of length n (from measured sweeps on MI355X; us per step).  More
// points per lane are fewer instructions per point and fewer waves.
// * 4 on small grids, where a pass is one lane's chain of latencies: rows below 2^18 points, columns
//   below 2^17 (8 instances of 128^2: 12.0 imaginary / 8.1 real with 4 and 8, 12.8 / 9.8 with 8 and 8).
// * 8 below 2^20 points (1024 x 512: 15.6 / 11.0 with 8, 17.9 / 13.2 with 16; 512 x 1024: 18.4 / 12.2
//   against 20.3 / 14.7).
// * From there 16 on long lines (1024^2: 23.3 / 16.4; 8 and 8: 26.4 / 18.4), 8 on rows up to 256 points
//   (256 x 2048: 24.2 / 16.5 against 25.1 / 17.6) and columns up to 512 (2048 x 256: 16.3 / 11.8
//   against 17.1 / 12.8; 8 instances of 512^2: 37.1 / 29.8 against 38.1 / 33.2), whose shorter
//   transforms hold fewer registers at 8 without a third exchange more.
// Row prefetching (two row groups per workgroup) pays only for small rows whose one-group grid is a
// single round of resident workgroups (two per compute unit): then nothing else would overlap the first
// loads and last stores.  Column prefetching needs the narrower tile and measured slower everywhere; it
// stays off by default.
int default_points(int n, size_t npts, bool col) {
  if (n > sgpe::kMaxNSmallP) return 16;
  if (npts < (size_t(1) << (col ? 17 : 18))) return 4;
  if (npts < (size_t(1) << 20)) return 8;
  return n <= (col ? 512 : 256) ? 8 : 16;
}

// The default column tile from one of at most 512 threads: twice that where such a tile of 2048- or
// 4096-point columns fills its workgroup with a row segment of only 32 or 16 bytes, the wider tile fits
// the LDS, and one workgroup per compute unit is left.  The pass holds its registers at the four waves per
// SIMD of 1024 threads (90 VGPRs), so the same waves are resident and the segments are twice as long
// (per step, imaginary / real time: 2048^2 79.8 / 64.6 -> 73.1 / 56.8 us, 1024 x 4096 126 / 79 -> 94 / 70,
// 512 x 4096 67.8 / 44.2 -> 54.7 / 40.1).
int wide_cols(const sgpe_ctx* c, int cols, int points) {
  const int nx = c->p.nx, ny = c->p.ny;
  return 2 * cols * (ny / points) == 512 && nx / (2 * cols) >= c->n_cu &&
                 sgpe::col_tile_supported(nx, ny, 2 * cols, 1, points, c->max_lds)
             ? 2 * cols
             : cols;
}

void default_schedule(sgpe_ctx* c) {
  const int nx = c->p.nx, ny = c->p.ny;
  const size_t npts = size_t(nx) * size_t(ny);
  c->row_points = default_points(nx, npts, false);
  c->col_points = default_points(ny, npts, true);
  c->rows = sgpe::row_rows_per_block(nx, ny, c->row_points, c->max_lds);
  c->cols = sgpe::col_default_cols(nx, ny, c->col_points, c->max_lds);
  c->row_iters = 1;
  c->col_iters = 1;
  // Column tiles: as many workgroups as compute units, up to one per CU, where that tile is
  // supported (measured: 1 column at 128^2 and 256^2, -9 % and -4 % per step; 512^2-1024^2 already
  // have one per CU; at 2048^2 it would take 2048 threads).
  {
    const int cc = std::max(1, nx / c->n_cu);
    if ((cc & (cc - 1)) == 0 && sgpe::col_cols_supported(nx, ny, cc, 1, c->col_points, c->max_lds)) c->cols = cc;
  }
  c->cols = wide_cols(c, c->cols, c->col_points);
  // One row per workgroup where a row takes at least two waves (measured at 256^2-2048^2: fastest,
  // or within 1 % at 512^2; one 4-row workgroup per CU was 8 % slower per step at 1024^2 and row
  // prefetch slower everywhere).  Smaller rows keep the derived tile.
  if (nx / c->row_points >= 64 && sgpe::schedule_supported(nx, 1, 1, c->row_points) &&
      sgpe::row_lds_bytes(nx, 1) <= c->max_lds) {
    c->rows = 1;
    return;
  }
  const int groups = ny / c->rows;
  if (c->row_points == 16 && groups == 2 * c->n_cu && sgpe::schedule_supported(nx, c->rows, 2, 16))
    c->row_iters = 2;
}

int col_groups(const sgpe_ctx* c) { return c->p.nx / (c->cols * c->col_iters); }

// Columns per workgroup of a real-time pass along columns: the schedule's tile, or half of it where that
// takes more than the 512 threads of a pass with a spatial coupling (line_threads).
static int line_cols(const sgpe_ctx* c) {
  return c->full2x2 && 2 * c->cols * (c->p.ny / c->col_points) > 512 ? c->cols / 2 : c->cols;
}

sgpe_status apply_schedule(sgpe_ctx* c, const sgpe_schedule& s) {
  const sgpe_params& p = c->p;
  if (s.row_points != 4 && s.row_points != 8 && s.row_points != 16) return SGPE_EINVAL;
  if (s.col_tile < 1) return SGPE_EINVAL;
  if (s.row_tile < 0) return SGPE_EINVAL;
  const int rows = s.row_tile > 0 ? s.row_tile : sgpe::row_rows_per_block(p.nx, p.ny, s.row_points, c->max_lds);
  if (rows > p.ny || !sgpe::schedule_supported(p.nx, rows, s.row_iters, s.row_points) ||
      p.ny % (rows * s.row_iters) != 0 ||
      sgpe::row_lds_bytes(p.nx, rows) > c->max_lds)
    return SGPE_EINVAL;
  if (!sgpe::col_tile_supported(p.nx, p.ny, s.col_tile, s.col_iters, s.col_points, c->max_lds)) return SGPE_EINVAL;
  c->rows = rows;
  c->cols = s.col_tile;
  c->row_iters = s.row_iters;
  c->col_iters = s.col_iters;
  c->row_points = s.row_points;
  c->col_points = s.col_points;
  return SGPE_OK;
}

sgpe_schedule get_schedule(const sgpe_ctx* c) {
  sgpe_schedule s{};
  s.col_tile = c->cols;
  s.row_tile = c->rows;
  s.row_iters = c->row_iters;
  s.col_iters = c->col_iters;
  s.row_points = c->row_points;
  s.col_points = c->col_points;
  return s;
}

sgpe_status status_of(hipError_t e) {
  if (e == hipSuccess) return SGPE_OK;
  if (e == hipErrorOutOfMemory || e == hipErrorMemoryAllocation) return SGPE_ENOMEM;
  return SGPE_EDEVICE;
}

template <class T>
sgpe::RowArgsT<T> row_args_t(const sgpe_ctx* c, double h_sub) {
  const sgpe_params& p = c->p;
  sgpe::RowArgsT<T> a{};
  if constexpr (std::is_same<T, double>::value) {
    a.psi = c->psi64;
    a.tw = c->twp64_x;
    a.hbx = c->hbx64;
    a.hby = c->hby64;
  } else {
    a.psi = c->psi;
    a.tw = c->twp_x;
    a.hbx = c->hbx;
    a.hby = c->hby;
  }
  a.nx = p.nx;
  a.ny = p.ny;
  a.rows_per_block = c->rows;
  a.scale = T(1);
  a.partials = nullptr;
  a.n_partials = 0;
  const double dx = 2.0 * p.xmax / p.nx, dy = 2.0 * p.ymax / p.ny;
  const double npts = double(p.nx) * double(p.ny);
  a.norm0 = p.norm0;
  a.parseval_w = dx * dy / npts;
  a.inv_npts = 1.0 / npts;
  a.x0 = T(-p.xmax);
  a.dx = T(dx);
  a.y0 = T(-p.ymax);
  a.dy = T(dy);
  const double h = h_sub > 0.0 ? h_sub : p.dt;
  a.hfrac = T(h / p.dt);
  a.hvx = T(0.5 * h * p.wx * p.wx);
  a.hvy = T(0.5 * h * p.wy * p.wy);
  a.hdelta2 = T(0.5 * h * p.delta);
  a.hg_uu = T(h * p.g_uu);
  a.hg_dd = T(h * p.g_dd);
  a.hg_ud = T(h * p.g_ud);
  a.nonfinite = c->status_dev;
  return a;
}

RowArgs row_args(const sgpe_ctx* c, double h_sub) { return row_args_t<float>(c, h_sub); }

template <class T>
sgpe::ColArgsT<T> col_args_t(const sgpe_ctx* c, bool half) {
  sgpe::ColArgsT<T> a{};
  if constexpr (std::is_same<T, double>::value) {
    a.psi = c->psi64;
    a.tw = c->twp64_y;
    a.kx_tab = c->kx64_imag[half];
    a.ky_tab = c->ky64_imag[half];
  } else {
    a.psi = c->psi;
    a.tw = c->twp_y;
    a.kx_tab = c->kx_imag[half];
    a.ky_tab = c->ky_imag[half];
  }
  a.nx = c->p.nx;
  a.ny = c->p.ny;
  a.cols = c->cols;
  a.partials = c->partials;
  return a;
}

ColArgs col_args(const sgpe_ctx* c, bool half) { return col_args_t<float>(c, half); }

// Line-pass arguments along columns (col) or rows with ops of K(pre), K(post) (LineOp) and n_r real-space
// sub-steps R(h_sub) (h_sub <= 0: dt).  x is the axis along the line.
template <class T>
sgpe::LineArgsT<T> line_args_t(const sgpe_ctx* c, bool col, LineOp pre, LineOp post, int n_r, double h_sub) {
  const sgpe_params& p = c->p;
  const sgpe::RowArgsT<T> r = row_args_t<T>(c, h_sub);
  sgpe::LineArgsT<T> a{};
  a.psi = r.psi;
  a.nx = p.nx;
  a.lines = col ? line_cols(c) : c->rows;
  auto op = [&](LineOp o) -> const void* {
    if (o == LINE_NONE) return nullptr;
    const bool half = o == LINE_HALF;
    if constexpr (std::is_same<T, double>::value)
      return col ? static_cast<const void*>(c->ky64_real[half]) : static_cast<const void*>(c->kx64_real[half]);
    else
      return col ? static_cast<const void*>(c->ky_real[half]) : static_cast<const void*>(c->kx_real[half]);
  };
  a.op_pre = op(pre);
  a.op_post = op(post);
  a.n_r = n_r;
  a.hfrac = r.hfrac;
  a.hdelta2 = r.hdelta2;
  a.hg_uu = r.hg_uu;
  a.hg_dd = r.hg_dd;
  a.hg_ud = r.hg_ud;
  a.tw = col ? col_args_t<T>(c, false).tw : r.tw;
  a.x0 = col ? r.y0 : r.x0;
  a.dx = col ? r.dy : r.dx;
  a.y0 = col ? r.x0 : r.y0;
  a.dy = col ? r.dx : r.dy;
  a.hvx = col ? r.hvy : r.hvx;
  a.hvy = col ? r.hvx : r.hvy;
  a.hbx = col ? r.hby : r.hbx;
  a.hby = col ? r.hbx : r.hby;
  return a;
}

sgpe::LineArgs line_args(const sgpe_ctx* c, bool col, LineOp pre, LineOp post, int n_r, double h_sub) {
  return line_args_t<float>(c, col, pre, post, n_r, h_sub);
}

// One line pass of the context on its stream.
static hipError_t line_pass(const sgpe_ctx* c, bool col, LineOp pre, LineOp post, int n_r, double h_sub = 0.0) {
  const int n = col ? c->p.ny : c->p.nx, n_lines = col ? c->p.nx : c->p.ny;
  const int points = col ? c->col_points : c->row_points;
  if (c->prec == SGPE_C128)
    return sgpe::launch_line(line_args_t<double>(c, col, pre, post, n_r, h_sub), n, n_lines, col, c->full2x2, points,
                             c->stream);
  return sgpe::launch_line(line_args_t<float>(c, col, pre, post, n_r, h_sub), n, n_lines, col, c->full2x2,
                           c->split_rs == SGPE_RSPLIT_NLN, points, c->stream);
}

// n real-time steps K(dt/2) R K(dt/2) in n + 2 sweeps (see line_launch.hpp), either precision and either
// real-space split.  A context on its own state stops after the last R, which leaves K(dt/2) pending
// (tail_pending, tail_col): a call that continues starts with the pending axis's op of the merged K(dt)
// alone, and its passes go on from the other axis, so that calls of n1 and n2 steps do the arithmetic
// of one call of n1 + n2.  With ev, a HIP event pair around the leading pass and each of the n others.
static sgpe_status run_steps_real(sgpe_ctx* c, int64_t n, std::vector<hipEvent_t>* ev) {
  if (c->tail_pending != 0 && (c->tail_pending != 1 || ev)) {
    const sgpe_status st = flush_tail(c);
    if (st != SGPE_OK) return st;
  }
  size_t evi = 0;
  auto mark = [&] {
    if (ev) (void)hipEventRecord((*ev)[evi++], c->stream);
  };
  const bool cont = c->tail_pending == 1;
  const bool defer = c->own_psi && !ev;
  bool col = cont && c->tail_col;
  c->tail_pending = 0;
  mark();
  hipError_t e = line_pass(c, col, cont ? LINE_FULL : LINE_HALF, LINE_NONE, 0);
  mark();
  for (int64_t i = 1; i <= n && e == hipSuccess; ++i) {
    col = !col;
    const bool last = i == n;
    mark();
    e = line_pass(c, col, (i == 1 && !cont) ? LINE_HALF : LINE_FULL, !last ? LINE_FULL : defer ? LINE_NONE : LINE_HALF,
                  1);
    mark();
  }
  if (e != hipSuccess) return status_of(e);
  if (defer) {
    c->tail_pending = 1;
    c->tail_col = col;
    return SGPE_OK;
  }
  return status_of(line_pass(c, !col, LINE_HALF, LINE_NONE, 0));
}

// The fused imaginary-time schedule on a complex128 state: the same sequence of passes as run_steps,
// with the fp64 instantiations of the kernels (16 or 8 points per lane, no prefetch).
static sgpe_status run_steps_c128(sgpe_ctx* c, int64_t n) {
  const double npts = double(c->p.nx) * double(c->p.ny);
  hipStream_t s = c->stream;
  sgpe::RowArgsT<double> ra = row_args_t<double>(c, 0.0);
  // a pending imaginary-time tail continues as in run_steps; a real-time one completes first
  if (c->tail_pending == 1) {
    const sgpe_status st = flush_tail(c);
    if (st != SGPE_OK) return st;
  }
  const bool cont = c->tail_pending == 2;
  c->tail_pending = 0;
  hipError_t e;
  if (cont) {
    e = sgpe::launch_col(col_args_t<double>(c, false), sgpe::NORM_DOT, c->col_points, s);
  } else {
    e = sgpe::launch_row(ra, sgpe::ROW_FWD, false, c->row_points, s);
    if (e == hipSuccess) e = sgpe::launch_col(col_args_t<double>(c, true), sgpe::NORM_NONE, c->col_points, s);
  }
  const bool defer = c->own_psi;
  for (int64_t i = 1; i <= n && e == hipSuccess; ++i) {
    sgpe::RowArgsT<double> r = ra;
    r.scale = 1.0 / npts;
    if (i > 1 || cont) {
      r.partials = c->partials;
      r.n_partials = col_groups(c);
    }
    e = sgpe::launch_row(r, sgpe::ROW_STEP, c->full2x2, c->row_points, s);
    const bool last = (i == n);
    if (last && defer) break;   // the last K(dt/2) and the inverse x-transform wait (flush_tail)
    if (e == hipSuccess)
      e = sgpe::launch_col(col_args_t<double>(c, last), last ? sgpe::NORM_SQ : sgpe::NORM_DOT, c->col_points, s);
  }
  if (e == hipSuccess && defer) {
    c->tail_pending = 2;
    return SGPE_OK;
  }
  if (e == hipSuccess) {
    sgpe::RowArgsT<double> r = ra;
    r.scale = 1.0 / npts;
    r.partials = c->partials;
    r.n_partials = col_groups(c);
    e = sgpe::launch_row(r, sgpe::ROW_INV, false, c->row_points, s);
  }
  return status_of(e);
}

// The fused imaginary-time schedule of n steps: K(dt/2) [R K(dt)]^(n-1) R K(dt/2), with the
// normalisation of step i applied (as a scale) at the start of the next row pass.
static sgpe_status run_steps_variant(sgpe_ctx* c, int64_t n, bool imag);

sgpe_status run_steps(sgpe_ctx* c, int64_t n, bool imag, std::vector<hipEvent_t>* ev) {
  if (n == 0) return SGPE_OK;
  const bool rkr = c->split_order != SGPE_SPLIT_KRK;
  const bool nln = c->split_rs != SGPE_RSPLIT_FROZEN;
  if (ev && (rkr || nln || c->prec == SGPE_C128)) return SGPE_ESTATE;
  if (rkr) {
    // R-K-R completes every call; a tail of K-R-K completes first
    const sgpe_status st = flush_tail(c);
    if (st != SGPE_OK) return st;
    return run_steps_variant(c, n, imag);
  }
  if (!imag) return run_steps_real(c, n, ev);
  if (c->prec == SGPE_C128) return run_steps_c128(c, n);
  // K-R-K with R = N L N differs from the default only inside the row pass's R
  const int step_mode = nln ? sgpe::ROW_STEP_NLN : sgpe::ROW_STEP;
  const double npts = double(c->p.nx) * double(c->p.ny);
  const float inv_n = float(1.0 / npts);  // exact: a power of two
  hipStream_t s = c->stream;
  hipError_t e;
  RowArgs ra = row_args(c);
  // A real-time tail (or any tail before a timed profile) completes first.  An imaginary-time one
  // continues: the merged K(dt) below completes the previous call's last step and begins this
  // call's first, exactly as inside one call (its NORM_DOT partials give the norm at that step
  // boundary, and the first row pass rescales by it).
  if (c->tail_pending != 0 && (c->tail_pending != 2 || ev)) {
    const sgpe_status st = flush_tail(c);
    if (st != SGPE_OK) return st;
  }
  const bool cont = c->tail_pending == 2;
  c->tail_pending = 0;
  if (cont) {
    e = sgpe::launch_col(col_args(c, false), sgpe::NORM_DOT, c->col_iters, c->col_points, s);
  } else {
    e = sgpe::launch_row(ra, sgpe::ROW_FWD, false, c->row_iters, c->row_points, s);
    if (e == hipSuccess)
      e = sgpe::launch_col(col_args(c, true), sgpe::NORM_NONE, c->col_iters, c->col_points, s);
  }
  if (e != hipSuccess) return status_of(e);
  // a context on a caller's state buffer, and a timed profile, complete every call
  const bool defer = c->own_psi && !ev;
  size_t evi = 0;
  for (int64_t i = 1; i <= n; ++i) {
    RowArgs r = ra;
    r.scale = inv_n;
    if (i > 1 || cont) {
      r.partials = c->partials;
      r.n_partials = col_groups(c);
    }
    if (ev) (void)hipEventRecord((*ev)[evi++], s);
    e = sgpe::launch_row(r, step_mode, c->full2x2, c->row_iters, c->row_points, s);
    if (e != hipSuccess) return status_of(e);
    if (ev) (void)hipEventRecord((*ev)[evi++], s);
    const bool last = (i == n);
    if (last && defer) break;   // the last K(dt/2) and the inverse x-transform wait (flush_tail)
    e = sgpe::launch_col(col_args(c, last), last ? sgpe::NORM_SQ : sgpe::NORM_DOT, c->col_iters, c->col_points, s);
    if (e != hipSuccess) return status_of(e);
    if (ev) (void)hipEventRecord((*ev)[evi++], s);
  }
  if (defer) {
    c->tail_pending = 2;
    return SGPE_OK;
  }
  RowArgs r = ra;
  r.scale = inv_n;
  r.partials = c->partials;
  r.n_partials = col_groups(c);
  e = sgpe::launch_row(r, sgpe::ROW_INV, false, c->row_iters, c->row_points, s);
  return status_of(e);
}

// The tail a K-R-K step call left (either precision): in real time the last step's K(dt/2), the pending
// axis first; in imaginary time its K(dt/2) (with the norm partials of the finished step) and the
// inverse x-transform (with its rescaling), exactly as the call would have ended.
sgpe_status flush_tail(sgpe_ctx* c) {
  if (c->tail_pending == 0) return SGPE_OK;
  const bool imag = c->tail_pending == 2;
  c->tail_pending = 0;
  if (!imag) {
    hipError_t e = line_pass(c, c->tail_col, LINE_HALF, LINE_NONE, 0);
    if (e == hipSuccess) e = line_pass(c, !c->tail_col, LINE_HALF, LINE_NONE, 0);
    return status_of(e);
  }
  if (c->prec == SGPE_C128) {
    hipError_t e = sgpe::launch_col(col_args_t<double>(c, true), sgpe::NORM_SQ, c->col_points, c->stream);
    if (e != hipSuccess) return status_of(e);
    sgpe::RowArgsT<double> r = row_args_t<double>(c, 0.0);
    r.scale = 1.0 / (double(c->p.nx) * double(c->p.ny));
    r.partials = c->partials;
    r.n_partials = col_groups(c);
    return status_of(sgpe::launch_row(r, sgpe::ROW_INV, false, c->row_points, c->stream));
  }
  hipError_t e = sgpe::launch_col(col_args(c, true), sgpe::NORM_SQ, c->col_iters, c->col_points, c->stream);
  if (e != hipSuccess) return status_of(e);
  RowArgs r = row_args(c);
  r.scale = float(1.0 / (double(c->p.nx) * double(c->p.ny)));
  r.partials = c->partials;
  r.n_partials = col_groups(c);
  e = sgpe::launch_row(r, sgpe::ROW_INV, false, c->row_iters, c->row_points, c->stream);
  return status_of(e);
}

// R-K-R (sgpe_set_splitting):
//   real time:       line passes; K(dt) = X Y lies between two R halves, so with the axes' order
//                    alternating: R(dt/2) X(dt) | Y(dt) R(dt/2) R(dt/2) Y(dt) | X(dt) R R X(dt) | ... |
//                    Z(dt) R(dt/2), n + 1 sweeps, the densities refreshed between the two halves;
//   imaginary time:  built from the general row pass.  The norm falls between the two R halves, so
//                    each step takes a column pass and two row passes: (inv-x, R(dt/2), norm partials)
//                    that stores nothing, then (inv-x, R(dt/2), scale, R(dt/2), fwd-x).  The second
//                    recomputes the first's R(dt/2) from the same input with the same code, so the
//                    partials belong to exactly the state it rescales, and no intermediate state is
//                    stored (one complex64 rounding fewer per step, and 48 instead of 64 bytes per point
//                    of row traffic).
static sgpe_status run_steps_variant(sgpe_ctx* c, int64_t n, bool imag) {
  if (n == 0) return SGPE_OK;
  const sgpe_params& p = c->p;
  hipError_t e = hipSuccess;
  const double h = 0.5 * p.dt;
  if (!imag) {
    bool col = false;
    e = line_pass(c, col, LINE_NONE, LINE_FULL, 1, h);
    for (int64_t i = 1; i <= n && e == hipSuccess; ++i) {
      col = !col;
      const bool last = i == n;
      e = line_pass(c, col, LINE_FULL, last ? LINE_NONE : LINE_FULL, last ? 1 : 2, h);
    }
    return status_of(e);
  }
  const double npts = double(p.nx) * double(p.ny);
  const float inv_n = float(1.0 / npts);
  const int rs = c->split_rs;
  // the general row pass is built for 256-thread workgroups (512 only at 4096 points)
  const int var_rows = std::min(c->rows, sgpe::row_rows_per_block(p.nx, p.ny, c->row_points, c->max_lds));
  const int row_groups = p.ny / var_rows;
  hipStream_t s = c->stream;
  auto row = [&](int flags, int nr, const double* parts, int nparts) {
    RowArgs r = row_args(c, h);
    r.rows_per_block = var_rows;
    r.var_flags = flags;
    r.var_r = nr;
    r.var_nln = rs;
    r.scale = (flags & sgpe::VAR_INV) ? inv_n : 1.0f;   // with VAR_MID_SCALE: the inverse's 1/N only
    r.partials = parts;
    r.n_partials = nparts;
    if (parts) {   // of the real-space state
      r.parseval_w = (2.0 * p.xmax / p.nx) * (2.0 * p.ymax / p.ny);
      r.inv_npts = 1.0;
    }
    r.partials_out = c->partials;
    if (e == hipSuccess) e = sgpe::launch_row(r, sgpe::ROW_VAR, c->full2x2, 1, c->row_points, s);
  };
  row(sgpe::VAR_FWD, 1, nullptr, 0);
  for (int64_t i = 1; i <= n; ++i) {
    const bool last = (i == n);
    if (e == hipSuccess)
      e = sgpe::launch_col(col_args(c, false), sgpe::NORM_NONE, c->col_iters, c->col_points, s);
    row(sgpe::VAR_INV | sgpe::VAR_NORM_OUT | sgpe::VAR_NO_STORE, 1, nullptr, 0);
    row(sgpe::VAR_INV | sgpe::VAR_MID_SCALE | (last ? 0 : sgpe::VAR_FWD), last ? 1 : 2, c->partials, row_groups);
  }
  return status_of(e);
}

EnergyArgs energy_args(const sgpe_ctx* c, double* row_partials, double* col_partials) {
  const sgpe_params& p = c->p;
  EnergyArgs a{};
  a.psi = c->psi;
  a.psi64 = c->psi64;
  a.nx = p.nx;
  a.ny = p.ny;
  a.norm0 = p.norm0;
  a.result = nullptr;
  a.rows = sgpe::energy_rows_per_block(p.nx, p.ny);
  a.cols = sgpe::energy_cols_per_block(p.nx, p.ny, c->max_lds);
  a.twx = c->twp64_x;
  a.twy = c->twp64_y;
  a.xmin = -p.xmax;
  a.dx = 2.0 * p.xmax / p.nx;
  a.ymin = -p.ymax;
  a.dy = 2.0 * p.ymax / p.ny;
  a.wx2h = 0.5 * p.wx * p.wx;
  a.wy2h = 0.5 * p.wy * p.wy;
  a.delta = p.delta;
  a.g_uu = p.g_uu;
  a.g_dd = p.g_dd;
  a.g_ud = p.g_ud;
  a.k_l = p.k_l;
  a.omega = p.omega;
  a.om_x = c->full2x2 ? c->omx : nullptr;
  a.om_y = c->full2x2 ? c->omy : nullptr;
  a.dkx = M_PI / p.xmax;
  a.dky = M_PI / p.ymax;
  a.row_partials = row_partials;
  a.col_partials = col_partials;
  return a;
}

sgpe_status check_ctx_no_flush(sgpe_ctx* c) {
  if (!c) return SGPE_EINVAL;
  if (hipSetDevice(c->device) != hipSuccess) {
    (void)hipGetLastError();
    return SGPE_EDEVICE;
  }
  return SGPE_OK;
}

sgpe_status check_ctx(sgpe_ctx* c) {
  const sgpe_status st = check_ctx_no_flush(c);
  return st != SGPE_OK ? st : flush_tail(c);
}

sgpe_status latched_status(sgpe_ctx* c) {
  if (c->status_host && __atomic_load_n(c->status_host, __ATOMIC_ACQUIRE) != 0u) c->latched = SGPE_ENONFINITE;
  return c->latched;
}

sgpe_status sync_and_latch(sgpe_ctx* c) {
  hipError_t e = hipStreamSynchronize(c->stream);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    return SGPE_EDEVICE;
  }
  return latched_status(c);
}

sgpe_status host_partials(sgpe_ctx* c, size_t n) {
  if (n <= c->host_part_n) return SGPE_OK;
  // the old buffer may still be the destination of queued work
  if (hipStreamSynchronize(c->stream) != hipSuccess) {
    (void)hipGetLastError();
    return SGPE_EDEVICE;
  }
  if (c->host_part) (void)hipHostFree(c->host_part);
  c->host_part = c->host_part_dev = nullptr;
  c->host_part_n = 0;
  void *ptr = nullptr, *dev = nullptr;
  if (hipHostMalloc(&ptr, n * sizeof(double), hipHostMallocMapped | hipHostMallocCoherent) != hipSuccess) {
    (void)hipGetLastError();
    return SGPE_ENOMEM;
  }
  if (hipHostGetDevicePointer(&dev, ptr, 0) != hipSuccess) {
    (void)hipGetLastError();
    (void)hipHostFree(ptr);
    return SGPE_EDEVICE;
  }
  c->host_part = static_cast<double*>(ptr);
  c->host_part_dev = static_cast<double*>(dev);
  c->host_part_n = n;
  return SGPE_OK;
}

// The partials that queued kernels write to host_part_dev are there once this returns.
static sgpe_status wait_partials(sgpe_ctx* c) {
  if (hipStreamSynchronize(c->stream) == hipSuccess) return SGPE_OK;
  (void)hipGetLastError();
  return SGPE_EDEVICE;
}

sgpe_status fetch_partials(sgpe_ctx* c, const double* dev, size_t n, const double** host) {
  *host = nullptr;
  if (const sgpe_status st = host_partials(c, n); st != SGPE_OK) return st;
  if (hipMemcpyAsync(c->host_part, dev, n * sizeof(double), hipMemcpyDeviceToHost, c->stream) != hipSuccess ||
      hipStreamSynchronize(c->stream) != hipSuccess) {
    (void)hipGetLastError();
    return SGPE_EDEVICE;
  }
  *host = c->host_part;
  return SGPE_OK;
}

}  // namespace sgpe_host

using namespace sgpe_host;

extern "C" {

sgpe_status sgpe_validate_params(const sgpe_params* p) {
  if (!p) return SGPE_EINVAL;
  if (!is_pow2(p->nx) || !is_pow2(p->ny)) return SGPE_EINVAL;
  if (p->nx < kMinN || p->ny < kMinN || p->nx > kMaxN || p->ny > kMaxN) return SGPE_EINVAL;
  const double vals[] = {p->xmax, p->ymax, p->g_uu, p->g_dd, p->g_ud, p->k_l, p->omega, p->delta,
                         p->wx, p->wy, p->omega_r0, p->omega_rw, p->dt, p->norm0};
  for (double v : vals)
    if (!is_finite(v)) return SGPE_EINVAL;
  if (!(p->xmax > 0.0) || !(p->ymax > 0.0)) return SGPE_EINVAL;
  if (!(p->dt > 0.0) || !(p->norm0 > 0.0)) return SGPE_EINVAL;
  if (p->wx < 0.0 || p->wy < 0.0) return SGPE_EINVAL;
  if (p->omega_r0 != 0.0 && !(p->omega_rw > 0.0)) return SGPE_EINVAL;
  return SGPE_OK;
}

int32_t sgpe_device_count(void) {
  int n = 0;
  hipError_t e = hipGetDeviceCount(&n);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    return -int32_t(e);
  }
  return n;
}

const char* sgpe_strerror(sgpe_status s) {
  switch (s) {
    case SGPE_OK: return "success";
    case SGPE_EINVAL: return "invalid argument";
    case SGPE_ENOMEM: return "out of device memory or grid too large";
    case SGPE_EDEVICE: return "no usable gfx950 device or HIP runtime error";
    case SGPE_ENONFINITE: return "non-finite value in the state";
    case SGPE_ESTATE: return "call not valid in the current state";
  }
  return "unknown status";
}

// Columns per column-pass tile for complex128: at most 4, 256 threads where one column allows it,
// within the LDS (double2 slots take twice the bytes); at 8 points per lane also at least as many
// workgroups as compute units where one column allows it (measured at 256^2 and 512^2: 1 and 2
// columns, 90.8k and 48.3k imaginary steps/s, against 88.5k and 44.2k for 2 and 1).
static int c128_cols(int nx, int ny, int points, int n_cu, size_t max_lds) {
  int c = 4;
  while (c > 1 && (2 * c * (ny / points) > 256 || c > nx || nx % c != 0 ||
                   !sgpe::schedule_supported(ny, c, 1, points) ||
                   sgpe::col_lds_bytes_c128(ny, c, points) > max_lds || (points == 8 && nx / c < n_cu)))
    c >>= 1;
  return c;
}

static int c128_rows(const sgpe_ctx* c, int points) {
  // one row per workgroup where a row takes at least one wave (measured: 29.1 -> 27.5 us per
  // imaginary step at 512^2, 64.3 -> 63.8 at 1024^2, unchanged at 2048^2), else the derived tile
  const sgpe_params& p = c->p;
  return p.nx / points >= 32 ? 1 : sgpe::row_rows_per_block(p.nx, p.ny, points, c->max_lds / 2);
}

// 8 points per lane where the length allows it, 16 beyond.  An fp64 lane at 16 points holds 64
// registers of points and more of roots (over 200 in all, two waves per SIMD, the column kernel
// spilling); at 8 it runs about 1.1-1.5x the steps/s (1024^2: 17.6k -> 19.3k imaginary, 16.1k ->
// 21.7k real; 512^2: 37.3k -> 48.3k; 256^2: 61.7k -> 90.8k imaginary steps/s).
static void default_schedule_c128(sgpe_ctx* c) {
  const int rp = c->p.nx <= sgpe::kMaxNSmallP ? 8 : 16;
  const int cp = c->p.ny <= sgpe::kMaxNSmallP ? 8 : 16;
  c->rows = c128_rows(c, rp);
  c->cols = c128_cols(c->p.nx, c->p.ny, cp, c->n_cu, c->max_lds);
  c->row_points = rp;
  c->col_points = cp;
  c->row_iters = c->col_iters = 1;
}

// complex128 schedules: 16 or 8 points per lane in each pass (8 for lengths up to kMaxNSmallP),
// one row group / column tile per workgroup, at most 256 threads per workgroup unless one line
// alone needs 512, double2 LDS slots within the device's LDS.
static sgpe_status apply_schedule_c128(sgpe_ctx* c, const sgpe_schedule& s) {
  const sgpe_params& p = c->p;
  auto points_ok = [](int pts, int n) { return pts == 16 || (pts == 8 && n <= sgpe::kMaxNSmallP); };
  auto bound = [](int n, int pts) { return 2 * n / pts > 256 ? 512 : 256; };
  if (!points_ok(s.row_points, p.nx) || !points_ok(s.col_points, p.ny)) return SGPE_EINVAL;
  if (s.row_iters != 1 || s.col_iters != 1 || s.row_tile < 0 || s.col_tile < 1) return SGPE_EINVAL;
  const int rows = s.row_tile > 0 ? s.row_tile : c128_rows(c, s.row_points);
  if (rows > p.ny || p.ny % rows != 0 || !sgpe::schedule_supported(p.nx, rows, 1, s.row_points) ||
      2 * rows * (p.nx / s.row_points) > bound(p.nx, s.row_points) ||
      2 * sgpe::row_lds_bytes(p.nx, rows) > c->max_lds)
    return SGPE_EINVAL;
  const int cols = s.col_tile;
  if (cols > p.nx || p.nx % cols != 0 || !sgpe::schedule_supported(p.ny, cols, 1, s.col_points) ||
      2 * cols * (p.ny / s.col_points) > bound(p.ny, s.col_points) ||
      sgpe::col_lds_bytes_c128(p.ny, cols, s.col_points) > c->max_lds)
    return SGPE_EINVAL;
  c->rows = rows;
  c->cols = cols;
  c->row_points = s.row_points;
  c->col_points = s.col_points;
  c->row_iters = c->col_iters = 1;
  return SGPE_OK;
}

sgpe_status sgpe_create(const sgpe_params* p, void* hip_stream, void* psi_dev, sgpe_ctx** out) {
  return sgpe_create_ex(p, SGPE_C64, hip_stream, psi_dev, out);
}

sgpe_status sgpe_create_ex(const sgpe_params* p, int32_t precision, void* hip_stream, void* psi_dev, sgpe_ctx** out) {
  if (!out) return SGPE_EINVAL;
  *out = nullptr;
  if (precision != SGPE_C64 && precision != SGPE_C128) return SGPE_EINVAL;
  sgpe_status st = sgpe_validate_params(p);
  if (st != SGPE_OK) return st;
  int ndev = 0;
  if (hipGetDeviceCount(&ndev) != hipSuccess || ndev <= 0) {
    (void)hipGetLastError();
    return SGPE_EDEVICE;
  }
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return SGPE_EDEVICE;
  hipDeviceProp_t prop;
  if (hipGetDeviceProperties(&prop, dev) != hipSuccess) return SGPE_EDEVICE;
  if (std::strncmp(prop.gcnArchName, "gfx950", 6) != 0) return SGPE_EDEVICE;
  if (psi_dev && (reinterpret_cast<uintptr_t>(psi_dev) & 15u) != 0) return SGPE_EINVAL;

  sgpe_ctx* c = new (std::nothrow) sgpe_ctx();
  if (!c) return SGPE_ENOMEM;
  c->p = *p;
  c->device = dev;
  c->stream = static_cast<hipStream_t>(hip_stream);
  c->max_lds = prop.sharedMemPerBlock > sgpe::kStaticLds ? size_t(prop.sharedMemPerBlock) - sgpe::kStaticLds : 0;
  c->n_cu = prop.multiProcessorCount > 0 ? prop.multiProcessorCount : 1;
  c->prec = precision;
  default_schedule(c);
  const bool c128 = precision == SGPE_C128;
  if (c128) default_schedule_c128(c);
  c->full2x2 = (p->omega_r0 != 0.0);
  const size_t wb = c128 ? 2 : 1;   // LDS bytes per slot relative to complex64
  const size_t col_lds = c128 ? sgpe::col_lds_bytes_c128(p->ny, c->cols, c->col_points) : sgpe::col_lds_bytes(p->ny, c->cols);
  if (wb * sgpe::row_lds_bytes(p->nx, c->rows) > c->max_lds || col_lds > c->max_lds ||
      !sgpe::energy_fits(p->nx, p->ny, c->max_lds)) {
    delete c;
    return SGPE_ENOMEM;
  }

  const size_t npts = size_t(p->nx) * size_t(p->ny);
  auto fail = [&](sgpe_status s) {
    sgpe_destroy(c);
    return s;
  };
  const size_t state_bytes = npts * (c128 ? sizeof(double4) : sizeof(float4));
  void* state = psi_dev;
  if (!state) {
    if ((st = dev_alloc(c, &state, state_bytes)) != SGPE_OK) return fail(st);
    c->own_psi = true;
  }
  if (c128) c->psi64 = static_cast<double4*>(state);
  else c->psi = static_cast<float4*>(state);
  if ((st = upload(c, &c->twp64_x, root_table<double>(p->nx))) != SGPE_OK) return fail(st);
  if ((st = upload(c, &c->twp64_y, root_table<double>(p->ny))) != SGPE_OK) return fail(st);
  if (!c128) {
    if ((st = upload(c, &c->twp_x, root_table(p->nx))) != SGPE_OK) return fail(st);
    if ((st = upload(c, &c->twp_y, root_table(p->ny))) != SGPE_OK) return fail(st);
  }
  auto k_upload = [&](auto type, auto** kxr, auto** kyr, auto** kxi, auto** kyi) {
    using T = decltype(type);
    for (int half = 0; half < 2; ++half) {
      const double h = half ? 0.5 * p->dt : p->dt;
      std::vector<sgpe::point_t<T>> kx;
      std::vector<sgpe::cplx_t<T>> ky, kxm;
      std::vector<T> kym;
      k_tables_real<T>(*p, h, kx, ky);
      k_tables_imag<T>(*p, h, kxm, kym);
      sgpe_status u;
      if ((u = upload(c, &kxr[half], kx)) != SGPE_OK || (u = upload(c, &kyr[half], ky)) != SGPE_OK ||
          (u = upload(c, &kxi[half], kxm)) != SGPE_OK || (u = upload(c, &kyi[half], kym)) != SGPE_OK)
        return u;
    }
    return SGPE_OK;
  };
  st = c128 ? k_upload(double(), c->kx64_real, c->ky64_real, c->kx64_imag, c->ky64_imag)
            : k_upload(float(), c->kx_real, c->ky_real, c->kx_imag, c->ky_imag);
  if (st != SGPE_OK) return fail(st);
  if (c->full2x2) {
    std::vector<double> om(p->nx);
    const double dx = 2.0 * p->xmax / p->nx;
    for (int j = 0; j < p->nx; ++j) om[j] = p->omega_r0 * std::tanh((-p->xmax + dx * j) / p->omega_rw);
    if ((st = raman_tables(c, om.data(), nullptr)) != SGPE_OK) return fail(st);
  }
  void* ptr = nullptr;
  if ((st = dev_alloc(c, &ptr, kMaxPartials * sizeof(double))) != SGPE_OK) return fail(st);
  c->partials = static_cast<double*>(ptr);
  if ((st = dev_alloc(c, &ptr, (sgpe::kEnergyRowParts * size_t(kMaxN) + kMaxPartials) * sizeof(double))) !=
      SGPE_OK)
    return fail(st);
  c->epart = static_cast<double*>(ptr);
  {
    void* hptr = nullptr;
    void* dptr = nullptr;
    if (hipHostMalloc(&hptr, sizeof(unsigned int), hipHostMallocMapped | hipHostMallocCoherent) != hipSuccess) {
      (void)hipGetLastError();
      return fail(SGPE_ENOMEM);
    }
    c->status_host = static_cast<unsigned int*>(hptr);
    *c->status_host = 0u;
    if (hipHostGetDevicePointer(&dptr, hptr, 0) != hipSuccess) {
      (void)hipGetLastError();
      return fail(SGPE_EDEVICE);
    }
    c->status_dev = static_cast<unsigned int*>(dptr);
  }
  *out = c;
  return SGPE_OK;
}

void sgpe_destroy(sgpe_ctx* c) {
  if (!c) return;
  (void)hipSetDevice(c->device);
  (void)hipStreamSynchronize(c->stream);
  for (void* ptr : c->allocations) (void)hipFree(ptr);
  if (c->host_part) (void)hipHostFree(c->host_part);
  if (c->status_host) (void)hipHostFree(c->status_host);
  if (c->relax_host) (void)hipHostFree(c->relax_host);
  for (hipEvent_t ev : c->relax_ev)
    if (ev) (void)hipEventDestroy(ev);
  (void)hipGetLastError();
  delete c;
}

sgpe_status sgpe_set_col_tile(sgpe_ctx* c, int32_t columns) {
  if (!c || c->prec == SGPE_C128) return SGPE_EINVAL;
  if (const sgpe_status st = check_ctx(c); st != SGPE_OK) return st;   // the pending tail, old schedule
  if (columns == 0) {
    default_schedule(c);
    return SGPE_OK;
  }
  const sgpe_params& p = c->p;
  if (columns < 1) return SGPE_EINVAL;
  int iters = c->col_iters;
  if (!sgpe::col_tile_supported(p.nx, p.ny, columns, iters, c->col_points, c->max_lds)) iters = 1;
  if (!sgpe::col_tile_supported(p.nx, p.ny, columns, iters, c->col_points, c->max_lds)) return SGPE_EINVAL;
  c->cols = columns;
  c->col_iters = iters;
  return SGPE_OK;
}

sgpe_status sgpe_get_schedule(sgpe_ctx* c, sgpe_schedule* out) {
  if (!c || !out) return SGPE_EINVAL;
  *out = get_schedule(c);
  return SGPE_OK;
}

sgpe_status sgpe_set_schedule(sgpe_ctx* c, const sgpe_schedule* s) {
  if (!c) return SGPE_EINVAL;
  if (const sgpe_status st = check_ctx(c); st != SGPE_OK) return st;   // the pending tail, old schedule
  if (c->prec == SGPE_C128) {
    if (!s) {
      default_schedule_c128(c);
      return SGPE_OK;
    }
    return apply_schedule_c128(c, *s);
  }
  if (!s) {
    default_schedule(c);
    return SGPE_OK;
  }
  return apply_schedule(c, *s);
}

sgpe_status sgpe_set_psi(sgpe_ctx* c, const double* h) {
  sgpe_status st = check_ctx_no_flush(c);
  if (st != SGPE_OK) return st;
  if (!h) return SGPE_EINVAL;
  const size_t nx = size_t(c->p.nx), ny = size_t(c->p.ny), npts = nx * ny;
  for (size_t i = 0; i < 4 * npts; ++i)
    if (!std::isfinite(h[i])) return SGPE_ENONFINITE;
  const double* up = h;
  const double* dn = h + 2 * npts;
  hipError_t e;
  if (c->prec == SGPE_C128) {
    std::vector<double4> buf(npts);
    for (size_t i = 0; i < npts; ++i) buf[i] = make_double4(up[2 * i], up[2 * i + 1], dn[2 * i], dn[2 * i + 1]);
    e = hipMemcpyAsync(c->psi64, buf.data(), npts * sizeof(double4), hipMemcpyHostToDevice, c->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
  } else {
    std::vector<float4> buf(npts);
    for (size_t i = 0; i < npts; ++i)
      buf[i] = make_float4(float(up[2 * i]), float(up[2 * i + 1]), float(dn[2 * i]), float(dn[2 * i + 1]));
    e = hipMemcpyAsync(c->psi, buf.data(), npts * sizeof(float4), hipMemcpyHostToDevice, c->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
  }
  if (e != hipSuccess) {
    (void)hipGetLastError();
    return SGPE_EDEVICE;
  }
  c->has_state = true;
  c->tail_pending = 0;
  c->latched = SGPE_OK;
  if (c->status_host) __atomic_store_n(c->status_host, 0u, __ATOMIC_RELEASE);   // the stream is idle
  return SGPE_OK;
}

sgpe_status sgpe_set_psi_device(sgpe_ctx* c, const void* d) {
  sgpe_status st = check_ctx(c);   // a pending tail completes: d may be the state buffer itself
  if (st != SGPE_OK) return st;
  if (!d || reinterpret_cast<uintptr_t>(d) % 16 != 0) return SGPE_EINVAL;
  const long long npts = (long long)c->p.nx * c->p.ny;
  const int nb = sgpe::norm_blocks();
  const bool c128 = c->prec == SGPE_C128;
  if ((st = host_partials(c, size_t(nb))) != SGPE_OK) return st;
  const double* part = c->host_part;
  double* to = c->host_part_dev;
  hipError_t e = c128 ? sgpe::launch_nonfinite(static_cast<const double4*>(d), npts, to, nb, c->stream)
                      : sgpe::launch_nonfinite(static_cast<const float4*>(d), npts, to, nb, c->stream);
  if (e != hipSuccess) return status_of(e);
  if ((st = wait_partials(c)) != SGPE_OK) return st;
  double bad = 0.0;
  for (int b = 0; b < nb; ++b) bad += part[b];
  if (bad != 0.0) return SGPE_ENONFINITE;   // the state is unchanged
  // the stream is idle: no step kernel can set the status word any more
  if (c->status_host) __atomic_store_n(c->status_host, 0u, __ATOMIC_RELEASE);
  void* dst = c128 ? static_cast<void*>(c->psi64) : static_cast<void*>(c->psi);
  const size_t bytes = size_t(npts) * (c128 ? sizeof(double4) : sizeof(float4));
  e = dst == d ? hipSuccess : hipMemcpyAsync(dst, d, bytes, hipMemcpyDeviceToDevice, c->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    return SGPE_EDEVICE;
  }
  c->has_state = true;
  c->tail_pending = 0;
  c->latched = SGPE_OK;
  return SGPE_OK;
}

sgpe_status sgpe_get_psi(sgpe_ctx* c, double* h) {
  sgpe_status st = check_ctx(c);
  if (st != SGPE_OK) return st;
  if (!h) return SGPE_EINVAL;
  if (!c->has_state) return SGPE_ESTATE;
  const size_t npts = size_t(c->p.nx) * size_t(c->p.ny);
  bool ok = true;
  double* up = h;
  double* dn = h + 2 * npts;
  auto unpack = [&](const auto& buf) {
    for (size_t i = 0; i < npts; ++i) {
      const auto w = buf[i];
      up[2 * i] = w.x;
      up[2 * i + 1] = w.y;
      dn[2 * i] = w.z;
      dn[2 * i + 1] = w.w;
      ok = ok && std::isfinite(w.x) && std::isfinite(w.y) && std::isfinite(w.z) && std::isfinite(w.w);
    }
  };
  hipError_t e;
  if (c->prec == SGPE_C128) {
    std::vector<double4> buf(npts);
    e = hipMemcpyAsync(buf.data(), c->psi64, npts * sizeof(double4), hipMemcpyDeviceToHost, c->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
    if (e == hipSuccess) unpack(buf);
  } else {
    std::vector<float4> buf(npts);
    e = hipMemcpyAsync(buf.data(), c->psi, npts * sizeof(float4), hipMemcpyDeviceToHost, c->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
    if (e == hipSuccess) unpack(buf);
  }
  if (e != hipSuccess) {
    (void)hipGetLastError();
    return SGPE_EDEVICE;
  }
  if (!ok) c->latched = SGPE_ENONFINITE;
  return latched_status(c);
}

static sgpe_status step_common(sgpe_ctx* c, int64_t n, bool imag) {
  sgpe_status st = check_ctx_no_flush(c);
  if (st != SGPE_OK) return st;
  if (n < 0) return SGPE_EINVAL;
  if (!c->has_state) return SGPE_ESTATE;
  return run_steps(c, n, imag, nullptr);
}

sgpe_status sgpe_step_real(sgpe_ctx* c, int64_t n) { return step_common(c, n, false); }
sgpe_status sgpe_step_imag(sgpe_ctx* c, int64_t n) { return step_common(c, n, true); }

sgpe_status sgpe_synchronize(sgpe_ctx* c) {
  sgpe_status st = check_ctx(c);
  if (st != SGPE_OK) return st;
  return sync_and_latch(c);
}

sgpe_status sgpe_norm(sgpe_ctx* c, double* out) {
  sgpe_status st = check_ctx(c);
  if (st != SGPE_OK) return st;
  if (!out) return SGPE_EINVAL;
  if (!c->has_state) return SGPE_ESTATE;
  const long long npts = (long long)c->p.nx * c->p.ny;
  const int nb = sgpe::norm_blocks();
  // The 256 blocks write their partials straight to the host's buffer (13.6 us per call on small grids;
  // with a copy behind the kernel 16.6).  The energy's keep the copy: its thousands of blocks come in many
  // rounds, and each would wait for the host's memory before it ends (2048^2: 87 us, that way 116).
  if ((st = host_partials(c, size_t(nb))) != SGPE_OK) return st;
  const double* part = c->host_part;
  hipError_t e = c->prec == SGPE_C128 ? sgpe::launch_norm(c->psi64, npts, c->host_part_dev, nb, c->stream)
                                      : sgpe::launch_norm(c->psi, npts, c->host_part_dev, nb, c->stream);
  if (e != hipSuccess) return status_of(e);
  if ((st = wait_partials(c)) != SGPE_OK) return st;
  double s = 0.0;
  for (int b = 0; b < nb; ++b) s += part[b];
  const double dx = 2.0 * c->p.xmax / c->p.nx, dy = 2.0 * c->p.ymax / c->p.ny;
  *out = dx * dy * s;
  if (!std::isfinite(*out)) c->latched = SGPE_ENONFINITE;
  return latched_status(c);
}

sgpe_status sgpe_set_splitting(sgpe_ctx* c, int32_t order, int32_t real_space) {
  if (!c) return SGPE_EINVAL;
  if (const sgpe_status st = check_ctx(c); st != SGPE_OK) return st;   // the pending tail, old scheme
  if ((order != SGPE_SPLIT_KRK && order != SGPE_SPLIT_RKR) ||
      (real_space != SGPE_RSPLIT_FROZEN && real_space != SGPE_RSPLIT_NLN))
    return SGPE_EINVAL;
  if (c->prec == SGPE_C128 && (order != SGPE_SPLIT_KRK || real_space != SGPE_RSPLIT_FROZEN)) return SGPE_EINVAL;
  const int row_groups = c->p.ny / std::min(c->rows, sgpe::row_rows_per_block(c->p.nx, c->p.ny, c->row_points,
                                                                               c->max_lds));
  if (order == SGPE_SPLIT_RKR && row_groups > kMaxPartials) return SGPE_EINVAL;
  c->split_order = order;
  c->split_rs = real_space;
  return SGPE_OK;
}

sgpe_status sgpe_energy(sgpe_ctx* c, double* out) {
  sgpe_status st = check_ctx(c);
  if (st != SGPE_OK) return st;
  if (!out) return SGPE_EINVAL;
  if (!c->has_state) return SGPE_ESTATE;
  const sgpe_params& p = c->p;
  const size_t npts = size_t(p.nx) * size_t(p.ny);
  const double dx = 2.0 * p.xmax / p.nx, dy = 2.0 * p.ymax / p.ny;
  const int nrb = p.ny / sgpe::energy_rows_per_block(p.nx, p.ny);   // row blocks
  constexpr int RP = sgpe::kEnergyRowParts;
  EnergyArgs a = energy_args(c, c->epart, c->epart + RP * nrb);
  const int ncb = p.nx / a.cols;
  hipError_t e = sgpe::launch_energy(a, c->stream);
  if (e != hipSuccess) return status_of(e);
  const double* part = nullptr;
  if ((st = fetch_partials(c, c->epart, RP * size_t(nrb) + ncb, &part)) != SGPE_OK) return st;
  double er = 0.0, ei = 0.0, nr = 0.0, ek = 0.0;
  for (int b = 0; b < nrb; ++b) {
    er += part[RP * b];
    ei += part[RP * b + 1];
    nr += part[RP * b + 2];
  }
  for (int b = 0; b < ncb; ++b) ek += part[RP * nrb + b];
  // per particle of the state rescaled to norm0: quadratic terms over the norm, the interaction
  // (quartic) terms over norm^2 / norm0
  const double w = dx * dy;
  const double nrm = w * nr;
  *out = (w / double(npts) * ek + w * er) / nrm + w * ei * p.norm0 / (nrm * nrm);
  if (!std::isfinite(*out)) c->latched = SGPE_ENONFINITE;
  return latched_status(c);
}

sgpe_status sgpe_profile_steps(sgpe_ctx* c, int32_t imag, int64_t n, double* row_ms, double* col_ms) {
  sgpe_status st = check_ctx(c);
  if (st != SGPE_OK) return st;
  if (n <= 0) return SGPE_EINVAL;
  if (!c->has_state || c->split_order != SGPE_SPLIT_KRK || c->split_rs != SGPE_RSPLIT_FROZEN ||
      c->prec == SGPE_C128)
    return SGPE_ESTATE;
  // imaginary time: three events per step (row pass, column pass); real time: a pair around the
  // leading row pass and around each step's one pass (columns first, then alternating)
  std::vector<hipEvent_t> ev(imag ? 3 * size_t(n) : 2 * size_t(n) + 2);
  for (auto& x : ev) {
    if (hipEventCreate(&x) != hipSuccess) {
      (void)hipGetLastError();
      return SGPE_EDEVICE;
    }
  }
  st = run_steps(c, n, imag != 0, &ev);
  if (st == SGPE_OK) st = sync_and_latch(c);
  double tr = 0.0, tc = 0.0;
  if (st == SGPE_OK) {
    auto ms = [&](size_t i) {
      float t = 0.f;
      (void)hipEventElapsedTime(&t, ev[i], ev[i + 1]);
      return double(t);
    };
    if (imag) {
      for (int64_t i = 0; i < n; ++i) {
        tr += ms(3 * i) / double(n);
        tc += ms(3 * i + 1) / double(n);
      }
    } else {
      const int64_t ncol = (n + 1) / 2, nrow = n / 2;
      for (int64_t i = 1; i <= n; ++i) (i % 2 ? tc : tr) += ms(2 * size_t(i)) / double(i % 2 ? ncol : nrow);
      if (nrow == 0) tr = ms(0);   // one step has no row pass with R: the leading one
    }
  }
  for (auto& x : ev) (void)hipEventDestroy(x);
  if (st != SGPE_OK) return st;
  if (row_ms) *row_ms = tr;
  if (col_ms) *col_ms = tc;
  return SGPE_OK;
}

sgpe_status sgpe_profile_kernels(sgpe_ctx* c, int32_t imag, int64_t n, double* row_ms, double* col_ms) {
  sgpe_status st = check_ctx(c);
  if (st != SGPE_OK) return st;
  if (n <= 0) return SGPE_EINVAL;
  if (!c->has_state || c->split_order != SGPE_SPLIT_KRK || c->split_rs != SGPE_RSPLIT_FROZEN ||
      c->prec == SGPE_C128)
    return SGPE_ESTATE;
  const sgpe_params& p = c->p;
  const size_t bytes = size_t(p.nx) * size_t(p.ny) * sizeof(float4);
  if (!c->scratch) {
    void* ptr = nullptr;
    if ((st = dev_alloc(c, &ptr, bytes)) != SGPE_OK) return st;
    c->scratch = static_cast<float4*>(ptr);
  }
  hipEvent_t ev[4];
  int made = 0;
  for (; made < 4; ++made) {
    if (hipEventCreate(&ev[made]) != hipSuccess) break;
  }
  hipStream_t s = c->stream;
  hipError_t e = made == 4 ? hipSuccess : hipErrorOutOfMemory;
  // keep the state; in imaginary time enter the mixed representation with valid norm partials
  if (e == hipSuccess) e = hipMemcpyAsync(c->scratch, c->psi, bytes, hipMemcpyDeviceToDevice, s);
  RowArgs r = row_args(c);
  if (imag) {
    if (e == hipSuccess) e = sgpe::launch_row(r, sgpe::ROW_FWD, false, c->row_iters, c->row_points, s);
    if (e == hipSuccess) e = sgpe::launch_col(col_args(c, true), sgpe::NORM_DOT, c->col_iters, c->col_points, s);
    r.scale = float(1.0 / (double(p.nx) * double(p.ny)));
    r.partials = c->partials;
    r.n_partials = col_groups(c);
  }
  const ColArgs ca = col_args(c, false);
  if (e == hipSuccess) e = hipEventRecord(ev[0], s);
  for (int64_t i = 0; i < n && e == hipSuccess; ++i)
    e = imag ? sgpe::launch_row(r, sgpe::ROW_STEP, c->full2x2, c->row_iters, c->row_points, s)
             : line_pass(c, false, LINE_FULL, LINE_FULL, 1);
  if (e == hipSuccess) e = hipEventRecord(ev[1], s);
  if (e == hipSuccess) e = hipEventRecord(ev[2], s);
  for (int64_t i = 0; i < n && e == hipSuccess; ++i)
    e = imag ? sgpe::launch_col(ca, sgpe::NORM_DOT, c->col_iters, c->col_points, s)
             : line_pass(c, true, LINE_FULL, LINE_FULL, 1);
  if (e == hipSuccess) e = hipEventRecord(ev[3], s);
  if (e == hipSuccess) e = hipMemcpyAsync(c->psi, c->scratch, bytes, hipMemcpyDeviceToDevice, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  float a = 0.f, b = 0.f;
  if (e == hipSuccess) e = hipEventElapsedTime(&a, ev[0], ev[1]);
  if (e == hipSuccess) e = hipEventElapsedTime(&b, ev[2], ev[3]);
  for (int i = 0; i < made; ++i) (void)hipEventDestroy(ev[i]);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    return status_of(e);
  }
  if (row_ms) *row_ms = double(a) / double(n);
  if (col_ms) *col_ms = double(b) / double(n);
  return latched_status(c);
}

}  // extern "C"
