// Device bodies of the row pass (see row_pass.hip for the kernels and the pass's place in a
// step): the norm scale from the column pass's partials, the real-space exponential R(h) of
// Eqs. (H2)-(H4) (closed form with frozen densities, or N(h/2) L(h) N(h/2)), and the row body
// itself -- inverse x-FFT, scale, R, forward x-FFT -- shared by every kernel that runs rows.
#pragma once

#include <type_traits>

#include "fft_device.hpp"
#include "sgpe_internal.hpp"

namespace sgpe {


// -------------------------------------------------------------------------------------------
// Sum of the previous column pass's partials -> scale for the row pass.  Every wave computes
// the same sum in the same order (lane l adds partials l, l + 64, ... in turn, then a fixed
// butterfly across the wave), so every workgroup applies bit-identical scales.  Up to 64 K partials
// are loaded at kernel start as masked loads, ahead of the data, and summed while the data is on its
// way; more, or workgroups narrower than a wave, take a loop behind the data's loads.
// K = 4 (256 partials: one per compute unit), and 16 (1024) for complex128 rows of up to 1024 points,
// whose 1-column tiles leave nx partials.  (16 everywhere: 18 VGPRs more in the row passes, of which
// the full 2x2 one at 2048 points would then keep two waves per SIMD instead of three.)
// -------------------------------------------------------------------------------------------
template <class R, int N>
constexpr int prefetch_per_lane() { return sizeof(R) == 8 && N <= 1024 ? 16 : 4; }

template <class A, int K>
__device__ __forceinline__ void prefetch_partials(const A& a, double (&pv)[K]) {
  const int lane = threadIdx.x & 63;
  // uniform branches around unconditional loads (indices clamped into range; the surplus
  // masked out at the sum), so no lane-dependent control flow waits on a load
  const bool early = a.partials != nullptr && a.n_partials <= 64 * K && blockDim.x >= 64;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    pv[k] = 0.0;
    if (early && 64 * k < a.n_partials) pv[k] = a.partials[min(lane + 64 * k, a.n_partials - 1)];
  }
}

template <class A, int K>
__device__ __forceinline__ decltype(A::scale) row_scale(const A& a, const double (&pv)[K]) {
  if (a.partials == nullptr) return a.scale;
  double s = 0.0;
  if (blockDim.x >= 64) {
    const int lane = threadIdx.x & 63;
    if (a.n_partials <= 64 * K) {
#pragma unroll
      for (int k = 0; k < K; ++k) s += (lane + 64 * k < a.n_partials) ? pv[k] : 0.0;
    } else {
      // eight loads in flight at a time (a loop of load and add waits for each)
      for (int i0 = 0; i0 < a.n_partials; i0 += 512) {
        double q[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) q[k] = a.partials[min(i0 + 64 * k + lane, a.n_partials - 1)];
#pragma unroll
        for (int k = 0; k < 8; ++k) s += i0 + 64 * k + lane < a.n_partials ? q[k] : 0.0;
      }
    }
    s = wave_sum(s);
  } else {
    for (int i = 0; i < a.n_partials; ++i) s += a.partials[i];
  }
  const double norm = a.parseval_w * s;
  return static_cast<decltype(A::scale)>(sqrt(a.norm0 / norm) * a.inv_npts);
}

// A norm-derived scale that is not finite and positive means that the norm the partials gave was
// zero, infinite or NaN (a diverging or overflowing imaginary-time run).  Workgroup 0 records it in
// the context's status word; the host reports it at the next synchronising call.
template <class A, class R>
__device__ __forceinline__ void check_scale(const A& a, R s, int wg) {
  if (a.partials != nullptr && a.nonfinite != nullptr && wg == 0 && threadIdx.x == 0 &&
      !(s > R(0) && __builtin_isfinite(s)))
    __hip_atomic_store(a.nonfinite, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// -------------------------------------------------------------------------------------------
// Real-space exponential R(h) (Eqs. (H2)-(H4), densities of the input).  Each lane applies its
// component's row of the 2x2 exponential to its value w; o is the partner lane's value at the
// same point.  hv = h V(x, y); hbx = h Omega(x, y) / 2 with Omega(x, y) = Omega_x(x) + Omega_y(y).
// -------------------------------------------------------------------------------------------
template <class T>
struct RCoef {
  T hd_own;          // +- h delta / 2 for this component
  T hg_own;          // h g_{ss} of this component
  T hg_ud;           // h g_{up dn}
  T sgn;             // +1 up, -1 down
  T hg_uu, hg_dd, hdelta2;
};

// Diagonal R (no spatial Raman coupling): w exp(-ph) in imaginary time, w exp(-i ph) in real
// time, with ph = h (V + g_own n_own + g_ud n_other +- delta/2).  Both are applied as w plus a small
// correction formed first.  SMALL: |ph| <= angle_limit; the general forms choose by the angle and give
// the same bits for small ones, so results do not depend on a wave's vote.
template <bool IMAG, class T>
constexpr T angle_limit() { return IMAG ? T(kSmallExp) : T(kSmallPhase); }

template <bool IMAG, bool SMALL, class C, class T>
__device__ __forceinline__ C apply_r_diag(C w, T ph) {
  if constexpr (!IMAG) {
    const auto sc = sincos_m1_t<SMALL>(ph);
    return mk2(w.x + fma_(w.x, sc.cm1, w.y * sc.s), w.y + fma_(w.y, sc.cm1, -w.x * sc.s));
  } else {
    if (SMALL || fabs_(ph) <= angle_limit<IMAG, T>()) {
      const T e = expm1_small(-ph);
      return mk2(fma_(w.x, e, w.x), fma_(w.y, e, w.y));
    }
    return vscale(w, exp_(-ph));
  }
}

// Full 2x2 R: H_R = A 1 + Bx sigma_x + Bz sigma_z (all times h).  The angles (A, |B|) of this
// point.
template <class T>
struct RFull {
  T ha, hbz, th;
};
template <class T>
__device__ __forceinline__ RFull<T> r_full_angles(T n_own, T n_oth, T hv, const RCoef<T>& c, T hbx) {
  const T nu = c.sgn > T(0) ? n_own : n_oth;
  const T nd = c.sgn > T(0) ? n_oth : n_own;
  const T gu = fma_(c.hg_uu, nu, c.hg_ud * nd);
  const T gd = fma_(c.hg_dd, nd, c.hg_ud * nu);
  RFull<T> f;
  f.ha = fma_(T(0.5), gu + gd, hv);
  f.hbz = fma_(T(0.5), gu - gd, c.hdelta2);
  f.th = sqrt_(fma_(hbx, hbx, f.hbz * f.hbz));
  return f;
}

// cosh(th) and sinh(th) / th by Taylor polynomials for th below this
constexpr float kSmallHyp = 0.25f;
__device__ __forceinline__ void hyp_small(float th, float& ch, float& shc) {
  const float t2 = th * th;
  ch = fmaf(t2, fmaf(t2, fmaf(t2, fmaf(t2, 2.48015873e-5f, 1.38888889e-3f), 4.16666667e-2f), 0.5f), 1.0f);
  shc = fmaf(t2, fmaf(t2, fmaf(t2, fmaf(t2, 2.75573192e-6f, 1.98412698e-4f), 8.33333333e-3f), 1.66666667e-1f), 1.0f);
}
__device__ __forceinline__ void hyp_small(double th, double& ch, double& shc) {
  const double t2 = th * th;
  ch = fma(t2, fma(t2, fma(t2, fma(t2, fma(t2, fma(t2, 1.0 / 479001600.0, 1.0 / 3628800.0), 1.0 / 40320.0),
                                   1.0 / 720.0), 1.0 / 24.0), 0.5), 1.0);
  shc = fma(t2, fma(t2, fma(t2, fma(t2, fma(t2, fma(t2, 1.0 / 6227020800.0, 1.0 / 39916800.0), 1.0 / 362880.0),
                                    1.0 / 5040.0), 1.0 / 120.0), 1.0 / 6.0), 1.0);
}

template <bool IMAG, bool SMALL, class C, class T>
__device__ __forceinline__ C apply_r_full(C w, C o, const RFull<T>& f, T hbx, T sgn) {
  if constexpr (!IMAG) {
    // M = cos(th) 1 - i sin(th)/th (hB . sigma): this component's row of (M - 1) psi is
    // cm1 w - i X with X = +-pz w + px o.
    const auto sb = sincos_m1_t<SMALL>(f.th);
    const T px = sb.sinc * hbx, pz = sgn * sb.sinc * f.hbz;
    const T xr = fma_(pz, w.x, px * o.x), xi = fma_(pz, w.y, px * o.y);
    const T mr = fma_(sb.cm1, w.x, xi), mi = fma_(sb.cm1, w.y, -xr);
    // E M psi - psi = c_M + (E - 1)(w + c_M), E - 1 = cm1_A - i s_A; added to w once.
    const auto se = sincos_m1_t<SMALL>(f.ha);
    const T cr = fma_(se.s, w.y, fma_(se.cm1, w.x, fma_(se.s, mi, fma_(se.cm1, mr, mr))));
    const T ci = fma_(-se.s, w.x, fma_(se.cm1, w.y, fma_(-se.s, mr, fma_(se.cm1, mi, mi))));
    return mk2(w.x + cr, w.y + ci);
  } else {
    T ea, ch, shc;  // exp(-A), cosh(th), sinh(th)/th
    if (SMALL || fabs_(f.ha) <= angle_limit<IMAG, T>()) ea = T(1) + expm1_small(-f.ha);
    else ea = exp_(-f.ha);
    if (SMALL || f.th < T(kSmallHyp)) {
      hyp_small(f.th, ch, shc);
    } else if constexpr (sizeof(T) == 8) {
      ch = cosh(f.th);
      shc = sinh(f.th) / f.th;
    } else {
      const float ep = expf(f.th);
      const float em = 1.0f / ep;
      ch = 0.5f * (ep + em);
      shc = 0.5f * (ep - em) / f.th;
    }
    const T m_own = ea * fma_(-sgn * shc, f.hbz, ch);
    const T m_x = -ea * shc * hbx;
    return mk2(fma_(m_own, w.x, m_x * o.x), fma_(m_own, w.y, m_x * o.y));
  }
}

// -------------------------------------------------------------------------------------------
// R on the thread's points
// -------------------------------------------------------------------------------------------
// A: any argument struct with the real-space fields of RowArgsT (x along the line the lane holds, y
// across).
template <class R, class A>
__device__ __forceinline__ RCoef<R> r_coefs(const A& a, bool up) {
  RCoef<R> c;
  c.sgn = up ? R(1) : R(-1);
  c.hd_own = up ? a.hdelta2 : -a.hdelta2;
  c.hg_uu = a.hg_uu;
  c.hg_dd = a.hg_dd;
  c.hg_ud = a.hg_ud;
  c.hg_own = up ? c.hg_uu : c.hg_dd;
  c.hdelta2 = a.hdelta2;
  return c;
}

// Imaginary time: whether the SMALL routines hold for every point of the wave, from bounds: the
// potential at the ends of the line, the largest density of the lane's points, the largest coupling.
// The bounds are sums of maxima over different points, and a wave that they send the general way gets
// the same bits.
template <bool FULL, bool NLN, int P, class C, class R, class A>
__device__ __forceinline__ bool small_angles(const C (&v)[P], const A& a, const RCoef<R>& c, R hvy,
                                             const R (&hbx_r)[P], R hb_row) {
  R n = R(0);
#pragma unroll
  for (int m = 0; m < P; ++m) n = fmax_(n, fmax_(fabs_(v[m].x), fabs_(v[m].y)));
  n = R(2) * n * n;   // at least the largest density (and no density that R would want to keep)
  n += pair_swap(n);
  const R g = fmax_(fmax_(fabs_(c.hg_uu), fabs_(c.hg_dd)), fabs_(c.hg_ud)) * n;
  const R pot = fma_(a.hvx * a.x0, a.x0, hvy), det = fabs_(a.hdelta2);
  R angle = NLN ? (FULL ? pot : pot + det) : (FULL ? pot + g : pot + det + g);
  // the second mean-field factor of N L N sees densities that L has changed, by less than
  // exp(2 (0.35 + 0.25)) < 4 below the limits
  if constexpr (NLN) angle = fmax_(angle, R(2) * g);
  bool ok = angle <= R(kSmallExp);
  if constexpr (FULL) {
    R b = R(0);
#pragma unroll
    for (int m = 0; m < P; ++m) b = fmax_(b, fabs_(hbx_r[m]));
    b += fabs_(hb_row) + det + (NLN ? R(0) : g);
    ok = ok && b <= R(0.99f * kSmallHyp);
  }
  return wave_all(ok);
}

// hbx_r: this lane's h Omega_x / 2 at its P positions, hb_row: h Omega_y / 2 of the row (full
// 2x2 variant only; loaded by the caller ahead of the transforms).  NLN: R(h) split to second order as
// N(h/2) L(h) N(h/2), the mean-field phase with the densities of its input, the exponential of the
// linear real-space terms (trap, detuning, spatial coupling), the mean-field phase again with the
// updated densities.
//
// A wave takes the SMALL routines or the general ones by a vote of its lanes.  Real time votes per
// point and factor.  Imaginary time votes once for all points, so that the small forms are one straight
// line without branches, whose points fill each other's dependency chains (full 2x2 row pass at 2048^2:
// with the polynomial exp, 68 -> 52 us; one vote in real time was 2-4 % slower than sixteen).
template <int N, bool IMAG, bool FULL, bool NLN, bool ANEW = IMAG || NLN, int P, class C, class R, class A>
__device__ __forceinline__ void row_apply_r(C (&v)[P], const A& a, int row, int t, bool up,
                                            const R (&hbx_r)[P], R hb_row) {
  const LanePos<N / P> pos = real_pos<N, P>(t);
  const RCoef<R> c = r_coefs<R>(a, up);
  const R y = fma_(static_cast<R>(row), a.dy, a.y0);
  const R hvy = a.hvy * y * y;
  auto apply = [&](auto small) {
    constexpr bool SMALL = decltype(small)::value;
    // ANEW: opaque to the compiler.  The terms that depend on the position alone would else be formed
    // once for both forms (and once for all sub-steps of a pass) and held, a register each per point.
    R hv0 = hvy, j0 = static_cast<R>(pos.p0), jb = static_cast<R>(pos.b), hb0 = hb_row;
    if constexpr (ANEW) asm volatile("; %4" : "+v"(hv0), "+v"(j0), "+v"(jb), "+v"(hb0) : "i"(int(SMALL)));
    auto diag = [&](C w, R ph) {
      if constexpr (!IMAG) {
        if (wave_all(fabs_(ph) <= angle_limit<IMAG, R>())) return apply_r_diag<IMAG, true>(w, ph);
      }
      return apply_r_diag<IMAG, SMALL>(w, ph);
    };
    auto half_n = [&](C w) {
      const R n_own = fma_(w.x, w.x, w.y * w.y);
      const R n_oth = pair_swap(n_own);
      return diag(w, R(0.5) * fma_(c.hg_own, n_own, c.hg_ud * n_oth));
    };
#pragma unroll
    for (int m = 0; m < P; ++m) {
      if constexpr (IMAG && !SMALL) {
        // a branch the compiler cannot fold keeps it from running the general form of all points
        // side by side, which takes every register there is (1024 points with a spatial coupling: 243
        // VGPRs, where the small form takes 168)
        int go = 1;
        asm volatile("" : "+s"(go));
        if (go == 0) continue;
      }
      const R x = fma_(m == 0 ? j0 : jb + R(N / P * m), a.dx, a.x0);   // the position is exact
      const R hv = fma_(a.hvx * x, x, hv0);
      C w = v[m];
      if constexpr (NLN) w = half_n(w);
      if constexpr (!FULL) {
        R ph = hv + c.hd_own;
        if constexpr (!NLN) {
          const R n_own = fma_(w.x, w.x, w.y * w.y);
          const R n_oth = pair_swap(n_own);
          ph = fma_(c.hg_own, n_own, fma_(c.hg_ud, n_oth, ph));
        }
        w = diag(w, ph);
      } else {
        const R hbx = hbx_r[m] + hb0;
        const C o = pair_swap(w);
        RFull<R> f;
        if constexpr (NLN) {
          f.ha = hv;
          f.hbz = c.hdelta2;
          f.th = sqrt_(fma_(hbx, hbx, f.hbz * f.hbz));
        } else {
          f = r_full_angles(fma_(w.x, w.x, w.y * w.y), fma_(o.x, o.x, o.y * o.y), hv, c, hbx);
        }
        if (!IMAG && wave_all(fabs_(f.ha) <= R(kSmallPhase) && f.th <= R(kSmallPhase)))
          w = apply_r_full<IMAG, true>(w, o, f, hbx, c.sgn);
        else
          w = apply_r_full<IMAG, SMALL>(w, o, f, hbx, c.sgn);
      }
      if constexpr (NLN) w = half_n(w);
      v[m] = w;
    }
  };
  if constexpr (IMAG) {
    if (small_angles<FULL, NLN>(v, a, c, hvy, hbx_r, hb_row)) apply(std::true_type{});
    else apply(std::false_type{});
  } else {
    apply(std::false_type{});
  }
}

// -------------------------------------------------------------------------------------------
// Row pass
// -------------------------------------------------------------------------------------------
// A workgroup handles ITERS groups of rows_per_block rows, one after the other; the next group's
// data is loaded into registers before the current group is transformed, so its memory latency
// hides behind this group's arithmetic.  P points per lane: T = N / P lanes per transform.
// The kernels' dynamic LDS, typed per precision where it is used.
extern __shared__ __align__(16) unsigned char row_lds[];

template <int N, int MODE, bool FULL, int ITERS, int P, bool WT, class R>
__device__ __forceinline__ void row_body(const RowArgsT<R>& a, int wg) {
  using C = cplx_t<R>;
  constexpr int T = N / P;
  constexpr uint32_t PB = sizeof(point_t<R>), CB = sizeof(C);   // bytes per point / component
  const int tid = threadIdx.x;
  const int comp = tid & 1;
  const int pair = tid >> 1;
  const int rloc = pair / T;
  const int t = pair - rloc * T;
  const int row0 = wg * ITERS * a.rows_per_block + rloc;
  constexpr bool STEP = MODE == ROW_STEP || MODE == ROW_STEP_NLN;
  const LdsView<C> lds = lds_line<N, C>(row_lds, rloc, a.rows_per_block, comp);
  // element j of this lane's component is at byte offset PB j from the row start; 32-bit offsets from
  // a wave-uniform base.  The pass reads k-space positions and writes them back, except at the ends
  // of a call (ROW_FWD reads and ROW_INV writes real space).
  const char* __restrict__ base = reinterpret_cast<const char*>(a.psi);
  char* __restrict__ out = reinterpret_cast<char*>(a.psi);
  const LanePos<T> rp = real_pos<N, P>(t), sp = spec_pos<N, P>(t);
  const LanePos<T> in = MODE == ROW_FWD ? rp : sp, to = MODE == ROW_INV ? rp : sp;
  const uint32_t group_stride = static_cast<uint32_t>(a.rows_per_block) * (PB * N);

  double pv[prefetch_per_lane<R, N>()];
  if constexpr (MODE != ROW_FWD) prefetch_partials(a, pv);
  C v[P], nxt[P];
  uint32_t off = static_cast<uint32_t>(row0) * (PB * N) + CB * comp;
  // Load order: the inverse transform starts with the last forward stage, whose butterfly u
  // takes positions u + U k; issuing those loads together lets it start before the rest land.
  constexpr int RL = MODE == ROW_FWD ? P : last_radix<N, P>();
  constexpr int UL = P / RL;
#pragma unroll
  for (int i = 0; i < P; ++i) {
    const int m = i / RL + UL * (i % RL);
    v[m] = *reinterpret_cast<const C*>(base + (off + PB * in.at(m)));
  }
  TwPlain<N, P, R> tr;
  load_twiddles<N>(tr, t, a.tw);
  // spatial Raman tables: the x part is the same for every row of the workgroup
  R hbx_r[P], hby_r[ITERS];
  if constexpr (FULL && STEP) {
#pragma unroll
    for (int m = 0; m < P; ++m) hbx_r[m] = a.hbx[rp.at(m)];
#pragma unroll
    for (int it = 0; it < ITERS; ++it) hby_r[it] = a.hby[row0 + it * a.rows_per_block];
  }
  // the norm's sum, square root and division while the state's loads are in flight
  R s = R(1);
  if constexpr (MODE != ROW_FWD) {
    s = row_scale(a, pv);
    check_scale(a, s, wg);
  }

#pragma unroll
  for (int it = 0; it < ITERS; ++it) {
    if (it + 1 < ITERS) {
#pragma unroll
      for (int i = 0; i < P; ++i) {
        const int m = i / RL + UL * (i % RL);
        nxt[m] = *reinterpret_cast<const C*>(base + (off + group_stride + PB * in.at(m)));
      }
    }
    if constexpr (MODE == ROW_FWD) {
      fwd_pass<N>(v, lds, t, tr);
    } else {
      inv_pass<N>(v, lds, t, tr);
#pragma unroll
      for (int m = 0; m < P; ++m) v[m] = vscale(v[m], s);
      if constexpr (STEP) {
        row_apply_r<N, true, FULL, MODE == ROW_STEP_NLN>(v, a, row0 + it * a.rows_per_block, t, comp == 0, hbx_r,
                                                         FULL ? hby_r[it] : R(0));
        fwd_pass<N>(v, lds, t, tr);
      }
    }
    if constexpr (many_waves<WT, N>()) forget(off);
#pragma unroll
    for (int m = 0; m < P; ++m) store_state<WT>(reinterpret_cast<C*>(out + (off + PB * to.at(m))), v[m]);
    if (it + 1 < ITERS) {
#pragma unroll
      for (int m = 0; m < P; ++m) v[m] = nxt[m];
      off += group_stride;
    }
  }
}

// The general row pass of the splitting variants (one row group per workgroup); see RowVarFlags.
template <int N, bool FULL, int P>
__device__ __forceinline__ void row_var_body(const RowArgs& a, int wg) {
  __shared__ double red[kRedDoubles];
  static_assert(sizeof red <= kStaticLds);
  constexpr int T = N / P;
  const int tid = threadIdx.x;
  const int comp = tid & 1;
  const int pair = tid >> 1;
  const int rloc = pair / T;
  const int t = pair - rloc * T;
  const int row = wg * a.rows_per_block + rloc;
  const LdsView<float2> lds = lds_line<N, float2>(row_lds, rloc, a.rows_per_block, comp);
  const char* __restrict__ base = reinterpret_cast<const char*>(a.psi);
  char* __restrict__ out = reinterpret_cast<char*>(a.psi);
  const uint32_t off = static_cast<uint32_t>(row) * (16u * N) + 8u * comp;
  const int flags = a.var_flags;
  // k-space positions on entry after a column pass, on return after a forward transform
  const LanePos<T> rp = real_pos<N, P>(t), sp = spec_pos<N, P>(t);
  const LanePos<T> in = (flags & VAR_INV) ? sp : rp, to = (flags & VAR_FWD) ? sp : rp;

  double pv[prefetch_per_lane<float, N>()];
  prefetch_partials(a, pv);
  float2 v[P];
#pragma unroll
  for (int m = 0; m < P; ++m) v[m] = *reinterpret_cast<const float2*>(base + (off + 16u * in.at(m)));
  TwPlain<N, P> tr;
  load_twiddles<N>(tr, t, a.tw);
  float hbx_r[P], hb_row = 0.0f;
  if constexpr (FULL) {
#pragma unroll
    for (int m = 0; m < P; ++m) hbx_r[m] = a.hbx[rp.at(m)] * a.hfrac;
    hb_row = a.hby[row] * a.hfrac;
  }
  const bool mid = (flags & VAR_MID_SCALE) != 0;
  const float norm_scale = row_scale(a, pv);
  check_scale(a, norm_scale, wg);
  if (flags & VAR_INV) {
    inv_pass<N>(v, lds, t, tr);
    const float s = mid ? a.scale : norm_scale;
#pragma unroll
    for (int m = 0; m < P; ++m) v[m] = vscale(v[m], s);
  }
  for (int r = 0; r < a.var_r; ++r) {
    if (a.var_nln) row_apply_r<N, true, FULL, true>(v, a, row, t, comp == 0, hbx_r, hb_row);
    else row_apply_r<N, true, FULL, false>(v, a, row, t, comp == 0, hbx_r, hb_row);
    if (mid && r == 0) {
#pragma unroll
      for (int m = 0; m < P; ++m) v[m] = vscale(v[m], norm_scale);
    }
  }
  if (flags & VAR_NORM_OUT) {
    double acc = 0.0;
#pragma unroll
    for (int m = 0; m < P; ++m) acc += double(v[m].x) * double(v[m].x) + double(v[m].y) * double(v[m].y);
    acc = block_sum(acc, red);
    if (tid == 0) a.partials_out[wg] = acc;
  }
  if (flags & VAR_FWD) fwd_pass<N>(v, lds, t, tr);
  if (!(flags & VAR_NO_STORE)) {
#pragma unroll
    for (int m = 0; m < P; ++m) store_state<true>(reinterpret_cast<float2*>(out + (off + 16u * to.at(m))), v[m]);
  }
}

}  // namespace sgpe
