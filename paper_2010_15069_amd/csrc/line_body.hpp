// Device body of the line pass, the one sweep of a real-time step (see line_launch.hpp for the
// kernels and for why one sweep is enough).
#pragma once

#include "col_body.hpp"
#include "row_body.hpp"

namespace sgpe {

extern __shared__ __align__(16) unsigned char line_lds[];

// Lines of length N along the rows (COL = false) or the columns of the state.  P points per lane;
// lanes 2j and 2j+1 hold the two components of the same points, as in the row and column passes,
// whose memory and LDS layouts these are.
//
// Both ops run through one loop body, so an op is the same instructions whether it shares a pass with R
// or has one of its own: a call that leaves its last ops to a later pass gives the bits of one that
// does not.  The 1/N of an op's inverse transform is applied in k-space, where it costs nothing: the
// tables hold (U - 1) / N, and w + (U - 1) w becomes w / N + (U - 1) w / N.  It is a power of two, so
// the roundings are the same; and R sees the state itself, whose densities have N^2 more range than
// those of N times the state (a linear problem, g = 0, with values above 1e19 / N gave inf * 0).
template <int N, bool COL, bool FULL, bool NLN, int P, bool WT, class R>
__device__ __forceinline__ void line_body(const LineArgsT<R>& a, int wg, int ngroups) {
  using C = cplx_t<R>;
  using Q = point_t<R>;
  constexpr int T = N / P;
  constexpr uint32_t PB = sizeof(Q), CB = sizeof(C);   // bytes per point / component
  const int tid = threadIdx.x;
  const int comp = tid & 1;
  const int pair = tid >> 1;
  int line, t, lane_line;
  uint32_t off, pstride;   // of the lane's line, between its positions
  if constexpr (COL) {
    const int sh = __builtin_ctz(a.lines);
    const int cc = pair & (a.lines - 1);
    t = pair >> sh;
    line = (col_group(wg, ngroups) << sh) + cc;
    lane_line = cc;
    off = PB * static_cast<uint32_t>(line) + CB * comp;
    pstride = PB * static_cast<uint32_t>(a.nx);
  } else {
    const int rloc = pair / T;
    t = pair - rloc * T;
    line = wg * a.lines + rloc;
    lane_line = rloc;
    off = static_cast<uint32_t>(line) * (PB * N) + CB * comp;
    pstride = PB;
  }
  const LdsView<C> lds = lds_line<N, C>(line_lds, lane_line, a.lines, comp);
  const LanePos<T> rp = real_pos<N, P>(t), sp = spec_pos<N, P>(t);
  uint32_t off0 = off + static_cast<uint32_t>(rp.p0) * pstride, offb = off + static_cast<uint32_t>(rp.b) * pstride;
  const uint32_t mstride = static_cast<uint32_t>(T) * pstride;
  const char* __restrict__ base = reinterpret_cast<const char*>(a.psi);
  char* __restrict__ out = reinterpret_cast<char*>(a.psi);
  C v[P];
#pragma unroll
  for (int m = 0; m < P; ++m) v[m] = *reinterpret_cast<const C*>(base + (m == 0 ? off0 : offb + mstride * m));
  // In complex128 at 16 points per lane the state takes 64 VGPRs, the roots up to 64, the couplings 32 and
  // the library's sincos the rest: 4096-point lines, whose 512 threads have 256, spilled 105 to 181 of
  // them, and 2048-point columns (256 threads) were left with one wave per SIMD.  There the roots are
  // loaded for each op and the couplings for each R, neither is held across the other, and the op's
  // table values go four points at a time: 21 to 49 spilled, two waves in the columns.  Real time, us
  // per step: 1024 x 4096 with a coupling 251 -> 196 (two sweeps per step took 261), 4096 x 256 48 -> 38,
  // 4096^2 1490 -> 925, 1024 x 2048 69 -> 60.  Rows of 2048 points stay at one wave either way and lost
  // 3-5 %.
  constexpr bool LEAN = sizeof(R) == 8 && P == 16 && N >= (COL ? 2048 : 4096);
  TwPlain<N, P, R> tr;
  if constexpr (!LEAN) load_twiddles<N>(tr, t, a.tw);
  R hb_line[P], hb_cross = R(0);
  auto load_hb = [&](const LanePos<T>& pos) {
#pragma unroll
    for (int m = 0; m < P; ++m) hb_line[m] = a.hbx[pos.at(m)] * a.hfrac;
  };
  if constexpr (FULL) {
    if constexpr (!LEAN) load_hb(rp);
    hb_cross = a.hby[line] * a.hfrac;
  }
  // An op's table values of the lane's points are loaded before the forward transform, so that their
  // latency hides behind it, at 8 or 4 points per lane (complex128 at 64^2: 7.3 us per step, against 7.6
  // loaded where used); at 16 points they would take the registers of another wave (1024-point rows with
  // a coupling: 205 VGPRs instead of 152) and are loaded where used (2048^2: 55 us per step, 61 held;
  // 2048 x 1024 31.2 and 32.7; 1024^2 level).
  constexpr R inv_n = R(1) / R(N);
#pragma unroll 1
  for (int stage = 0; stage < 2; ++stage) {
    const void* const op = stage == 0 ? a.op_pre : a.op_post;
    if (op != nullptr) {
      if constexpr (LEAN) {
        int tt = t;
        asm volatile("" : "+v"(tt));
        load_twiddles<N>(tr, tt, a.tw);
      }
      if constexpr (COL) {
        const C* __restrict__ tab = static_cast<const C*>(op);   // (P(k_y) - 1) / N
        constexpr bool EARLY = P < 16;
        C q[EARLY ? P : 1];
        if constexpr (EARLY) {
#pragma unroll
          for (int m = 0; m < P; ++m) q[m] = tab[sp.at(m)];
        }
        fwd_pass<N>(v, lds, t, tr);
#pragma unroll
        for (int m = 0; m < P; ++m) {
          if (LEAN && m % 4 == 0) __builtin_amdgcn_sched_barrier(0);
          C e;
          if constexpr (EARLY) e = q[m];
          else e = tab[sp.at(m)];
          const C w = v[m];
          v[m] = mk2(fma_(w.x, inv_n, fma_(-e.y, w.y, e.x * w.x)), fma_(w.y, inv_n, fma_(e.y, w.x, e.x * w.y)));
        }
      } else {
        // this component's row of (M'(k_x) - 1) / N, {own, other}
        const Q* __restrict__ tab = static_cast<const Q*>(op);
        constexpr bool EARLY = P < 16;
        Q d[EARLY ? P : 1];
        if constexpr (EARLY) {
#pragma unroll
          for (int m = 0; m < P; ++m) d[m] = tab[2 * sp.at(m) + comp];
        }
        fwd_pass<N>(v, lds, t, tr);
#pragma unroll
        for (int m = 0; m < P; ++m) {
          if (LEAN && m % 4 == 0) __builtin_amdgcn_sched_barrier(0);
          Q e;
          if constexpr (EARLY) e = d[m];
          else e = tab[2 * sp.at(m) + comp];
          const C w = v[m];
          const C o = pair_swap(w);
          const R cr = fma_(-e.w, o.y, fma_(e.z, o.x, fma_(-e.y, w.y, e.x * w.x)));
          const R ci = fma_(e.w, o.x, fma_(e.z, o.y, fma_(e.y, w.x, e.x * w.y)));
          v[m] = mk2(fma_(w.x, inv_n, cr), fma_(w.y, inv_n, ci));
        }
      }
      inv_pass<N>(v, lds, t, tr);
    }
    if (stage == 0) {
#pragma unroll 1
      for (int r = 0; r < a.n_r; ++r) {
        if constexpr (FULL && LEAN) {
          int tt = t;
          asm volatile("" : "+v"(tt));
          load_hb(real_pos<N, P>(tt));
        }
        row_apply_r<N, false, FULL, NLN, NLN || LEAN>(v, a, line, t, comp == 0, hb_line, hb_cross);
      }
    }
  }
  // Formed anew (see forget) the offsets free 28 to 30 VGPRs at 16 points per lane, of 140 to 182: up to one
  // more wave per SIMD, and the wide column workgroups stay within 128 but for a few.  Held: at 4 and 8 points, where
  // four waves and more are resident either way and a pass is one lane's chain of latencies (1024 x 256:
  // 7.9 us per step, 8.3 formed anew; with a spatial coupling 9.1 and 9.4); in rows of 2048 and 4096
  // points, whose grids of few rows are resident as a whole and whose workgroups of 4096 points are not
  // joined by another (4096 x 256: 16.9 and 17.3; 2048 x 256 with a coupling: 12.7 and 12.9); and with a
  // coupling in lines below 1024 points (2048 x 128 at 16 points: 11.9 and 12.7).  Elsewhere, held -> formed
  // anew: 1024^2 16.4 -> 16.1, 512 x 2048 20.0 -> 19.8, 64 x 4096 with a coupling 19.6 -> 18.5.
  if constexpr (!WT || (P == 16 && (COL || N <= 1024) && (!FULL || N >= 1024))) {
    forget(off0);
    forget(offb);
  }
#pragma unroll
  for (int m = 0; m < P; ++m)
    store_state<WT>(reinterpret_cast<C*>(out + (m == 0 ? off0 : offb + mstride * m)), v[m]);
}

}  // namespace sgpe
