// Device building blocks of the split-step solver's step kernels: register-resident Stockham FFT
// passes, the (U - 1) sine/cosine helpers of the unit-modulus real-space propagators, lane-pair
// exchange and fp64 reductions.
//
// FFT organisation (transform length N, P points per lane, P in {4, 8, 16}): T = N/P lanes own one
// transform, lane t holding the P positions = t mod T; in the step kernels each lane owns one spinor
// component and the neighbouring lane the other component of the same positions.  Each Stockham stage
// of radix R (P, then a smaller remainder) performs P/R butterflies per lane on registers; the outputs
// of every stage but the last go through LDS, and the last stage's outputs land back in the lane's own
// registers.  So the first stage reads and the last stage writes positions that are contiguous across
// lanes: global loads and stores are coalesced and no digit-reversal pass exists.  Which register holds
// which of its positions a lane learns from real_pos (before the forward transform, after the inverse)
// and spec_pos (between them).  The inverse transform is the exact inverse of the forward one (see
// "Step-kernel transforms" below).
#pragma once

#include <hip/hip_runtime.h>

#include "sgpe_internal.hpp"

namespace sgpe {

// ---------------------------------------------------------------------------------------------
// Complex arithmetic on float2 (one complex) and float4 (two complexes sharing the operation).
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ float2 vadd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float2 vsub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ float2 vneg(float2 a) { return make_float2(-a.x, -a.y); }
__device__ __forceinline__ float2 vscale(float2 a, float s) { return make_float2(a.x * s, a.y * s); }
__device__ __forceinline__ float4 vadd(float4 a, float4 b) {
  return make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w);
}
__device__ __forceinline__ float4 vsub(float4 a, float4 b) {
  return make_float4(a.x - b.x, a.y - b.y, a.z - b.z, a.w - b.w);
}
__device__ __forceinline__ float4 vneg(float4 a) { return make_float4(-a.x, -a.y, -a.z, -a.w); }
__device__ __forceinline__ float4 vscale(float4 a, float s) {
  return make_float4(a.x * s, a.y * s, a.z * s, a.w * s);
}
__device__ __forceinline__ double2 vadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 vsub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ double2 vneg(double2 a) { return make_double2(-a.x, -a.y); }
__device__ __forceinline__ double2 vscale(double2 a, double s) { return make_double2(a.x * s, a.y * s); }

// The real type of a complex type (the complex types of a precision are in sgpe_internal.hpp).
template <class C> struct RealOf;
template <> struct RealOf<float2> { using T = float; };
template <> struct RealOf<double2> { using T = double; };
__device__ __forceinline__ float2 mk2(float x, float y) { return make_float2(x, y); }
__device__ __forceinline__ double2 mk2(double x, double y) { return make_double2(x, y); }
// fp32 intrinsics for float (the complex64 code is unchanged by the templating), fp64 for double
__device__ __forceinline__ float fma_(float a, float b, float c) { return fmaf(a, b, c); }
__device__ __forceinline__ double fma_(double a, double b, double c) { return fma(a, b, c); }
__device__ __forceinline__ float exp_(float x) { return expf(x); }
__device__ __forceinline__ double exp_(double x) { return exp(x); }
__device__ __forceinline__ float sqrt_(float x) { return sqrtf(x); }
__device__ __forceinline__ double sqrt_(double x) { return sqrt(x); }
__device__ __forceinline__ float fmax_(float a, float b) { return fmaxf(a, b); }
__device__ __forceinline__ double fmax_(double a, double b) { return fmax(a, b); }
__device__ __forceinline__ float fabs_(float x) { return fabsf(x); }
__device__ __forceinline__ double fabs_(double x) { return fabs(x); }

// ---------------------------------------------------------------------------------------------
// State stores of the step kernels.  Consecutive passes split the grid between workgroups by
// rows, then by columns, so almost every point a pass writes is next read on another XCD, whose
// L2 it must leave first.  A plain store parks the line dirty in the writer's L2, and the end of
// the kernel writes back every XCD's dirty lines in one burst that the next kernel then waits
// for.  A device-scope store goes through the L2 to the memory side as it is issued, so that
// traffic overlaps the rest of the pass.  Relaxed order: the scope is the only property wanted
// (every point has a single writer in a pass, and kernel boundaries order the passes).
// Measured per launch kind: write-through wins for single-instance complex64 passes (one round
// of workgroups, nothing behind the last stores); batched launches, whose later workgroups
// already overlap the write-back, and complex128 points (two 8-byte device-scope stores per
// 16-byte component) are faster with plain stores.
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ void store_through(float2* p, float2 v) {
  unsigned long long b;
  __builtin_memcpy(&b, &v, sizeof b);
  __hip_atomic_store(reinterpret_cast<unsigned long long*>(p), b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <bool WT, class C>
__device__ __forceinline__ void store_state(C* p, C v) {
  if constexpr (WT && sizeof(C) == sizeof(float2)) {
    store_through(p, v);
  } else {
    *p = v;
  }
}

// Makes the compiler form anew what it would derive from x, instead of holding what it derived earlier
// across the transforms: the offsets of a pass's loads, wanted again by its stores, take a register per
// point.  Worth it where the registers decide how many waves are resident (row pass at 16 points per
// lane: 142 -> 123 VGPRs, 168 -> 138 with a spatial Raman coupling; column pass 126 -> 90): batches,
// complex128 and lines of 2048 points and more (24-instance sweep 15.0 -> 14.7 ms, complex128 at 1024^2
// 42.4 -> 40.5 us per step, 2048^2 90.0 -> 88.5).  A single complex64 grid of shorter lines is resident
// as a whole either way, and the offsets then only delay its stores (1024^2: 23.4 -> 23.8 us per step).
template <bool WT, int N>
constexpr bool many_waves() { return !WT || N >= 2048; }
__device__ __forceinline__ void forget(uint32_t& x) { asm volatile("" : "+v"(x)); }

// ---------------------------------------------------------------------------------------------
// Batched launches (grid x = work items of one instance, grid y = instances).  The dispatcher
// deals a launch's workgroups to the eight XCDs in turn, by linear workgroup index (x fastest),
// continuing its rotation from where the previous launch left it.  Reading the grid as
// instance-major (instance, item) pairs and giving the workgroups L = k mod 8 the k-th eighth of
// that sequence keeps all of an instance's items on one XCD within a launch; when consecutive
// launches start the rotation at the same XCD (every launch of a batch has a multiple of 8
// workgroups), a pass also reads what the previous pass wrote into the same L2.  The map is a
// bijection whenever the grid holds a multiple of 8 workgroups (the identity otherwise); results do
// not depend on where a workgroup runs.
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ int2 batch_item() {
  const unsigned gx = gridDim.x, total = gx * gridDim.y;
  unsigned l = blockIdx.y * gx + blockIdx.x;
  if ((total & 7u) == 0) l = (l & 7u) * (total >> 3) + (l >> 3);
  return make_int2(int(l / gx), int(l % gx));   // (instance, item)
}

// ---------------------------------------------------------------------------------------------
// Positions of a lane's registers: m T + t, or -- where a stage works with signed digits (below) --
// that sequence rotated by one register, (m - 1) T + t with register 0 wrapping to the end.
// ---------------------------------------------------------------------------------------------
template <int STEP>
struct LanePos {
  int b, p0;   // register m > 0 holds b + STEP m (b may be negative), register 0 holds p0
  __device__ __forceinline__ int at(int m) const { return m == 0 ? p0 : b + STEP * m; }
};

// ---------------------------------------------------------------------------------------------
// LDS addressing: a transform's N positions occupy N + N/16 slots (one pad slot per 16 positions) of
// two values, the components of a line interleaved.  The lines of a workgroup follow one another,
// each kLdsSkew / lines bytes further than its slots: lanes that own neighbouring lines (column tiles)
// would else meet in the same banks.  A lane's accesses of a stage are then one register and constants;
// with the lines interleaved slot by slot, a stride only the launch knows, each took an address of its
// own (that change took the column pass at 1024 points from 213 to 147 VGPRs).  Skews of 0, 128 and 256 bytes: 28.8, 24.6 and
// 25.7 us per step at 1024^2 (imaginary time, paired accesses).  Both changes: 24.3 -> 24.0 us per step
// at 1024^2 in imaginary time and 17.7 -> 16.6 in real time, 7.8 -> 7.4 at 64^2, the 24-instance sweep
// 17.0 -> 16.3 ms.
// ---------------------------------------------------------------------------------------------
// A value in one 8-byte access.  Volatile keeps the compiler from pairing accesses into the two-address
// forms: ds_read2_b64 took 4.4 LDS cycles per value and wave in these exchanges, two single reads 3.7.
// (complex128 values are 16 bytes and have no such form.)
using LdsWord = volatile __attribute__((address_space(3))) unsigned long long;
__device__ __forceinline__ float2 lds_get(const float2* p) {
  const unsigned long long b = *(const LdsWord*)(p);
  float2 v;
  __builtin_memcpy(&v, &b, sizeof v);
  return v;
}
__device__ __forceinline__ void lds_put(float2* p, float2 v) {
  unsigned long long b;
  __builtin_memcpy(&b, &v, sizeof b);
  *(LdsWord*)(p) = b;
}
__device__ __forceinline__ double2 lds_get(const double2* p) { return *p; }
__device__ __forceinline__ void lds_put(double2* p, double2 v) { *p = v; }

template <class V>
struct LdsView {
  V* base;     // slot 0 of this lane's line and component
  static __device__ __forceinline__ int slot(int pos) { return pos + (pos >> 4); }
  // the address of position pos.at(m); steps of a multiple of 16 positions are steps of a fixed number
  // of slots, so the lane's one base serves every m > 0
  template <int STEP>
  __device__ __forceinline__ V* at(const LanePos<STEP>& pos, int m) const {
    if constexpr (STEP % 16 == 0) {
      return m == 0 ? base + 2 * slot(pos.p0) : (base + 2 * slot(pos.b)) + 2 * (STEP / 16 * 17) * m;
    } else {
      return base + 2 * slot(pos.at(m));
    }
  }
  template <int STEP>
  __device__ __forceinline__ V get(const LanePos<STEP>& pos, int m) const { return lds_get(at(pos, m)); }
  template <int STEP>
  __device__ __forceinline__ void put(const LanePos<STEP>& pos, int m, V v) const { lds_put(at(pos, m), v); }
};
// The view of line `line` of `lines` (a power of two) of length N.
template <int N, class V>
__device__ __forceinline__ LdsView<V> lds_line(unsigned char* lds, int line, int lines, int comp) {
  const int skew = ((line * kLdsSkew) >> __builtin_ctz(lines)) & -int(sizeof(V));
  return {reinterpret_cast<V*>(lds + line * (2 * (N + N / 16) * int(sizeof(V))) + skew) + comp};
}

// ---------------------------------------------------------------------------------------------
// Step-kernel transforms: a forward transform with rounded roots, and its exact inverse.
//
// A transform with rounded roots is a slightly perturbed DFT.  Followed by the textbook inverse
// (conjugate roots), the round trip is not the identity: rounded roots have |w| != 1, and that same
// map is re-applied every step (a coherent drift).  Here every rotation by an angle phi is three
// shears (lifting steps)
//     x += p y,  y -= u x,  x += p y,     p = tan(phi / 2), u = sin(phi),
// and its inverse the same shears with the signs turned, which undoes them exactly in exact arithmetic
// whatever p and u were rounded to.  The inverse transform undoes the forward one stage by stage, so
// the pair is an exact inverse, the round trip carries only unbiased rounding, and the rounded
// constants enter the split step only through commutators with the step's operators, O(dt eps) per step.
// A rotation costs 3 instructions either way (a rounded complex product takes 4, its exact inverse 8
// and two more for the root's modulus correction) and a root 2 registers.
//
// Shears are well conditioned for |phi| <= pi/2 (p <= 1), and all roots stay there: a stage of radix R
// that combines R transforms of length L rotates by 2 pi s r / (R L), and both s and r are taken as
// signed digits, -L/2 <= s < L/2 and -R/2 < r <= R/2 (the residues beyond the middle counted from
// above).  A signed r shifts the subsequence its transform runs over by one period, a signed s the
// index k of the outputs, so both only rotate a sequence of P positions by one (LanePos); no data moves.
// And the root of -r is the root of r with the shears' signs turned, so a butterfly of radix R holds
// R/2 roots instead of R - 1: 32 registers of roots at N = 1024 and P = 16, where rounded roots with
// modulus corrections took 81.
// The forward error and the round trip's (against fp64, random data, N = 16 to 4096) are those of
// rounded roots or smaller: 1.07e-7 and 1.33e-7 at N = 1024, P = 16, against 1.09e-7 and 1.35e-7.
// Larger grids are bound by instruction issue at the two waves per SIMD that the registers allow; a
// row pass at 1024 points went from 1945 to 1658 VALU instructions and from 192 to 142 VGPRs, the column
// pass from 1990 to 1663 instructions.  Per step, rounded roots -> shears: 26.8 -> 24.2 us at
// 1024^2 and 135 -> 118 us at 2048^2 (imaginary time), 20.0 -> 17.5 us at 1024^2 (real time).
// ---------------------------------------------------------------------------------------------
// p and u of the fixed rotations by pi/8, pi/4 and 3 pi/8
template <class T> struct Roots {
  static constexpr T P1 = T(0.198912367379658006912), U1 = T(0.382683432365089771728);
  static constexpr T P2 = T(0.414213562373095048802), U2 = T(0.707106781186547524401);
  static constexpr T P3 = T(0.668178637919298919998), U3 = T(0.923879532511286756128);
};

// a e^{-i phi}, and its exact inverse (which is a e^{+i phi})
template <class C, class T = typename RealOf<C>::T>
__device__ __forceinline__ C rot_neg(C a, T p, T u) {
  const T x = fma_(p, a.y, a.x);
  const T y = fma_(-u, x, a.y);
  return mk2(fma_(p, y, x), y);
}
template <class C, class T = typename RealOf<C>::T>
__device__ __forceinline__ C rot_pos(C a, T p, T u) {
  const T x = fma_(-p, a.y, a.x);
  const T y = fma_(u, x, a.y);
  return mk2(fma_(-p, y, x), y);
}
template <class C>
__device__ __forceinline__ C pf_rot90(C a) { return mk2(a.y, -a.x); }   // * (-i)
template <class C>
__device__ __forceinline__ C pi_rot90(C a) { return mk2(-a.y, a.x); }   // * (+i)
// * W16^k (k = 1, 2, 3) and its exact inverse
template <int K, class C>
__device__ __forceinline__ C pf_rot(C a) {
  using R = Roots<typename RealOf<C>::T>;
  if constexpr (K == 1) return rot_neg(a, R::P1, R::U1);
  else if constexpr (K == 2) return rot_neg(a, R::P2, R::U2);
  else return rot_neg(a, R::P3, R::U3);
}
template <int K, class C>
__device__ __forceinline__ C pi_rot(C a) {
  using R = Roots<typename RealOf<C>::T>;
  if constexpr (K == 1) return rot_pos(a, R::P1, R::U1);
  else if constexpr (K == 2) return rot_pos(a, R::P2, R::U2);
  else return rot_pos(a, R::P3, R::U3);
}

// forward small DFTs (sign -1)
template <class C>
__device__ __forceinline__ void pf_dft4(C& a0, C& a1, C& a2, C& a3) {
  const C t0 = vadd(a0, a2), t1 = vsub(a0, a2);
  const C t2 = vadd(a1, a3), t3 = pf_rot90(vsub(a1, a3));
  a0 = vadd(t0, t2);
  a2 = vsub(t0, t2);
  a1 = vadd(t1, t3);
  a3 = vsub(t1, t3);
}
// its exact inverse times 4 (conjugate structure; the constants are exact)
template <class C>
__device__ __forceinline__ void pi_dft4(C& a0, C& a1, C& a2, C& a3) {
  const C t0 = vadd(a0, a2), t1 = vsub(a0, a2);
  const C t2 = vadd(a1, a3), t3 = pi_rot90(vsub(a1, a3));
  a0 = vadd(t0, t2);
  a2 = vsub(t0, t2);
  a1 = vadd(t1, t3);
  a3 = vsub(t1, t3);
}

template <class C>
__device__ __forceinline__ void pf_dft8(C (&a)[8]) {
  C e0 = a[0], e1 = a[2], e2 = a[4], e3 = a[6];
  C o0 = a[1], o1 = a[3], o2 = a[5], o3 = a[7];
  pf_dft4(e0, e1, e2, e3);
  pf_dft4(o0, o1, o2, o3);
  o1 = pf_rot<2>(o1);
  o2 = pf_rot90(o2);
  o3 = pf_rot90(pf_rot<2>(o3));
  a[0] = vadd(e0, o0); a[4] = vsub(e0, o0);
  a[1] = vadd(e1, o1); a[5] = vsub(e1, o1);
  a[2] = vadd(e2, o2); a[6] = vsub(e2, o2);
  a[3] = vadd(e3, o3); a[7] = vsub(e3, o3);
}
// exact inverse of pf_dft8, times 8
template <class C>
__device__ __forceinline__ void pi_dft8(C (&a)[8]) {
  C e0 = vadd(a[0], a[4]), o0 = vsub(a[0], a[4]);
  C e1 = vadd(a[1], a[5]), o1 = vsub(a[1], a[5]);
  C e2 = vadd(a[2], a[6]), o2 = vsub(a[2], a[6]);
  C e3 = vadd(a[3], a[7]), o3 = vsub(a[3], a[7]);
  o1 = pi_rot<2>(o1);
  o2 = pi_rot90(o2);
  o3 = pi_rot<2>(pi_rot90(o3));
  pi_dft4(e0, e1, e2, e3);
  pi_dft4(o0, o1, o2, o3);
  a[0] = e0; a[2] = e1; a[4] = e2; a[6] = e3;
  a[1] = o0; a[3] = o1; a[5] = o2; a[7] = o3;
}

// forward 16-point DFT (4x4; input r = r1 + 4 r2, output k = k2 + 4 k1)
template <class C>
__device__ __forceinline__ void pf_dft16(C (&a)[16]) {
#pragma unroll
  for (int r1 = 0; r1 < 4; ++r1) pf_dft4(a[r1], a[r1 + 4], a[r1 + 8], a[r1 + 12]);
  a[5] = pf_rot<1>(a[5]);                                // W16^1
  a[9] = pf_rot<2>(a[9]);                                // W16^2
  a[13] = pf_rot<3>(a[13]);                              // W16^3
  a[6] = pf_rot<2>(a[6]);                                // W16^2
  a[10] = pf_rot90(a[10]);                               // W16^4
  a[14] = pf_rot90(pf_rot<2>(a[14]));                    // W16^6
  a[7] = pf_rot<3>(a[7]);                                // W16^3
  a[11] = pf_rot90(pf_rot<2>(a[11]));                    // W16^6
  a[15] = vneg(pf_rot<1>(a[15]));                        // W16^9 = -W16^1
#pragma unroll
  for (int k2 = 0; k2 < 4; ++k2) pf_dft4(a[4 * k2], a[4 * k2 + 1], a[4 * k2 + 2], a[4 * k2 + 3]);
  C t[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) t[i] = a[i];
#pragma unroll
  for (int k1 = 0; k1 < 4; ++k1)
#pragma unroll
    for (int k2 = 0; k2 < 4; ++k2) a[k2 + 4 * k1] = t[k1 + 4 * k2];
}
// exact inverse of pf_dft16, times 16: the same steps undone in reverse order
template <class C>
__device__ __forceinline__ void pi_dft16(C (&a)[16]) {
  C t[16];
#pragma unroll
  for (int k1 = 0; k1 < 4; ++k1)
#pragma unroll
    for (int k2 = 0; k2 < 4; ++k2) t[k1 + 4 * k2] = a[k2 + 4 * k1];
#pragma unroll
  for (int k2 = 0; k2 < 4; ++k2) pi_dft4(t[4 * k2], t[4 * k2 + 1], t[4 * k2 + 2], t[4 * k2 + 3]);
  t[5] = pi_rot<1>(t[5]);
  t[9] = pi_rot<2>(t[9]);
  t[13] = pi_rot<3>(t[13]);
  t[6] = pi_rot<2>(t[6]);
  t[10] = pi_rot90(t[10]);
  t[14] = pi_rot<2>(pi_rot90(t[14]));
  t[7] = pi_rot<3>(t[7]);
  t[11] = pi_rot<2>(pi_rot90(t[11]));
  t[15] = pi_rot<1>(vneg(t[15]));
#pragma unroll
  for (int r1 = 0; r1 < 4; ++r1) pi_dft4(t[r1], t[r1 + 4], t[r1 + 8], t[r1 + 12]);
#pragma unroll
  for (int i = 0; i < 16; ++i) a[i] = t[i];
}

template <int R, class C>
__device__ __forceinline__ void pf_dft(C (&a)[R]) {
  if constexpr (R == 2) {
    const C t = a[0];
    a[0] = vadd(t, a[1]);
    a[1] = vsub(t, a[1]);
  } else if constexpr (R == 4) {
    pf_dft4(a[0], a[1], a[2], a[3]);
  } else if constexpr (R == 8) {
    pf_dft8(a);
  } else {
    static_assert(R == 16, "radix");
    pf_dft16(a);
  }
}
template <int R, class C>
__device__ __forceinline__ void pi_dft(C (&a)[R]) {
  if constexpr (R == 2) {
    const C t = a[0];
    a[0] = vadd(t, a[1]);
    a[1] = vsub(t, a[1]);
  } else if constexpr (R == 4) {
    pi_dft4(a[0], a[1], a[2], a[3]);
  } else if constexpr (R == 8) {
    pi_dft8(a);
  } else {
    static_assert(R == 16, "radix");
    pi_dft16(a);
  }
}

// Step-kernel transforms with P points per thread (P = 4, 8 or 16; T = N / P threads per
// transform).  Stages have radix P, then the remainder.
template <int N, int P, int L>
constexpr int stage_radix() { return N / L >= P ? P : N / L; }

// Radix of the last stage of a length-N transform.
template <int N, int P, int L = 1>
constexpr int last_radix() {
  constexpr int REM = N / L;
  if constexpr (REM <= P) return REM;
  else return last_radix<N, P, L * P>();
}

// The stage that combines transforms of length L reads, for the output offset o, the offsets
// o + (N / R L) r with signed r.  The offsets of a stage's inputs to the later stages therefore run over
// (h - N / L, h] instead of [0, N / L), with this h for the offsets of the stage's own outputs.
template <int N, int P, int L>
constexpr int offset_top() {
  constexpr int LN = L * stage_radix<N, P, L>();   // length after this stage
  if constexpr (LN == N) return 0;
  else return stage_radix<N, P, LN>() / 2 * (N / (LN * stage_radix<N, P, LN>())) + offset_top<N, P, LN>();
}

// Positions of the lane's inputs of the stage at length L: rotated where its offset is a negative one
// (only the last stage, whose one offset is 0, has P != R and it is never rotated).
template <int N, int P, int L = 1>
__device__ __forceinline__ LanePos<N / P> stage_in_pos(int t) {
  constexpr int T = N / P;
  if constexpr (N / L <= P) {
    return {t, t};
  } else {
    const bool neg = t / L > offset_top<N, P, L>();
    return {neg ? t - T : t, neg ? t + (N - T) : t};
  }
}
// Positions (within the array after the stage) of the lane's outputs of a stage of radix P at length L.
template <int N, int P, int L>
__device__ __forceinline__ LanePos<L> stage_out_pos(int t) {
  const int s = t & (L - 1), o = (t / L) * (P * L) + s;
  if constexpr (L == 1) {
    return {o, o};
  } else {
    const bool neg = s >= L / 2;
    return {neg ? o - L : o, neg ? o + L * (P - 1) : o};
  }
}
// The lane's positions in real space (the forward transform's input) and in k-space (its output).
template <int N, int P>
__device__ __forceinline__ LanePos<N / P> real_pos(int t) { return stage_in_pos<N, P>(t); }
template <int N, int P>
__device__ __forceinline__ LanePos<N / P> spec_pos(int t) {
  constexpr int T = N / P;
  if constexpr (T > 1 && last_radix<N, P>() == P) return stage_out_pos<N, P, T>(t);
  else return {t, t};   // a smaller last radix rotates at compile time (last_reg)
}
// The register of output k of the last stage's butterfly u (U butterflies of radix R).
template <int P, int R>
constexpr int last_reg(int u, int k) {
  constexpr int U = P / R;
  return u + U * (U > 1 && u >= U / 2 ? (k + R - 1) % R : k);
}

// Stage roots a thread holds: the first stage (L = 1) needs none; a later one of radix R the (p, u) of
// 2 pi s r / (R L) for its P/R butterflies and r = 1..R/2.
template <int N, int P, int L = 1>
constexpr int tw_count_p() {
  constexpr int R = stage_radix<N, P, L>();
  constexpr int here = L > 1 ? (P / R) * (R / 2) : 0;
  if constexpr (R * L == N) return here;
  else return here + tw_count_p<N, P, L * R>();
}

template <int N, int P = 16, class T = float>
struct TwPlain {
  static constexpr int COUNT = tw_count_p<N, P>() > 0 ? tw_count_p<N, P>() : 1;
  cplx_t<T> pu[COUNT];
};

// tw: the (p, u) of 2 pi j / N at entry j + N/4, |j| <= N/4.  Loaded once per kernel (they depend only on
// the thread index).
template <int N, int P, int L = 1, int BASE = 0, class TR>
__device__ __forceinline__ void load_twiddles(TwPlain<N, P, TR>& tr, int t, const cplx_t<TR>* __restrict__ tw) {
  using C = cplx_t<TR>;
  constexpr int T = N / P;
  constexpr int R = stage_radix<N, P, L>();
  constexpr int U = P / R;
  if constexpr (L > 1) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int s0 = (t + T * u) & (L - 1);
      const int s = s0 >= L / 2 ? s0 - L : s0;
      // byte offset of entry N/4 + s r N/(R L), 32-bit from the uniform table base
      const int d = s * int(sizeof(C) * (N / (R * L)));
      int o = int(sizeof(C)) * (N / 4);
#pragma unroll
      for (int r = 1; r <= R / 2; ++r) {
        o += d;
        tr.pu[BASE + u * (R / 2) + (r - 1)] =
            *reinterpret_cast<const C*>(reinterpret_cast<const char*>(tw) + static_cast<uint32_t>(o));
      }
    }
  }
  if constexpr (R * L != N) {
    constexpr int NEXT = BASE + (L > 1 ? U * (R / 2) : 0);
    load_twiddles<N, P, L * R, NEXT>(tr, t, tw);
  }
}

// forward stage
template <int N, int P, int L, int BASE, class C, class TR>
__device__ __forceinline__ void pf_stage(C (&v)[P], const LdsView<C>& lds, int t, const TwPlain<N, P, TR>& tr) {
  constexpr int R = stage_radix<N, P, L>();
  constexpr int U = P / R;
  constexpr bool LAST = R * L == N;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    C a[R];
#pragma unroll
    for (int r = 0; r < R; ++r) a[r] = v[u + U * r];
    if constexpr (L > 1) {
#pragma unroll
      for (int r = 1; r < R; ++r) {
        const C w = tr.pu[BASE + u * (R / 2) + ((r <= R / 2 ? r : R - r) - 1)];
        a[r] = r <= R / 2 ? rot_neg(a[r], w.x, w.y) : rot_pos(a[r], w.x, w.y);
      }
    }
    pf_dft<R>(a);
    if constexpr (LAST) {
#pragma unroll
      for (int k = 0; k < R; ++k) v[last_reg<P, R>(u, k)] = a[k];
    } else {
      const auto pos = stage_out_pos<N, P, L>(t);
#pragma unroll
      for (int k = 0; k < R; ++k) lds.put(pos, k, a[k]);
    }
  }
}

// Forward length-N transform (positions real_pos in, spec_pos out).
template <int N, int L = 1, int BASE = 0, int P, class C, class TR>
__device__ __forceinline__ void fwd_pass(C (&v)[P], const LdsView<C>& lds, int t, const TwPlain<N, P, TR>& tr) {
  constexpr int R = stage_radix<N, P, L>();
  if constexpr (R * L == N) {
    pf_stage<N, P, L, BASE>(v, lds, t, tr);
  } else {
    pf_stage<N, P, L, BASE>(v, lds, t, tr);
    __syncthreads();
    const auto pos = stage_in_pos<N, P, L * R>(t);
#pragma unroll
    for (int m = 0; m < P; ++m) v[m] = lds.get(pos, m);
    __syncthreads();
    constexpr int NEXT = BASE + (L > 1 ? (P / R) * (R / 2) : 0);
    fwd_pass<N, L * R, NEXT>(v, lds, t, tr);
  }
}

// Inverse stage: the forward stage's outputs (from LDS, or the registers for the last stage)
// through the exact inverse butterfly and inverse rotations, into registers {u + U r}.
template <int N, int P, int L, int BASE, class C, class TR>
__device__ __forceinline__ void pi_stage(C (&v)[P], const LdsView<C>& lds, int t, const TwPlain<N, P, TR>& tr) {
  constexpr int R = stage_radix<N, P, L>();
  constexpr int U = P / R;
  constexpr bool LAST = R * L == N;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    C a[R];
    if constexpr (LAST) {
#pragma unroll
      for (int k = 0; k < R; ++k) a[k] = v[last_reg<P, R>(u, k)];
    } else {
      const auto pos = stage_out_pos<N, P, L>(t);
#pragma unroll
      for (int k = 0; k < R; ++k) a[k] = lds.get(pos, k);
    }
    pi_dft<R>(a);
    if constexpr (L > 1) {
#pragma unroll
      for (int r = 1; r < R; ++r) {
        const C w = tr.pu[BASE + u * (R / 2) + ((r <= R / 2 ? r : R - r) - 1)];
        a[r] = r <= R / 2 ? rot_pos(a[r], w.x, w.y) : rot_neg(a[r], w.x, w.y);
      }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) v[u + U * r] = a[r];
  }
}

// Exact inverse of fwd_pass, times N: the stages undone in reverse order.  All threads of the
// workgroup call it; on return every LDS read is complete.
template <int N, int L = 1, int BASE = 0, int P, class C, class TR>
__device__ __forceinline__ void inv_pass(C (&v)[P], const LdsView<C>& lds, int t, const TwPlain<N, P, TR>& tr) {
  constexpr int R = stage_radix<N, P, L>();
  if constexpr (R * L == N) {
    pi_stage<N, P, L, BASE>(v, lds, t, tr);
  } else {
    constexpr int NEXT = BASE + (L > 1 ? (P / R) * (R / 2) : 0);
    inv_pass<N, L * R, NEXT>(v, lds, t, tr);
    // undo the forward's reads from LDS, then this stage
    const auto pos = stage_in_pos<N, P, L * R>(t);
#pragma unroll
    for (int m = 0; m < P; ++m) lds.put(pos, m, v[m]);
    __syncthreads();
    pi_stage<N, P, L, BASE>(v, lds, t, tr);
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------------------------
// Lane pairs: lanes 2j and 2j+1 hold the two spinor components of the same positions.  The
// partner's value comes over the DPP quad permutation [1,0,3,2] (no LDS traffic, no barrier).
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ float pair_swap(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0xB1, 0xF, 0xF, false));
}
__device__ __forceinline__ float2 pair_swap(float2 x) { return make_float2(pair_swap(x.x), pair_swap(x.y)); }
__device__ __forceinline__ double pair_swap(double x) {
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), 0xB1, 0xF, 0xF, false);
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), 0xB1, 0xF, 0xF, false);
  return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double2 pair_swap(double2 x) { return make_double2(pair_swap(x.x), pair_swap(x.y)); }

// ---------------------------------------------------------------------------------------------
// (cos(phi) - 1, sin(phi)) with relative accuracy on both parts for small |phi|, and
// sin(phi)/phi.  Cody-Waite reduction by pi/2 (the first product is exact inside the FMA for
// |k| < 2^10), Taylor polynomials on |r| <= pi/4.
// ---------------------------------------------------------------------------------------------
struct SinCosM1 {
  float cm1, s, sinc;
};

__host__ __device__ __forceinline__ SinCosM1 sincos_m1_reduced(float phi) {
  const float k = rintf(phi * 0.636619772367581343f);
  float r = fmaf(-k, 1.57079637050628662f, phi);   // pi/2 hi
  r = fmaf(-k, -4.37113900018624283e-8f, r);        // pi/2 lo
  const float r2 = r * r;
  const float ps = r2 * fmaf(r2, fmaf(r2, fmaf(r2, 2.75573192e-6f, -1.98412698e-4f), 8.33333333e-3f),
                             -1.66666667e-1f);   // sin r / r - 1
  const float sr = fmaf(r, ps, r);
  const float cr_m1 = r2 * fmaf(r2, fmaf(r2, fmaf(r2, fmaf(r2, -2.75573192e-7f, 2.48015873e-5f),
                                                  -1.38888889e-3f), 4.16666667e-2f), -0.5f);
  const int q = static_cast<int>(k) & 3;
  SinCosM1 out;
  if (q == 0) {
    // cos and sin have period 2 pi, so the reduced values serve for every k = 0 mod 4; sin(phi)/phi
    // does not: (1 + ps) = sin(r)/r equals it only for k = 0
    out.cm1 = cr_m1;
    out.s = sr;
    out.sinc = k == 0.0f ? 1.0f + ps : sr / phi;
  } else {
    const float cr = cr_m1 + 1.0f;
    const float c = q == 1 ? -sr : (q == 2 ? -cr : sr);
    out.s = q == 1 ? cr : (q == 2 ? -sr : -cr);
    out.cm1 = c - 1.0f;
    out.sinc = out.s / phi;
  }
  return out;
}

// |phi| <= pi/4 needs no reduction; the polynomials alone are accurate there.
__host__ __device__ __forceinline__ SinCosM1 sincos_m1_small(float phi) {
  const float r2 = phi * phi;
  const float ps = r2 * fmaf(r2, fmaf(r2, fmaf(r2, 2.75573192e-6f, -1.98412698e-4f), 8.33333333e-3f),
                             -1.66666667e-1f);
  SinCosM1 out;
  out.s = fmaf(phi, ps, phi);
  out.cm1 = r2 * fmaf(r2, fmaf(r2, fmaf(r2, fmaf(r2, -2.75573192e-7f, 2.48015873e-5f),
                                             -1.38888889e-3f), 4.16666667e-2f), -0.5f);
  out.sinc = 1.0f + ps;
  return out;
}

// The same with the routine fixed at compile time: SMALL requires |phi| <= pi/4; the reduced
// routine is exact for every phi and returns the same bits for small ones.  A wave picks one for all
// of its points (see small_angles), so it runs one straight line of code.
template <bool SMALL>
__device__ __forceinline__ SinCosM1 sincos_m1_t(float phi) {
  if constexpr (SMALL) return sincos_m1_small(phi);
  else return sincos_m1_reduced(phi);
}
constexpr float kSmallPhase = 0.785398163f;   // pi/4

// fp64.  |phi| <= pi/4: Taylor polynomials (the first terms left out are below 3e-18).  Beyond: one
// library sincos of phi/2 and the half-angle identities cos(phi) - 1 = -2 sin^2(phi/2), sin(phi) =
// 2 sin(phi/2) cos(phi/2).  The general routine chooses by the angle, so a wave's vote does not change
// results.
struct SinCosM1d {
  double cm1, s, sinc;
};
__device__ __forceinline__ SinCosM1d sincos_m1_small(double phi) {
  const double r = phi * phi;
  double p = -1.0 / 121645100408832000.0;   // sin(phi) / phi - 1 = r p
  p = fma(r, p, 1.0 / 355687428096000.0);
  p = fma(r, p, -1.0 / 1307674368000.0);
  p = fma(r, p, 1.0 / 6227020800.0);
  p = fma(r, p, -1.0 / 39916800.0);
  p = fma(r, p, 1.0 / 362880.0);
  p = fma(r, p, -1.0 / 5040.0);
  p = fma(r, p, 1.0 / 120.0);
  p = fma(r, p, -1.0 / 6.0);
  double q = -1.0 / 6402373705728000.0;     // cos(phi) - 1 = r q
  q = fma(r, q, 1.0 / 20922789888000.0);
  q = fma(r, q, -1.0 / 87178291200.0);
  q = fma(r, q, 1.0 / 479001600.0);
  q = fma(r, q, -1.0 / 3628800.0);
  q = fma(r, q, 1.0 / 40320.0);
  q = fma(r, q, -1.0 / 720.0);
  q = fma(r, q, 1.0 / 24.0);
  q = fma(r, q, -0.5);
  SinCosM1d out;
  p *= r;
  out.s = fma(phi, p, phi);
  out.cm1 = r * q;
  out.sinc = 1.0 + p;
  return out;
}
template <bool SMALL>
__device__ __forceinline__ SinCosM1d sincos_m1_t(double phi) {
  if (SMALL || fabs(phi) <= double(kSmallPhase)) return sincos_m1_small(phi);
  SinCosM1d out;
  double h, c;
  sincos(0.5 * phi, &h, &c);
  out.s = 2.0 * h * c;
  out.cm1 = -2.0 * h * h;
  out.sinc = out.s / phi;
  return out;
}

// exp(x) - 1 for |x| <= kSmallExp: x + x^2 p(x), with p of degree 4 in fp32 (Chebyshev; as a factor
// w + w (exp(x) - 1) the result is within 9.3e-8 of w exp(x), rms 2.6e-8, where a correctly rounded
// exp and a product reach 1.2e-7 and 3.6e-8) and Taylor's of degree 12 in fp64 (the first term left out
// is 0.35^15 / 15! = 1.1e-19).
constexpr float kSmallExp = 0.35f;
__device__ __forceinline__ float expm1_small(float x) {
  float p = fmaf(x, 1.3934535e-3f, 8.3637694e-3f);
  p = fmaf(x, p, 4.16664556e-2f);
  p = fmaf(x, p, 1.66665733e-1f);
  p = fmaf(x, p, 0.5f);
  return fmaf(x * x, p, x);
}
__device__ __forceinline__ double expm1_small(double x) {
  double p = 1.0 / 87178291200.0;
  p = fma(x, p, 1.0 / 6227020800.0);
  p = fma(x, p, 1.0 / 479001600.0);
  p = fma(x, p, 1.0 / 39916800.0);
  p = fma(x, p, 1.0 / 3628800.0);
  p = fma(x, p, 1.0 / 362880.0);
  p = fma(x, p, 1.0 / 40320.0);
  p = fma(x, p, 1.0 / 5040.0);
  p = fma(x, p, 1.0 / 720.0);
  p = fma(x, p, 1.0 / 120.0);
  p = fma(x, p, 1.0 / 24.0);
  p = fma(x, p, 1.0 / 6.0);
  p = fma(x, p, 0.5);
  return fma(x * x, p, x);
}

// True in every lane iff p holds in every active lane of the wave (a wave-uniform value).
__device__ __forceinline__ bool wave_all(bool p) { return __builtin_amdgcn_ballot_w64(!p) == 0; }

// ---------------------------------------------------------------------------------------------
// Deterministic reductions in fp64.
// ---------------------------------------------------------------------------------------------
// Across the wave without LDS traffic: lanes 1, 2, 4 and 8 apart by DPP permutations, rows of 16 and
// halves by the permlane swaps (shuffles through LDS cost two trips of ~100 cycles per step).  Every
// lane ends with the same bits: each step adds the two halves of a group, whichever half a lane is in.
template <int CTRL>
__device__ __forceinline__ double dpp_move(double v) {
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xF, 0xF, false);
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xF, 0xF, false);
  return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double wave_sum(double v) {
  v += dpp_move<0xB1>(v);    // quad_perm [1,0,3,2]
  v += dpp_move<0x4E>(v);    // quad_perm [2,3,0,1]
  v += dpp_move<0x141>(v);   // row_half_mirror: the other quad of eight lanes
  v += dpp_move<0x140>(v);   // row_mirror: the other eight lanes of the row
  {
    const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(v), __double2hiint(v), false, false);
    const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(v), __double2loint(v), false, false);
    v = __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
  }
  {
    const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(v), __double2hiint(v), false, false);
    const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(v), __double2loint(v), false, false);
    v = __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
  }
  return v;
}

// Sum over the workgroup in a fixed order; every thread must call it; red must hold kRedDoubles.
// Result valid in every thread.
__device__ __forceinline__ double block_sum(double v, double* red) {
  const int n = blockDim.x;
  double s = 0.0;
  if ((n & 63) == 0) {
    v = wave_sum(v);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    __syncthreads();
    if (lane == 0) red[wave] = v;
    __syncthreads();
    for (int w = 0; w < (n >> 6); ++w) s += red[w];
  } else {  // a workgroup smaller than one wave (small grids)
    __syncthreads();
    red[threadIdx.x] = v;
    __syncthreads();
    for (int i = 0; i < n; ++i) s += red[i];
  }
  __syncthreads();
  return s;
}

}  // namespace sgpe
