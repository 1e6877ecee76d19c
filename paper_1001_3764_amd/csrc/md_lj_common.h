// Pieces shared by the Lennard-Jones kernels (md_lj.hip, md_group.hip): payload access, cross-lane
// exchanges, the pair constants and the FP64 treatment of close contacts and cutoff-band pairs.
#pragma once

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "md_internal.h"

namespace mdk {
namespace {

struct alignas(32) Pay64 {
  double x, y, z, tagbits;
};

__device__ inline int32_t pay_tag(const int4& q) { return q.w; }
__device__ inline int32_t pay_tag(const Pay64& q) { return (int32_t)__double_as_longlong(q.tagbits); }

__device__ inline float rcp_f(float x) { return __builtin_amdgcn_rcpf(x); }

__device__ inline int lane() { return (int)(threadIdx.x & 63); }

// Number of set bits of a wave mask below this lane.
__device__ inline int lanes_below(uint64_t m) {
  return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// ---------------------------------------------------------------------------------
// Cross-lane exchanges that need no lane-address register.  A shuffle through
// ds_bpermute takes a per-lane byte address; the compiler computes those once and
// keeps them live for the whole kernel (one register per distinct pattern), which in
// the tile kernel pushed values out to scratch.  These use gfx950's 32- and 16-lane
// row swaps and DPP moves within 16-lane rows, so only the data travels.
//
// Swaps: after v_permlane32_swap(a, b) lanes 32-63 of a hold lanes 0-31 of b and lanes
// 0-31 of b hold lanes 32-63 of a; v_permlane16_swap does the same between the odd
// 16-lane rows of a and the even rows of b.  DPP: row_ror:8 reads lane l ^ 8 (rotation
// by half of a 16-lane row), row_half_mirror lane l ^ 7, quad_perm [2,3,0,1] lane l ^ 2
// and [1,0,3,2] lane l ^ 1.

enum class Xl { Swap32, Swap16, Ror8, Mirror8, Quad2, Quad1 };

// (every source lane is valid; with bound_ctrl set the move folds into the instruction that uses it)
__device__ __forceinline__ uint32_t dpp32(uint32_t x, Xl p) {
  switch (p) {
    case Xl::Ror8: return (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, 0x128, 0xf, 0xf, true);
    case Xl::Mirror8: return (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, 0x141, 0xf, 0xf, true);
    case Xl::Quad2: return (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, 0x4e, 0xf, 0xf, true);
    default: return (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, 0xb1, 0xf, 0xf, true);
  }
}

// Lanes below the split (l & 32, or l & 16, clear) get a[l] and a[partner]; lanes above
// get b[partner] and b[l].  Returned as {first, second}: first + second is the pair sum
// each side keeps.
__device__ __forceinline__ void swap32(uint32_t a, uint32_t b, Xl p, uint32_t& first, uint32_t& second) {
  if (p == Xl::Swap32) {
    const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
    first = r[0];
    second = r[1];
  } else {
    const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
    first = r[0];
    second = r[1];
  }
}

template <typename T>
struct XlBits;
template <>
struct XlBits<float> {
  static constexpr int n = 1;
  __device__ static void split(float x, uint32_t* w) { w[0] = __float_as_uint(x); }
  __device__ static float join(const uint32_t* w) { return __uint_as_float(w[0]); }
};
template <>
struct XlBits<double> {
  static constexpr int n = 2;
  __device__ static void split(double x, uint32_t* w) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(x);
    w[0] = (uint32_t)b;
    w[1] = (uint32_t)(b >> 32);
  }
  __device__ static double join(const uint32_t* w) {
    return __longlong_as_double((long long)(((unsigned long long)w[1] << 32) | w[0]));
  }
};
template <>
struct XlBits<int> {
  static constexpr int n = 1;
  __device__ static void split(int x, uint32_t* w) { w[0] = (uint32_t)x; }
  __device__ static int join(const uint32_t* w) { return (int)w[0]; }
};

// Sum kept by each side of a swap exchange: lanes below the split get a[l] + a[partner],
// lanes above b[partner] + b[l] (the halving step of a reduction of two value sets).
template <typename T>
__device__ __forceinline__ T swap_sum(T a, T b, Xl p) {
  uint32_t wa[XlBits<T>::n], wb[XlBits<T>::n], f[XlBits<T>::n], s[XlBits<T>::n];
  XlBits<T>::split(a, wa);
  XlBits<T>::split(b, wb);
#pragma unroll
  for (int i = 0; i < XlBits<T>::n; ++i) swap32(wa[i], wb[i], p, f[i], s[i]);
  return XlBits<T>::join(f) + XlBits<T>::join(s);
}

// The value of x on the partner lane (l ^ 32, l ^ 16, l ^ 8, l ^ 7, l ^ 2 or l ^ 1).
template <typename T>
__device__ __forceinline__ T partner(T x, Xl p) {
  uint32_t w[XlBits<T>::n], o[XlBits<T>::n];
  XlBits<T>::split(x, w);
  if (p == Xl::Swap32 || p == Xl::Swap16) {
    const bool above = (lane() & (p == Xl::Swap32 ? 32 : 16)) != 0;
#pragma unroll
    for (int i = 0; i < XlBits<T>::n; ++i) {
      uint32_t f, s;
      swap32(w[i], w[i], p, f, s);
      o[i] = above ? f : s;
    }
  } else {
#pragma unroll
    for (int i = 0; i < XlBits<T>::n; ++i) o[i] = dpp32(w[i], p);
  }
  return XlBits<T>::join(o);
}

// x + x[l ^ mask]; both lanes of a pair add the same two values, so they agree bitwise.
template <typename T>
__device__ __forceinline__ T pair_add(T x, Xl p) {
  if (p == Xl::Swap32 || p == Xl::Swap16) return swap_sum(x, x, p);
  return x + partner(x, p);
}

// The butterfly patterns from the widest down; masks 32, 16, 8, 7, 2, 1 span all six
// lane bits, so after levels [from, 6) every lane of a 2^(6 - from)-lane group holds the
// group's sum (the same value on each).
constexpr Xl kLevel[6] = {Xl::Swap32, Xl::Swap16, Xl::Ror8, Xl::Mirror8, Xl::Quad2, Xl::Quad1};

template <typename T>
__device__ __forceinline__ T group_sum(T x, int from) {
#pragma unroll
  for (int lv = from; lv < 6; ++lv) x = pair_add(x, kLevel[lv]);
  return x;
}

// Relative half-width of the band around rc^2 decided in FP64 (well above the FP32 error
// of r^2 from exact fixed-point differences, ~3e-7, plus the 2^-26 A position rounding).
constexpr double kBand = 1e-6;
// Close contacts (r < kCloseSigma sigma, where the pair force exceeds ~50 kcal/mol/A for the
// polyethylene parameters) are evaluated in FP64 (see Band).
constexpr double kCloseSigma = 0.75;
constexpr int kBandQueue = 64;   // band pairs a tile wave queues per home group
constexpr int kBandSteps = 8;    // candidate steps with band pairs a tile wave records per group

// Values that are the same on every lane, moved to scalar registers.
__device__ inline int uni(int x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ inline double uni(double x) {
  const long long b = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_readfirstlane((int)(b & 0xffffffffLL));
  const int hi = __builtin_amdgcn_readfirstlane((int)(b >> 32));
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// The value of x on lane k (k wave-uniform), in scalar registers.
__device__ inline int lane_value(int x, int k) { return __builtin_amdgcn_readlane(x, k); }
__device__ inline float lane_value(float x, int k) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), k));
}
__device__ inline double lane_value(double x, int k) {
  const long long b = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffLL), k);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), k);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Minimum and maximum over lanes [0, K) (K = 1, 2, 4, 8 or 16), as a vector-register value on every
// lane: a butterfly over the log2(K) lowest lane bits (xor 1, xor 2, the half-row mirror, xor 8),
// then lane 0's result moved to every lane.
template <typename T>
__device__ __forceinline__ T in_vgpr(T x) {
  if constexpr (sizeof(T) == 4) asm volatile("" : "+v"(x));
  return x;
}

template <int K, bool MAX, typename T>
__device__ __forceinline__ T first_lanes_ext(T x) {
  constexpr Xl lv[4] = {Xl::Quad1, Xl::Quad2, Xl::Mirror8, Xl::Ror8};
#pragma unroll
  for (int l = 0; (1 << l) < K; ++l) {
    const T y = partner(x, lv[l]);
    x = MAX ? max(x, y) : min(x, y);
  }
  return in_vgpr(lane_value(x, 0));
}
template <int K, typename T>
__device__ __forceinline__ T first_lanes_min(T x) { return first_lanes_ext<K, false>(x); }
template <int K, typename T>
__device__ __forceinline__ T first_lanes_max(T x) { return first_lanes_ext<K, true>(x); }

// LDS is written and read by one wavefront, which executes its LDS accesses in order: only the
// compiler has to keep them so.
__device__ __forceinline__ void lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

constexpr float kFix2F = 1.125899906842624e15f;   // 2^50

template <typename P>
struct LjPair {
  P f12[4], f6[4], e12[4], e6[4], ecut[4];
  P f12_fold;               // f12[0] / f6[0] (one type pair: the force factor's inline constant)
  float band_lo, band_hi;   // the cutoff band (see Band), computed once on the host
  float close;              // close-contact bound (see Band), computed once on the host
};

template <typename P>
__device__ inline P pick(const P* a, int t) {
  return t == 0 ? a[0] : (t == 1 ? a[1] : (t == 2 ? a[2] : a[3]));
}

// The two ends of the FP32 pair range, in the fixed-point units of r2s (2^-50 A^2).
// Cutoff band: the FP32 path counts a pair as inside when r2s < hi.  Pairs with
// lo <= r2s < hi are in the band: there the FP32 r^2 cannot tell the side of the cutoff, so
// each is re-decided in FP64 and, if the FP64 test puts it outside, its force is taken back
// out (remove_band_pair).
// Close contacts: pairs with r2s < close (r below kCloseSigma times the smallest LJ sigma)
// never enter the FP32 sums.  Their force grows as r^-13 and FP32's few-ulp relative error
// on it would exceed 1e-5 of the RMS force (a contact at 2.0 A in a grown melt carries
// ~80 times the RMS force); each is evaluated in FP64 from the FP64 positions instead and
// added to its home's force (add_close_pair).  They are rare in a melt.
struct Band {
  float lo, hi, close;
};
template <typename P>
__device__ inline Band band_of(const LjPair<P>& c) {
  return Band{c.band_lo, c.band_hi, c.close};
}
__device__ __forceinline__ bool in_band(float r2s, bool keep, const Band& b) {
  return keep && r2s >= b.lo && r2s < b.hi;
}
__device__ __forceinline__ bool is_close(float r2s, bool keep, const Band& b) { return keep && r2s < b.close; }

// Exact cutoff test for a band pair (about one candidate in 10^6): r^2 < rc^2 decided from
// the FP64 positions with the operation order of a plain FP64 evaluation (no fused
// multiply-add), so the pair set is the FP64 one.  The image shift uses t * (1/L); it can
// differ from rint(t / L) only for |t| ~ L/2, i.e. |d| ~ L/2 >= 1.5 rc, never for a pair
// near the cutoff.  Returns the minimum-image difference and r^2.
__device__ __forceinline__ bool inside_cutoff_f64(const double* __restrict__ pos, int64_t n, const BoxDev& B,
                                                  int32_t i, int32_t j, double rc2, double (&d)[3], double& r2) {
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    const double t = __dadd_rn(pos[q * n + i], -pos[q * n + j]);
    d[q] = __dadd_rn(t, -__dmul_rn(B.L[q], rint(__dmul_rn(t, B.invL[q]))));
    r2 = q == 0 ? __dmul_rn(d[q], d[q]) : __dadd_rn(r2, __dmul_rn(d[q], d[q]));
  }
  return r2 < rc2;
}

// Takes a band pair that the FP64 test puts outside back out of accumulators in units of
// 2^25.  The pair sits at r ~ rc, where the force is ~|F(rc)|; evaluating it from the
// FP64 difference instead of the fixed-point one leaves a residue ~1e-7 of that.
template <bool ENERGY>
__device__ __forceinline__ void remove_band_pair(const double (&d)[3], double r2, float f12, float f6, float e12,
                                                 float e6, float ecut, float& ax, float& ay, float& az, double& e,
                                                 double& es, double& w) {
  const float r2i = 1.0f / (float)r2;
  const float r6 = r2i * r2i * r2i;
  const float g = r6 * (f12 * r6 - f6);
  const float ffs = g * r2i * (float)kFix;
  ax -= ffs * (float)d[0];
  ay -= ffs * (float)d[1];
  az -= ffs * (float)d[2];
  if (ENERGY) {
    const float en = r6 * (e12 * r6 - e6);
    e -= (double)en;
    es -= (double)en - (double)ecut;
    w -= (double)g;
  }
}

// Adds a close contact to FP64 accumulators (kcal/mol/A): the force from the FP64
// minimum-image difference d = x_i - x_j, in a plain FP64 operation order.
template <bool ENERGY>
__device__ __forceinline__ void add_close_pair(const double (&d)[3], double r2, double f12, double f6, double e12,
                                               double e6, double ecut, double& cx, double& cy, double& cz,
                                               double& e, double& es, double& w) {
  const double r2i = 1.0 / r2;
  const double r6 = r2i * r2i * r2i;
  const double g = r6 * (f12 * r6 - f6);
  const double ffs = g * r2i;
  cx += ffs * d[0];
  cy += ffs * d[1];
  cz += ffs * d[2];
  if (ENERGY) {
    const double en = r6 * (e12 * r6 - e6);
    e += en;
    es += en - ecut;
    w += g;
  }
}

// FP32 r^2 of an exact fixed-point difference (units of 2^-50 A^2).  Written with explicit
// fused multiply-adds so that every call site rounds identically.
__device__ __forceinline__ float r2_fix(float dx, float dy, float dz) {
  return __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, dx * dx));
}

// One pair, mixed precision.  d* are exact fixed-point differences x_i - x_j; the force
// accumulated in a* is in units of 2^25 (the caller scales the final sum by 2^-25).
// Pairs in the cutoff band are counted; bmax keeps the bits of the largest r2s counted
// (r2s >= 0, so integer order is float order), so that the caller sees a band pair
// (bmax >= lo) at one integer max per pair and settles it.  A close contact (r2s < close)
// is not counted: near is set, and the caller evaluates it in FP64.
// Returns r2s.
// FOLD: f12 holds f12 / f6 and the caller multiplies the summed force by f6 (one type
// pair: the force factor is then one FMA with an inline constant and no register copy).
template <bool ENERGY, bool FOLD = false>
__device__ __forceinline__ float pair_fix(int dqx, int dqy, int dqz, bool keep, const Band& bd, float f12,
                                          float f6, float e12, float e6, float ecut, float& ax, float& ay,
                                          float& az, double& e, double& es, double& w, int32_t& bmax,
                                          bool& near) {
  const float dx = (float)dqx, dy = (float)dqy, dz = (float)dqz;
  const float r2s = r2_fix(dx, dy, dz);
  const bool lt_close = r2s < bd.close;   // one compare serves both masks
  const bool kh = keep && r2s < bd.hi;
  near = near || (kh && lt_close);
  const bool hit = kh && !lt_close;
  if (hit) {
    const float r2 = r2s * kInvFix2F;
    const float r2i = rcp_f(r2);
    const float r6 = r2i * r2i * r2i;
    const float g = FOLD ? r6 * __builtin_fmaf(f12, r6, -1.0f) : r6 * (f12 * r6 - f6);   // F . r (/ f6)
    float ffs = g * r2i;
    ax += ffs * dx;
    ay += ffs * dy;
    az += ffs * dz;
    bmax = max(bmax, __float_as_int(r2s));
    if (ENERGY) {
      const float en = r6 * (e12 * r6 - e6);
      e += (double)en;
      es += (double)en - (double)ecut;
      w += (double)(FOLD ? g * f6 : g);
    }
  }
  return r2s;
}

// One pair, FP64.
template <bool ENERGY>
__device__ __forceinline__ void pair_f64(double dx, double dy, double dz, bool keep, double rc2, double f12,
                                         double f6, double e12, double e6, double ecut, double& ax, double& ay,
                                         double& az, double& e, double& es, double& w) {
  const double r2 = dx * dx + dy * dy + dz * dz;
  if (keep && r2 < rc2) {
    const double r2i = 1.0 / r2;
    const double r6 = r2i * r2i * r2i;
    const double g = r6 * (f12 * r6 - f6);
    const double ffs = g * r2i;
    ax += ffs * dx;
    ay += ffs * dy;
    az += ffs * dz;
    if (ENERGY) {
      const double en = r6 * (e12 * r6 - e6);
      e += en;
      es += en - ecut;
      w += g;
    }
  }
}

template <int NW>
__device__ void block_energy(double e, double es, double w, dd (*red)[3], dd* out) {
  dd q[3] = {dd_from(0.5 * e), dd_from(0.5 * es), dd_from(0.5 * w)};
  for (int k = 0; k < 3; ++k)
#pragma unroll
    for (int lv = 0; lv < 6; ++lv) q[k] = dd_add(q[k], dd{partner(q[k].hi, kLevel[lv]), partner(q[k].lo, kLevel[lv])});
  if (lane() == 0)
    for (int k = 0; k < 3; ++k) red[threadIdx.x >> 6][k] = q[k];
  __syncthreads();
  if (threadIdx.x == 0)
    for (int k = 0; k < 3; ++k) {
      dd s = red[0][k];
      for (int wv = 1; wv < NW; ++wv) s = dd_add(s, red[wv][k]);
      out[k] = s;
    }
}

// Exclusive prefix sum of x >= 0 over the wave, bit plane by bit plane: the lanes below
// this one whose bit b is set add 2^b each (a ballot and a masked popcount per plane).
__device__ __forceinline__ int wave_exclusive_scan(int x, int& total) {
  int below = 0, tot = 0;
  for (int b = 0; b < 31; ++b) {
    if (__builtin_amdgcn_ballot_w64((x >> b) != 0) == 0) break;
    const uint64_t m = __builtin_amdgcn_ballot_w64(((x >> b) & 1) != 0);
    below += lanes_below(m) << b;
    tot += __popcll(m) << b;
  }
  total = tot;
  return below;
}

template <typename P>
LjPair<P> make_pair(const FFDev& ff) {
  LjPair<P> c;
  for (int t = 0; t < 4; ++t) {
    c.f12[t] = (P)ff.f12[t];
    c.f6[t] = (P)ff.f6[t];
    c.e12[t] = (P)ff.e12[t];
    c.e6[t] = (P)ff.e6[t];
    c.ecut[t] = (P)ff.ecut[t];
  }
  c.f12_fold = c.f12[0] / c.f6[0];
  c.band_lo = (float)(ff.rc2 * kFix * kFix * (1.0 - kBand));
  c.band_hi = (float)(ff.rc2 * kFix * kFix * (1.0 + kBand));
  // close contacts: r below kCloseSigma times the smallest sigma of a type pair that interacts
  // (sigma^6 = e12 / e6)
  double s6 = 0.0;
  for (int t = 0; t < 4; ++t)
    if (ff.e6[t] > 0.0) s6 = s6 > 0.0 ? std::min(s6, ff.e12[t] / ff.e6[t]) : ff.e12[t] / ff.e6[t];
  // (at most the band: with a cutoff below the bound every pair inside it is a close contact or in the
  // band, and [close, band_lo) is empty, as the kernels' range test on it needs)
  c.close = std::min((float)(kCloseSigma * kCloseSigma * std::cbrt(s6) * kFix * kFix), c.band_lo);
  return c;
}

}  // namespace
}  // namespace mdk
