// Truncated Lennard-Jones forces over the cell grid for gfx950: one wavefront per group of home
// atoms that follow one another along x (Section 3.2, Eq. 2).
//
// The payload is sorted by cell (x index fastest) and inside a cell by x, so the atoms of one row
// of cells (one ky, kz) lie in x order and any 8 consecutive ones of them are a compact group,
// whatever the cells hold.  The cells that can hold partners are, in each of the (2R + 1)^2 rows
// around the group's row, one contiguous run of the sorted order: the row's distance from the box
// bounding the group leaves a reach along x.  A wave
//   1. finds the runs, one row per lane (periodic images along x in up to three passes);
//   2. streams them 64 candidates at a time, the lane's run looked up from a bit mask of run
//      starts; a candidate nearer than rc to the group's bounding box goes to a list in LDS, in
//      the group's frame (416 of 776 in a melt of 0.80 g/cm^3 at R = 2);
//   3. takes 16 candidates at a time from the list against 4 homes at a time: lane 4 c + i holds
//      the pair of candidate c and home i, so nothing is broadcast, few registers are live and the
//      last block wastes at most 15 candidates.
// Each lane's sums are added over the 16 lanes of a home in a fixed order at the end: no atomics,
// every pair from both sides, the same result every run.  FP64 force error against 80-bit arithmetic, 12
// relaxed melts of 3,000 and 15,000 atoms: rms 7.8e-16 of the RMS force, largest 1.4e-14 (the same with
// a division for rcp_d; the kernels before 1.1e-15 to 1.4e-15 and 2.1e-14).
//
// Bound: VALU instructions (at 300,000 atoms ~2,400 per group and wave, half of them in the pair
// blocks), in small boxes the latency of one wave's chain of dependent loads and sums, which is why
// up to kSplitItems groups are shared by kSplit waves each (FP64, R = 2: 31 against 36 us at 12,000
// atoms, 48 against 43 us at 24,000; the groups of all such boxes together count: 24 boxes of 12,000 atoms
// 347 against 195 us, 100 of 3,000 375 against 203).  Measured against the kernels it replaces (LJ pass, event
// timing): one lane per atom, 3,000 atoms, FP64, R = 1: 388 -> 19 us; 36,720 atoms, mixed, R = 1:
// 517 -> 45 us; the FP64 cell tile, 300,000 atoms, R = 2: 246 -> 199 us.
#include "md_lj_common.h"

namespace mdk {
namespace {

constexpr int kBatch = 2;            // 64-candidate windows loaded together (1: 5-10% slower; 3: no faster)
constexpr int kCap = 160;            // filtered candidates a wave holds in LDS (16 B each mixed, 32 B FP64)
// Waves per SIMD the registers are held to.  FP64 spills 4 to 19 of them at 5; against 4 without, an
// evaluation of 300,000 atoms: with energies 285 against 287 us, two types 270 and 270, both 396 against 394.
template <bool FP64>
constexpr int kGroupEu = FP64 ? 5 : 4;
constexpr int kChunkWindows = 64;    // 64-candidate windows whose run starts are marked at a time

struct Cand32 {      // mixed: offsets from the group's first atom in 2^-25 A, biased by 2^31
  uint32_t x, y, z;
  int32_t tag;
};

template <bool FP64>
struct Geo;
template <>
struct Geo<false> {
  using Pay = int4;
  using Cand = Cand32;
  using Off = int32_t;    // offset added to a payload coordinate
  static constexpr float kUnit = 1.0f / kInvFixF;      // filter units per A
  static constexpr float kZero = 2147483648.0f;         // the group's first atom in filter units
  __device__ static Off origin(Off ref, double) { return (Off)(0x80000000u - (uint32_t)ref); }
  __device__ static uint32_t rel(int x, Off o) { return (uint32_t)x + (uint32_t)o; }
  __device__ static float filt(uint32_t u) { return (float)u; }
  __device__ static uint32_t far() { return 0u; }        // 64 A from the group's first atom
  __device__ static Cand cand(uint32_t x, uint32_t y, uint32_t z, int32_t tag) { return Cand{x, y, z, tag}; }
};
template <>
struct Geo<true> {
  using Pay = Pay64;
  using Cand = Pay64;
  using Off = double;
  static constexpr float kUnit = 1.0f;
  static constexpr float kZero = 0.0f;
  // The group's first coordinate rounded to a multiple of the box edge's last place, so that the origin of
  // a periodic image, one edge further, is exact: pairs across an edge lose nothing to the box's length.
  __device__ static Off origin(Off ref, double L) { return uni(L - (ref + L)); }
  __device__ static double rel(double x, Off o) { return x + o; }
  __device__ static float filt(double u) { return (float)u; }
  __device__ static double far() { return 1.0e150; }     // (its square is finite)
  __device__ static Cand cand(double x, double y, double z, int32_t tag) {
    return Cand{x, y, z, __longlong_as_double((long long)tag)};
  }
};
__device__ inline int32_t pay_tag(const Cand32& q) { return q.tag; }

// One run of the sorted order (a row's cells within reach): payload index of flat position t is
// t + src; the offsets put its atoms in the group's frame.
template <typename Off>
struct alignas(16) Run {
  Off oy, oz;
  int32_t src;
};

// r^-2 from v_rcp_f64 and two Newton steps (within an ulp of 1 / r2).
__device__ __forceinline__ double rcp_d(double x) {
  double y = __builtin_amdgcn_rcp(x);
  y = __builtin_fma(__builtin_fma(-x, y, 1.0), y, y);
  return __builtin_fma(__builtin_fma(-x, y, 1.0), y, y);
}

// Minimum / maximum over the first K lanes (K = 4, 8, 16), the same value on every lane.
template <int K, bool MAX>
__device__ __forceinline__ float ext(float x) {
  constexpr Xl lv[4] = {Xl::Quad1, Xl::Quad2, Xl::Mirror8, Xl::Ror8};
#pragma unroll
  for (int l = 0; (1 << l) < K; ++l) {
    const float y = partner(x, lv[l]);
    x = MAX ? fmaxf(x, y) : fminf(x, y);
  }
  return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(x)));
}

// x + x rotated by 4 within 16-lane rows
__device__ __forceinline__ float add_ror4(float x) {
  return x + __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x124, 0xf, 0xf, true));
}
__device__ __forceinline__ double add_ror4(double x) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(x);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)b, 0x124, 0xf, 0xf, true);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(b >> 32), 0x124, 0xf, 0xf, true);
  return x + __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
// Sum over the 16 lanes that share lane & 3.
__device__ __forceinline__ double home_sum(double x) {
  return add_ror4(pair_add(pair_add(pair_add(x, Xl::Swap32), Xl::Swap16), Xl::Ror8));
}

__device__ inline float lane_value_f(float x, int k) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), k));
}

// gap, rc: what is added to every reach (launch_e), the cutoff plus it.
// NW wavefronts work on one group, each on every NW-th batch of its candidates (NW > 1: boxes with
// too few groups to fill the chip); their sums are added in wave order.
template <bool FP64, bool ENERGY, bool UNI, int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(kGroupEu<FP64>)))
void k_lj_group(Views v, FFDev ff, LjPair<float> cf, LjPair<double> cd, float gap, float rc) {
  using G = Geo<FP64>;
  using PayT = typename G::Pay;
  using Cand = typename G::Cand;
  using Off = typename G::Off;
  using P = std::conditional_t<FP64, double, float>;
  constexpr int K = kGroupHomes, NH = K / 4;   // homes per group, quads of homes
  constexpr int CAP = kCap;
  __shared__ Cand lists[NW][CAP];
  __shared__ Run<Off> runs_[NW][64];
  __shared__ unsigned long long marks_[NW][kChunkWindows];
  __shared__ Cand homes_[NW][K];
  __shared__ int2 window_[NW][K];
  __shared__ double exact_[FP64 ? 1 : NW][FP64 ? 1 : K][3];   // mixed: forces of the pairs evaluated in FP64
  __shared__ double part[NW > 1 ? NW : 1][NW > 1 ? K : 1][3];  // each wave's sums
  __shared__ dd red[NW][3];

  const int ln = lane(), wave = NW > 1 ? uni((int)threadIdx.x >> 6) : 0;
  Cand* const list = lists[wave];
  Run<Off>* const runs = runs_[wave];
  unsigned long long* const marks = marks_[wave];
  Cand* const homes = homes_[wave];
  int2* const window = window_[wave];
  double (*const exact)[3] = exact_[FP64 ? 0 : wave];
  // Workgroups are dealt to the 8 XCDs round-robin; each XCD gets a contiguous run of groups (a
  // slab of the box), so its L2 holds one neighbourhood of the payload.
  const int per_xcd = (int)gridDim.x / kXcds;
  const int blk = ((int)blockIdx.x % kXcds) * per_xcd + (int)blockIdx.x / kXcds;
  if (blk >= v.n_lj_blocks) return;
  const int box = v.lj_blk_box[blk / kGroupPad];
  const BoxDev& B = v.boxes[box];
  const GroupDev& Q = v.groups[box];
  if (Q.waves() != NW) return;   // a box of the other launch
  const PayT* __restrict__ pay = static_cast<const PayT*>(v.payload);
  const int32_t* __restrict__ cs = v.cell_start;
  const int R = v.R, W = 2 * R + 1;
  const int M0 = B.M[0], M1 = B.M[1], M2 = B.M[2];
  // this lane's row of the stencil (W <= 7; the quotient lies 1/14 from an integer)
  const int oz = (int)(((float)ln + 0.5f) * rcp_f((float)W)) - R, oy = ln - (oz + R) * W - R;
  double e = 0.0, es = 0.0, w = 0.0;

  const int S = Q.slots, items = Q.items, stride = Q.blocks, KH = Q.homes();
  const int passes = Q.passes(), shift = Q.shift;
  for (int item = blk - B.lj_blk_off, pass = 0; item < items;) {   // (each item's passes, then the next)
    const int row_of = uni((int)(((double)item + 0.5) * Q.inv_slots));          // item / S
    int row = row_of + pass * shift;
    row -= row >= M1 * M2 ? M1 * M2 : 0;
    const int kz = uni((int)(((double)row + 0.5) * Q.inv_m1)), ky = row - kz * M1;
    const int row0 = B.cell_off + row * M0;
    const int rs = uni(cs[row0]), re = uni(cs[row0 + M0]);
    const int at = pass * S + item - row_of * S;
    if (++pass >= passes) { pass = 0; item += stride; }
    for (int p0 = rs + at * KH; p0 < re; p0 += passes * S * KH) {
      const int kc = min(KH, re - p0);
      // Homes further than Q.cap along x from the group's first one start a group of their own
      // (sparse rows): the frame stays within the fixed-point range and the runs stay short.
      for (int h0 = 0, h1 = 0; h0 < kc; h0 = h1) {
        P ax[NH], ay[NH], az[NH];
#pragma unroll
        for (int h = 0; h < NH; ++h) ax[h] = ay[h] = az[h] = (P)0;
        float xhi, ylo, yhi, zlo, zhi;        // the box bounding the group (filter units)
        float xr, yr, zr, xe;                 // the first atom, A from the low corner of its cell; x extent
        Off ox0, oy0, oz0;
        int kx;
        {
          const int hl = min(ln, kc - 1);
          const PayT hq = pay[p0 + hl];
          const int hcell = v.scell[p0 + hl] - row0;
          const int32_t i = tag_index(pay_tag(hq));
          const Off x0 = lane_value(hq.x, h0), y0 = lane_value(hq.y, h0), z0 = lane_value(hq.z, h0);
          ox0 = G::origin(x0, B.L[0]);
          oy0 = G::origin(y0, B.L[1]);
          oz0 = G::origin(z0, B.L[2]);
          const auto ux = G::rel(hq.x, ox0), uy = G::rel(hq.y, oy0), uz = G::rel(hq.z, oz0);
          const float fx = G::filt(ux), fy = G::filt(uy), fz = G::filt(uz);
          // (the cell distance tells apart what the offset modulo 128 A cannot)
          kx = lane_value(hcell, h0);
          const float dx0 = (fx - G::kZero) * (1.0f / G::kUnit), e0 = (float)B.edge[0], cap = (float)Q.cap;
          const bool apart = (float)(hcell - kx) * e0 > cap + e0 || dx0 > cap || dx0 < -1.0f;
          const uint64_t past = __builtin_amdgcn_ballot_w64(ln > h0 && ln < kc && apart);
          h1 = past ? __ffsll((unsigned long long)past) - 1 : kc;
          const bool mine = ln >= h0 && ln < h1;
          if (ln < K) {
            const int32_t c0 = chain_first(i, ff);
            const int32_t lo = max(i - ff.excl, c0);
            const uint32_t span = (uint32_t)(min(i + ff.excl, c0 + ff.chain_len - 1) - lo);
            homes[ln] = G::cand(ux, uy, uz, pay_tag(hq));
            if constexpr (!FP64) exact[ln][0] = exact[ln][1] = exact[ln][2] = 0.0;
            // in tag units; a slot without a home excludes every candidate
            window[ln] = mine ? make_int2(lo << 4, (int)((span << 4) | 15u)) : make_int2(0, -1);
          }
          // x order inside the group (up to the key's 1e-6 of a cell: the gap covers it)
          xhi = lane_value_f(fx, h1 - 1);
          xe = lane_value_f(dx0, h1 - 1);
          ylo = ext<K, false>(mine ? fy : G::kZero);
          yhi = ext<K, true>(mine ? fy : G::kZero);
          zlo = ext<K, false>(mine ? fz : G::kZero);
          zhi = ext<K, true>(mine ? fz : G::kZero);
          if constexpr (FP64) {
            xr = (float)(x0 - kx * B.edge[0]);
            yr = (float)(y0 - ky * B.edge[1]);
            zr = (float)(z0 - kz * B.edge[2]);
          } else {
            xr = (float)(int)((uint32_t)x0 - (uint32_t)fix_coord(kx * B.edge[0])) * kInvFixF;
            yr = (float)(int)((uint32_t)y0 - (uint32_t)fix_coord(ky * B.edge[1])) * kInvFixF;
            zr = (float)(int)((uint32_t)z0 - (uint32_t)fix_coord(kz * B.edge[2])) * kInvFixF;
          }
        }
        lds_order();
        int m = 0;   // candidates in list[]
        // The first nb blocks of 16 candidates of list[] against the group: lane 4 c + i holds the
        // pair of candidate c and home i of each quad.
        auto pairs = [&](int nb) {
          Cand hq[NH];
          int2 win[NH];
#pragma unroll
          for (int h = 0; h < NH; ++h) {
            hq[h] = homes[4 * h + (ln & 3)];
            win[h] = window[4 * h + (ln & 3)];
          }
#pragma unroll 1
          for (int c0 = 0; c0 < nb; ++c0) {
            const Cand q = list[16 * c0 + (ln >> 2)];
            const int32_t jt = pay_tag(q);
            if constexpr (FP64) {
#pragma unroll
              for (int h = 0; h < NH; ++h) {
                const bool keep = (uint32_t)(jt - win[h].x) > (uint32_t)win[h].y;
                const int tt = UNI ? 0 : tag_type(pay_tag(hq[h])) * 2 + tag_type(jt);
                const double dx = hq[h].x - q.x, dy = hq[h].y - q.y, dz = hq[h].z - q.z;
                const double r2 = dx * dx + dy * dy + dz * dz;
                const bool hit = keep && r2 < ff.rc2;
                const double r2i = rcp_d(r2);
                const double r6 = r2i * r2i * r2i;
                const double g = r6 * (pick(cd.f12, tt) * r6 - pick(cd.f6, tt));
                const double s = hit ? g * r2i : 0.0;
                ax[h] += s * dx;
                ay[h] += s * dy;
                az[h] += s * dz;
                if (ENERGY && hit) {
                  const double en = r6 * (pick(cd.e12, tt) * r6 - pick(cd.e6, tt));
                  e += en;
                  es += en - pick(cd.ecut, tt);
                  w += g;
                }
              }
            } else {
              uint64_t rare[NH];   // (lane masks: combined by the scalar unit)
              uint64_t any = 0;
#pragma unroll
              for (int h = 0; h < NH; ++h) {
                const uint64_t keep = __builtin_amdgcn_ballot_w64((uint32_t)(jt - win[h].x) > (uint32_t)win[h].y);
                const int tt = UNI ? 0 : tag_type(pay_tag(hq[h])) * 2 + tag_type(jt);
                const float dx = (float)(int)(hq[h].x - q.x), dy = (float)(int)(hq[h].y - q.y),
                            dz = (float)(int)(hq[h].z - q.z);
                const float r2s = r2_fix(dx, dy, dz);
                const uint64_t in = keep & __builtin_amdgcn_ballot_w64(r2s < cf.band_hi);
                // neither a close contact nor a pair whose side of the cutoff FP32 cannot tell
                const uint64_t plain =
                    __builtin_amdgcn_ballot_w64((uint32_t)(__float_as_int(r2s) - __float_as_int(cf.close)) <
                                                (uint32_t)(__float_as_int(cf.band_lo) - __float_as_int(cf.close)));
                rare[h] = in & ~plain;
                any |= rare[h];
                const bool hit = __builtin_amdgcn_inverse_ballot_w64(in & plain);
                const float r2i = rcp_f(r2s) * kFix2F;
                const float r4 = r2i * r2i, r6 = r4 * r2i;
                const float t = UNI ? __builtin_fmaf(cf.f12_fold, r6, -1.0f)
                                    : __builtin_fmaf(pick(cf.f12, tt), r6, -pick(cf.f6, tt));
                const float s = hit ? (r4 * r4) * t : 0.0f;
                ax[h] = __builtin_fmaf(s, dx, ax[h]);
                ay[h] = __builtin_fmaf(s, dy, ay[h]);
                az[h] = __builtin_fmaf(s, dz, az[h]);
                if (ENERGY && hit) {
                  const float en = r6 * (pick(cf.e12, tt) * r6 - pick(cf.e6, tt));
                  e += (double)en;
                  es += (double)en - (double)pick(cf.ecut, tt);
                  w += (double)(UNI ? r6 * t * cf.f6[0] : r6 * t);
                }
              }
              if (any != 0) {
                // from the FP64 positions; summed over each home's lanes into its FP64 slot
#pragma unroll
                for (int h = 0; h < NH; ++h) {
                  const int32_t ht = pay_tag(hq[h]);
                  const int tt = UNI ? 0 : tag_type(ht) * 2 + tag_type(jt);
                  double fx = 0.0, fy = 0.0, fz = 0.0;
                  if (__builtin_amdgcn_inverse_ballot_w64(rare[h])) {
                    double d[3], q2;
                    if (inside_cutoff_f64(v.pos, v.N, B, tag_index(ht), tag_index(jt), ff.rc2, d, q2))
                      add_close_pair<ENERGY>(d, q2, pick(cd.f12, tt), pick(cd.f6, tt), pick(cd.e12, tt),
                                             pick(cd.e6, tt), pick(cd.ecut, tt), fx, fy, fz, e, es, w);
                  }
                  fx = home_sum(fx);
                  fy = home_sum(fy);
                  fz = home_sum(fz);
                  if (ln < 4) {
                    exact[4 * h + ln][0] += fx;
                    exact[4 * h + ln][1] += fy;
                    exact[4 * h + ln][2] += fz;
                  }
                }
                lds_order();
              }
            }
          }
        };
        // ---- the candidates: one pass per periodic image along x that the group reaches ----
        int im = 0, im_left = -1;   // this pass's image; bit 0 / 1: image -1 / +1 still to do
        const float rcf = rc * rc * (G::kUnit * G::kUnit);
        do {
          // the runs, one stencil row per lane
          const float e0 = (float)B.edge[0], e1 = (float)B.edge[1], e2 = (float)B.edge[2];
          constexpr float iu = 1.0f / G::kUnit;
          const float gy = oy > 0 ? (float)oy * e1 - (yr + (yhi - G::kZero) * iu)
                                  : (yr + (ylo - G::kZero) * iu) - (float)(oy + 1) * e1;
          const float gz = oz > 0 ? (float)oz * e2 - (zr + (zhi - G::kZero) * iu)
                                  : (zr + (zlo - G::kZero) * iu) - (float)(oz + 1) * e2;
          // (in the group's own row and layer both forms are negative)
          const float hy = fmaxf(gy - gap, 0.0f), hz = fmaxf(gz - gap, 0.0f);
          const float left = rc * rc - hy * hy - hz * hz;
          const bool inrow = ln < W * W && left > 0.0f;
          const float reach = __builtin_amdgcn_sqrtf(fmaxf(left, 0.0f)) + gap, ie0 = rcp_f(e0);
          const int low = kx + (int)floorf((xr - reach) * ie0);
          const int high = kx + (int)floorf((xr + xe + reach) * ie0);
          if (im_left < 0)
            im_left = (__builtin_amdgcn_ballot_w64(inrow && low < 0) != 0 ? 1 : 0) |
                      (__builtin_amdgcn_ballot_w64(inrow && high >= M0) != 0 ? 2 : 0);
          int ny = ky + oy, nz = kz + oz;
          const int wy = ny < 0 ? -1 : (ny >= M1 ? 1 : 0), wz = nz < 0 ? -1 : (nz >= M2 ? 1 : 0);
          ny -= wy * M1;
          nz -= wz * M2;
          const int nrow0 = B.cell_off + M0 * (ny + M1 * nz);
          const int a = max(low, im * M0) - im * M0, b = min(high, im * M0 + M0 - 1) - im * M0;
          int n = 0, start = 0;
          if (inrow && a <= b) {
            start = cs[nrow0 + a];
            n = cs[nrow0 + b + 1] - start;
          }
          int total;
          int f = wave_exclusive_scan(n, total);
          total = uni(total);
          const uint64_t some = __builtin_amdgcn_ballot_w64(n > 0);
          Off sx;
          if constexpr (FP64) sx = uni(ox0 + (double)im * B.L[0]);
          else sx = (Off)((uint32_t)ox0 + (uint32_t)im * (uint32_t)Q.L_q[0]);
          if (n > 0) {
            Run<Off> r;
            if constexpr (FP64) {
              r.oy = oy0 + (double)wy * B.L[1];
              r.oz = oz0 + (double)wz * B.L[2];
            } else {
              r.oy = (Off)((uint32_t)oy0 + (uint32_t)wy * (uint32_t)Q.L_q[1]);
              r.oz = (Off)((uint32_t)oz0 + (uint32_t)wz * (uint32_t)Q.L_q[2]);
            }
            r.src = start - f;
            runs[lanes_below(some)] = r;
          }
          const int mark = n > 0 ? f - 1 : -1;   // a run (but the first) marks the position before it
          for (int t0 = 0; t0 < total; t0 += 64 * kChunkWindows) {
            // the run of a candidate: the runs marked before it
            marks[ln] = 0ull;
            lds_order();
            const int at = mark - t0;
            if (mark >= 0 && at >= 0 && at < 64 * kChunkWindows) atomicOr(&marks[at >> 6], 1ull << (at & 63));
            lds_order();
            const unsigned long long mk = marks[ln];
            const int mlo = (int)(uint32_t)mk, mhi = (int)(uint32_t)(mk >> 32);
            const int end = min(total, t0 + 64 * kChunkWindows), nw = (end - t0 + 63) >> 6;
#pragma unroll 1
            for (int w0 = wave * kBatch; w0 < nw; w0 += NW * kBatch) {
              PayT q[kBatch];
              Run<Off> run[kBatch];
              bool in[kBatch];
#pragma unroll
              for (int u = 0; u < kBatch; ++u) {
                // lanes past the candidates re-read the group's first atom and are dropped below
                const int win = w0 + u, t = t0 + 64 * win + ln;
                const int before = __popcll(__builtin_amdgcn_ballot_w64(mark >= 0 && mark < t0 + 64 * win));
                const int wl = __builtin_amdgcn_readlane(mlo, win & 63), wh = __builtin_amdgcn_readlane(mhi, win & 63);
                const int r = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)wh,
                                                             __builtin_amdgcn_mbcnt_lo((uint32_t)wl, (uint32_t)before));
                in[u] = t < end;
                run[u] = runs[in[u] ? r : 0];
                const uint32_t at_pay = (uint32_t)(in[u] ? t + run[u].src : p0);
                q[u] = pay[at_pay];
              }
#pragma unroll
              for (int u = 0; u < kBatch; ++u) {
                const auto cx = G::rel(q[u].x, sx), cy = G::rel(q[u].y, run[u].oy), cz = G::rel(q[u].z, run[u].oz);
                const float gx = G::filt(cx), gyf = G::filt(cy), gzf = G::filt(cz);
                const float bx = gx - __builtin_amdgcn_fmed3f(gx, G::kZero, xhi);
                const float by = gyf - __builtin_amdgcn_fmed3f(gyf, ylo, yhi);
                const float bz = gzf - __builtin_amdgcn_fmed3f(gzf, zlo, zhi);
                const uint64_t pm = __builtin_amdgcn_ballot_w64(__builtin_fmaf(bz, bz, __builtin_fmaf(by, by, bx * bx)) < rcf) &
                                    __builtin_amdgcn_ballot_w64(in[u]);
                if (__builtin_amdgcn_inverse_ballot_w64(pm))
                  list[__builtin_amdgcn_mbcnt_hi((uint32_t)(pm >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)pm, (uint32_t)m))] =
                      G::cand(cx, cy, cz, pay_tag(q[u]));
                m += __popcll(pm);
              }
              lds_order();
              if (m > CAP - 64 * kBatch) {   // no room for another batch: the whole blocks' pairs now
                pairs(m >> 4);
                const int rest = m & 15;
                if (ln < rest) list[ln] = list[(m & ~15) + ln];
                m = rest;
                lds_order();
              }
            }
          }
          im = (im_left & 1) ? -1 : 1;
          const int more = im_left;
          im_left &= im_left - 1;
          if (more == 0) break;
        } while (true);
        if (m > 0) {   // the last block padded with candidates out of reach
          if (ln < ((m + 15) & ~15) - m) list[m + ln] = G::cand(G::far(), G::far(), G::far(), 0);
          lds_order();
          pairs((m + 15) >> 4);
        }
        // ---- sums over the 16 lanes of each home: lanes below 32 keep quad 0, the others quad 1 ----
        static_assert(NH == 2, "two quads");
        P sx1 = pair_add(swap_sum(ax[0], ax[1], Xl::Swap32), Xl::Swap16);
        P sy1 = pair_add(swap_sum(ay[0], ay[1], Xl::Swap32), Xl::Swap16);
        P sz1 = pair_add(swap_sum(az[0], az[1], Xl::Swap32), Xl::Swap16);
        sx1 = add_ror4(pair_add(sx1, Xl::Ror8));
        sy1 = add_ror4(pair_add(sy1, Xl::Ror8));
        sz1 = add_ror4(pair_add(sz1, Xl::Ror8));
        const int slot = 4 * (ln >> 5) + (ln & 3);
        const bool writer = (ln & 28) == 0;
        double fx = (double)sx1, fy = (double)sy1, fz = (double)sz1;
        if constexpr (!FP64) {
          // fixed-point units, divided by f6 with one type pair
          const double sc = (double)kInvFixF * (UNI ? cd.f6[0] : 1.0);
          fx = fx * sc + exact[slot][0];
          fy = fy * sc + exact[slot][1];
          fz = fz * sc + exact[slot][2];
        }
        if constexpr (NW > 1) {
          if (writer) {
            part[wave][slot][0] = fx;
            part[wave][slot][1] = fy;
            part[wave][slot][2] = fz;
          }
          __syncthreads();
          fx = part[0][slot][0];
          fy = part[0][slot][1];
          fz = part[0][slot][2];
#pragma unroll
          for (int u = 1; u < NW; ++u) {
            fx += part[u][slot][0];
            fy += part[u][slot][1];
            fz += part[u][slot][2];
          }
        }
        if (wave == 0 && writer && slot >= h0 && slot < h1) {
          const int32_t i = tag_index(pay_tag(homes[slot]));
          P* f_out = static_cast<P*>(v.f_lj);
          f_out[i] = (P)fx;
          f_out[v.N + i] = (P)fy;
          f_out[2 * v.N + i] = (P)fz;
        }
        if constexpr (NW > 1) __syncthreads();
        else lds_order();
      }
    }
  }
  if (ENERGY) block_energy<NW>(e, es, w, red, v.part_lj + (int64_t)blk * 3);
}

template <bool FP64, bool ENERGY>
void launch_e(const Views& v, const FFDev& ff, hipStream_t s) {
  const LjPair<float> cf = make_pair<float>(ff);
  const LjPair<double> cd = make_pair<double>(ff);
  // The gap is added to every reach and to the filter for their FP32 rounding (and what the order along x leaves
  // open, 1e-6 of a cell): in the mixed form, whose coordinates round to 2^-17 A at most, in A; in FP64, whose
  // lengths may have any scale, as a part of the cutoff.
  const double rc = std::sqrt(ff.rc2);
  const float gap = FP64 ? (float)(1e-4 * rc) : 1e-3f, reach = (float)rc + gap;
  const dim3 g((v.n_lj_blocks + kXcds - 1) / kXcds * kXcds);
#define MDK_GROUP(U, NW) \
  hipLaunchKernelGGL((k_lj_group<FP64, ENERGY, U, NW>), g, dim3(64 * NW), 0, s, v, ff, cf, cd, gap, reach)
  if (v.lj_wave_mask & 1) {
    if (ff.uniform_lj) MDK_GROUP(true, 1);
    else MDK_GROUP(false, 1);
  }
  if (v.lj_wave_mask & 2) {
    if (ff.uniform_lj) MDK_GROUP(true, kSplit);
    else MDK_GROUP(false, kSplit);
  }
#undef MDK_GROUP
}

}  // namespace

void launch_lj_group(const Views& v, const FFDev& ff, bool fp32, bool energy, hipStream_t s) {
  if (fp32) {
    if (energy) launch_e<false, true>(v, ff, s);
    else launch_e<false, false>(v, ff, s);
  } else {
    if (energy) launch_e<true, true>(v, ff, s);
    else launch_e<true, false>(v, ff, s);
  }
}

}  // namespace mdk
