// Truncated Lennard-Jones forces over the cell stencil (Section 3.2, Eq. 2) for gfx950.
//
// Pair force as in the paper's inner loop: with r2inv = 1/r^2 and r6inv = r2inv^3,
// F_i += (x_i - x_j) * r2inv * r6inv * (12 ljp2 r6inv - 6 ljp1), ljp2 = 4 eps sigma^12,
// ljp1 = 4 eps sigma^6, counted only for r^2 < rc^2 and pairs more than excl bonds
// apart along a chain.  Every pair is evaluated from both sides (as the paper's
// thread-per-atom kernel does), so each atom's force is a private sum: no atomics,
// and the order of the sum is fixed by the sorted cell lists.
//
// Coordinates come from the sorted payload.  k_lj_cell's are box coordinates modulo 128 A.  The
// lists' and the half shell's are relative to the centre of each atom's cell: a neighbour cell
// at offset (ox, oy, oz) contributes x_j + (ox, oy, oz) * edge in the home cell's frame.  Mixed
// precision keeps them as int32 fixed point (2^-25 A), so x_i - x_j is an exact integer rounded
// once to FP32; FP64 uses doubles.
//
// Kernels (the rest of the cell path is in md_group.hip):
//   k_lj_cell        mixed precision, one wavefront per home cell: the cell's atoms are
//                    wave-uniform (KMAX at a time) and the stencil's atoms, filtered by the
//                    box bounding the homes, stream across the lanes 64 at a time;
//   k_lj_tile        the same layout over the cell's neighbour list (nl mode);
//   k_lj_half        the same layout over half the stencil, each pair once, both forces
//                    added to int64 fixed-point accumulators (opt-in);
//   k_nl_build,      neighbour-list builds (Sections 3.1-3.2), per atom and per cell, and
//   k_nl_build_tile, the per-atom list walk.
//   k_lj_nl
#include "md_lj_common.h"

namespace mdk {
namespace {

// ---------------------------------------------------------------------------------
// Cell tile: one wave per home cell.  The wave lists its (2R+1)^3 stencil once, as a flat
// array of candidates in LDS (sorted-array index << 7 | stencil offset code), and streams
// that list 64 lanes at a time against up to KMAX home atoms held wave-uniform.
constexpr int kListCap = 1024;   // candidates a wave lists at a time
static_assert(kListCap / 64 <= 32, "the list build keeps one bit per 64-candidate step");
constexpr int kMaxStencil = (2 * kTileMaxR + 1) * (2 * kTileMaxR + 1) * (2 * kTileMaxR + 1);
static_assert(kMaxStencil <= 128, "stencil code must fit 7 bits");

template <typename Q>
struct Shift {
  Q x, y, z;   // stencil offset (ox, oy, oz) times the cell edge, in the payload's units
};

// Box b's stencil shift table (kShiftSlots entries, built on the host) into LDS.
template <typename Q>
__device__ __forceinline__ void load_shifts(const Views& v, int b, Shift<Q>* shifts) {
  const Shift<Q>* __restrict__ tab = static_cast<const Shift<Q>*>(v.shift_tab) + (int64_t)b * kShiftSlots;
  static_assert(kShiftSlots == 128, "two entries per lane of one wave");
  if (blockDim.x == 64) {   // one wave: two entries per lane, both loads in flight together
    const Shift<Q> a = tab[threadIdx.x], c = tab[threadIdx.x + 64];
    shifts[threadIdx.x] = a;
    shifts[threadIdx.x + 64] = c;
  } else {
    for (int c = (int)threadIdx.x; c < kShiftSlots; c += (int)blockDim.x) shifts[c] = tab[c];
  }
}

// Writes entries [c0, c0 + kListCap) of home cell lc's candidate list to list[]; returns
// the list's full length (the same on every lane).  Lane l lists stencil codes 2l and
// 2l + 1 (x-neighbours, so consecutive entries are mostly consecutive in memory).
__device__ __forceinline__ int fill_list(const Views& v, const BoxDev& B, int lc, int c0, uint32_t* list) {
  const int ln = lane();
  const int R = v.R, W = 2 * R + 1, W3 = W * W * W;
  const int M0 = B.M[0], M1 = B.M[1], M2 = B.M[2];
  const Cell3 k3 = cell_coords(lc, B);
  // both cells' bounds are loaded together (a code past the stencil reads the home cell's
  // and counts nothing)
  int start[2], n[2], c[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int code = min(2 * ln + h, W3 - 1);
    const Cell3 o = stencil_offset(code, R);
    int nx = k3.x + o.x, ny = k3.y + o.y, nz = k3.z + o.z;
    nx += nx < 0 ? M0 : 0;
    nx -= nx >= M0 ? M0 : 0;
    ny += ny < 0 ? M1 : 0;
    ny -= ny >= M1 ? M1 : 0;
    nz += nz < 0 ? M2 : 0;
    nz -= nz >= M2 ? M2 : 0;
    c[h] = B.cell_off + nx + M0 * (ny + M1 * nz);
  }
  int e[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    start[h] = v.cell_start[c[h]];
    e[h] = v.cell_start[c[h] + 1];
  }
#pragma unroll
  for (int h = 0; h < 2; ++h) n[h] = 2 * ln + h < W3 ? e[h] - start[h] : 0;
  int total;
  int f = wave_exclusive_scan(n[0] + n[1], total);
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int a1 = min(n[h], c0 + kListCap - f);
    for (int a = max(0, c0 - f); a < a1; ++a) list[f + a - c0] = ((uint32_t)(start[h] + a) << 7) | (2 * ln + h);
    f += n[h];
  }
  return total;
}

// The candidate list of home cell lc, entries [c0, c0 + kListCap), into list[]; returns its
// full length: the cell's own list, the candidates within rc + skin of any of its atoms at
// the last build (k_nl_build_tile), copied from HBM; a cell whose list outgrew its capacity
// streams its whole stencil instead (the bins of the build: every atom has moved less than
// half the skin since, and the stencil covers rc + skin, so every pair within rc is in it).
// The chunk is padded with the sentinel entry from its end up to and including the next
// multiple of 64 (list holds kListCap + 65 entries).
__device__ __forceinline__ int load_list(const Views& v, const BoxDev& B, int lc, int c0, uint32_t* list) {
  int n = v.nl_count[B.cell_off + lc];
  if (n > v.nl_cap) {
    n = fill_list(v, B, lc, c0, list);
  } else {
    const uint32_t* __restrict__ src = v.nl_list + B.nl_off + (int64_t)lc * v.nl_cap;
    const int m = min(kListCap, n - c0);
    for (int t = lane(); t < m; t += 64) list[t] = src[c0 + t];
  }
  const int cn = min(kListCap, n - c0);
  if (lane() <= ((cn + 63) & ~63) - cn) list[cn + lane()] = kSentinelEntry;
  return n;
}

struct BandEnergy {
  double e, es, w;
};

// Settles the cutoff-band pairs and the close contacts of one home group of a mixed tile wave,
// after its home forces are stored.  The recorded candidate steps (flat list positions) are
// revisited and their band pairs and close contacts queued in (step, home, lane) order,
// refilling the list where a step lies in another chunk.  Each queued band pair is re-decided
// in FP64 and, when outside, its FP32 force is taken back out; each close contact is evaluated
// in FP64 and added.  Both are summed per home over the lanes in a fixed order and applied in
// one rounding by the lane that stored that home (lane k << SHIFT for home k).  With more
// steps or pairs than the slots hold (not expected in a melt) every candidate of the group is
// walked again instead, from the full list (total entries).  LDS executes a wave's accesses in
// order and only this wave wrote its slots, so no barrier is needed.  `resident` is the chunk
// the list holds; it is updated.
template <bool ENERGY, bool UNI, int SHIFT>
__device__ __forceinline__ BandEnergy settle_group(const Views& v, int chain_len, int excl, double rc2,
                                                   const LjPair<float>& cf, const LjPair<double>& cd,
                                                   const BoxDev& B, Band bd, int lc, int total,
                                                   uint32_t* list, int& resident, const Shift<int>* shifts,
                                                   const int* steps, int32_t* bq, const int4* __restrict__ pay,
                                                   int hs, int g0, int kc, int nsteps) {
  const int ln = lane();
  float* f = static_cast<float*>(v.f_lj);
  double e = 0.0, es = 0.0, w = 0.0;
  auto candidate = [&](int t, int cn, int& jx, int& jy, int& jz, int32_t& jt) -> bool {
    jx = jy = jz = 0;
    jt = 0;
    if (t < cn) {
      const uint32_t ent = list[t];
      const int4 q = pay[ent >> 7];
      const Shift<int> sh = shifts[ent & 127];
      jt = pay_tag(q);
      jx = q.x + sh.x;
      jy = q.y + sh.y;
      jz = q.z + sh.z;
    }
    return t < cn;
  };
  auto window = [&](int i, int32_t& hlo, uint32_t& hspan) {
    const int32_t c0 = i - i % chain_len;
    hlo = max(i - excl, c0);
    hspan = (uint32_t)(min(i + excl, c0 + chain_len - 1) - hlo);
  };
  // one queued pair's correction on this lane: band (FP32, units of 2^25) or close (FP64)
  auto correct = [&](int32_t i, int32_t j, int tt, bool close, float& bx, float& by, float& bz, double& cx,
                     double& cy, double& cz) {
    double d[3], r2;
    const bool inside = inside_cutoff_f64(v.pos, v.N, B, i, j, rc2, d, r2);
    if (close)
      add_close_pair<ENERGY>(d, r2, pick(cd.f12, tt), pick(cd.f6, tt), pick(cd.e12, tt), pick(cd.e6, tt),
                             pick(cd.ecut, tt), cx, cy, cz, e, es, w);
    else if (!inside)
      remove_band_pair<ENERGY>(d, r2, pick(cf.f12, tt), pick(cf.f6, tt), pick(cf.e12, tt), pick(cf.e6, tt),
                               pick(cf.ecut, tt), bx, by, bz, e, es, w);
  };
  // home k's corrections summed over the lanes, added to its stored force in one rounding
  auto apply = [&](int k, float bx, float by, float bz, double cx, double cy, double cz) {
    bx = group_sum(bx, 0);
    by = group_sum(by, 0);
    bz = group_sum(bz, 0);
    cx = group_sum(cx, 0);
    cy = group_sum(cy, 0);
    cz = group_sum(cz, 0);
    if (ln == k << SHIFT) {
      const int32_t i = tag_index(pay_tag(pay[hs + g0 + k]));
      f[i] = (float)((double)f[i] + ((double)(bx * kInvFixF) + cx));
      f[v.N + i] = (float)((double)f[v.N + i] + ((double)(by * kInvFixF) + cy));
      f[2 * v.N + i] = (float)((double)f[2 * v.N + i] + ((double)(bz * kInvFixF) + cz));
    }
  };
  int qn = 0;   // queued pairs: j << 6 | type_j << 5 | close << 4 | k
  if (nsteps <= kBandSteps) {
    for (int s = 0; s < nsteps; ++s) {
      const int fs = steps[s];
      const int c0 = fs - fs % kListCap;
      if (c0 != resident) {
        load_list(v, B, lc, c0, list);
        resident = c0;
      }
      int jx, jy, jz;
      int32_t jt;
      const bool act = candidate(fs - c0 + ln, min(kListCap, total - c0), jx, jy, jz, jt);
      for (int k = 0; k < kc; ++k) {
        const int4 hq = pay[hs + g0 + k];
        int32_t hlo;
        uint32_t hspan;
        window(tag_index(pay_tag(hq)), hlo, hspan);
        const bool keep = act && (uint32_t)(tag_index(jt) - hlo) > hspan;
        const float r2s = r2_fix((float)(hq.x - jx), (float)(hq.y - jy), (float)(hq.z - jz));
        const bool qc = is_close(r2s, keep, bd);
        const bool qb = qc || in_band(r2s, keep, bd);
        const uint64_t qm = __builtin_amdgcn_ballot_w64(qb);
        const int at = qn + lanes_below(qm);
        if (qb && at < kBandQueue) bq[at] = (tag_index(jt) << 6) | (tag_type(jt) << 5) | ((int)qc << 4) | k;
        qn += __popcll(qm);
      }
    }
  }
  if (nsteps <= kBandSteps && qn <= kBandQueue) {
    float bx = 0.0f, by = 0.0f, bz = 0.0f;
    double cx = 0.0, cy = 0.0, cz = 0.0;
    int kq = -1;
    if (ln < qn) {
      const int32_t ent = bq[ln];
      kq = ent & 15;
      const int32_t htag = pay_tag(pay[hs + g0 + kq]);
      const int tt = UNI ? 0 : tag_type(htag) * 2 + ((ent >> 5) & 1);
      correct(tag_index(htag), ent >> 6, tt, ((ent >> 4) & 1) != 0, bx, by, bz, cx, cy, cz);
    }
    for (int k = 0; k < kc; ++k) {
      if (__builtin_amdgcn_ballot_w64(kq == k) == 0) continue;
      const bool mine = kq == k;
      apply(k, mine ? bx : 0.0f, mine ? by : 0.0f, mine ? bz : 0.0f, mine ? cx : 0.0, mine ? cy : 0.0,
            mine ? cz : 0.0);
    }
  } else {
    for (int k = 0; k < kc; ++k) {
      const int4 hq = pay[hs + g0 + k];
      const int32_t i = tag_index(pay_tag(hq));
      int32_t hlo;
      uint32_t hspan;
      window(i, hlo, hspan);
      float bx = 0.0f, by = 0.0f, bz = 0.0f;
      double cx = 0.0, cy = 0.0, cz = 0.0;
      for (int c0 = 0; c0 < total; c0 += kListCap) {
        if (c0 != resident) {
          load_list(v, B, lc, c0, list);
          resident = c0;
        }
        const int cn = min(kListCap, total - c0);
        for (int t0 = 0; t0 < cn; t0 += 64) {
          int jx, jy, jz;
          int32_t jt;
          const bool act = candidate(t0 + ln, cn, jx, jy, jz, jt);
          const int32_t jidx = tag_index(jt);
          const bool keep = act && (uint32_t)(jidx - hlo) > hspan;
          const float r2s = r2_fix((float)(hq.x - jx), (float)(hq.y - jy), (float)(hq.z - jz));
          const bool qc = is_close(r2s, keep, bd);
          if (qc || in_band(r2s, keep, bd))
            correct(i, jidx, UNI ? 0 : tag_type(pay_tag(hq)) * 2 + tag_type(jt), qc, bx, by, bz, cx, cy, cz);
        }
      }
      apply(k, bx, by, bz, cx, cy, cz);
    }
  }
  return BandEnergy{e, es, w};
}

// Sums KMAX per-lane force accumulators (three components each) over the 64 lanes in a
// fixed order.  Recursive halving: at each of the first log2(KMAX) levels a lane keeps half of
// its values and adds the partner's copy of that half, so the 3 KMAX sums take 3 KMAX - 3
// exchanges (instead of 18 KMAX for separate butterflies); then a butterfly over the remaining
// lane bits.  Level lv splits the lanes by bit 5 - lv and exchanges through kLevel[lv] (for
// bit 2 the partner l ^ 7 also differs in bit 2 only among the bits not yet summed).
// Afterwards every lane of [h * 64/KMAX, (h + 1) * 64/KMAX) holds accumulator h's sums.
template <typename P, int KMAX>
__device__ __forceinline__ void sum_homes(int ln, P (&ax)[KMAX], P (&ay)[KMAX], P (&az)[KMAX], P& sx, P& sy,
                                          P& sz) {
  constexpr int LV = KMAX == 16 ? 4 : (KMAX == 8 ? 3 : (KMAX == 4 ? 2 : (KMAX == 2 ? 1 : 0)));
  static_assert((1 << LV) == KMAX, "KMAX must be 1, 2, 4, 8 or 16");
  constexpr int NV = 3 * KMAX;
  P val[NV];
#pragma unroll
  for (int k = 0; k < KMAX; ++k) {
    val[3 * k] = ax[k];
    val[3 * k + 1] = ay[k];
    val[3 * k + 2] = az[k];
  }
#pragma unroll
  for (int lv = 0; lv < LV; ++lv) {
#pragma unroll
    for (int i = 0; i < (NV >> lv) / 2; ++i) {
      const int h = (NV >> lv) / 2 + i;
      if (lv < 2) {
        // lanes below the split keep val[i], those above val[h]
        val[i] = swap_sum(val[i], val[h], kLevel[lv]);
      } else {
        const bool hi = (ln & (32 >> lv)) != 0;
        const P send = hi ? val[i] : val[h];
        const P keep = hi ? val[h] : val[i];
        val[i] = keep + partner(send, lv == 2 ? Xl::Ror8 : Xl::Mirror8);
      }
    }
  }
#pragma unroll
  for (int c = 0; c < 3; ++c) val[c] = group_sum(val[c], LV);
  sx = val[0];
  sy = val[1];
  sz = val[2];
}

// Occupancy: the mixed form with 8 homes is held to 6 waves per SIMD (80 VGPRs; it uses 77 to 79, and with
// energies spills 7 to 12 of them).  The bounds of the other forms are not met or not reached: 4 homes run
// at 6 waves (77 to 79 VGPRs; with energies 4 or 5), 16 at 5 (with energies 4), FP64 at 5 or 6 (72 to 91).
// (the homes and the sorted order are those of the last build, the payload the one refreshed since)
template <bool FP64, bool ENERGY, bool UNI, int KMAX>
__global__ __launch_bounds__(64 * kTileWaves)
__attribute__((amdgpu_waves_per_eu(FP64 ? 8 : (KMAX >= 16 ? 4 : (KMAX <= 4 ? 8 : 6)))))
void k_lj_tile(Views v, FFDev ff, LjPair<float> cf, LjPair<double> cd) {
  using PayT = std::conditional_t<FP64, Pay64, int4>;
  using P = std::conditional_t<FP64, double, float>;
  using Q = std::conditional_t<FP64, double, int>;     // coordinate type
  constexpr int LV = KMAX == 16 ? 4 : (KMAX == 8 ? 3 : (KMAX == 4 ? 2 : (KMAX == 2 ? 1 : 0)));   // log2(KMAX)
  static_assert((1 << LV) == KMAX, "KMAX must be 1, 2, 4, 8 or 16");
  __shared__ uint32_t list[kTileWaves][kListCap + 65];   // + the padding to a whole step, + 1
  __shared__ Shift<Q> shifts[kShiftSlots];
  __shared__ dd red[kTileWaves][3];
  __shared__ int32_t bq[kTileWaves][kBandQueue];   // queued pairs: j << 6 | type_j << 5 | close << 4 | k
  __shared__ int bsteps[kTileWaves][kBandSteps];    // flat list position of each recorded step

  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int ln = lane();
  // Workgroups are dealt to the 8 XCDs round-robin; give each XCD a contiguous run of
  // home cells (a slab of the box) so its L2 holds one neighbourhood of the payload.
  const int per_xcd = (int)gridDim.x / kXcds;
  const int blk = ((int)blockIdx.x % kXcds) * per_xcd + (int)blockIdx.x / kXcds;
  if (blk >= v.n_lj_blocks) return;
  const int b = v.lj_blk_box[blk];
  const BoxDev& B = v.boxes[b];
  const int lc = (blk - B.lj_blk_off) * kTileWaves + wave;   // home cell within the box
  const bool wact = lc < B.n_cells;
  const int32_t* __restrict__ cs = v.cell_start;
  const PayT* __restrict__ pay = static_cast<const PayT*>(v.payload);

  // stencil offsets in the payload's units (the same for every wave of the block)
  load_shifts(v, b, shifts);
  int total = 0, resident = 0;
  if (wact) total = __builtin_amdgcn_readfirstlane(load_list(v, B, lc, 0, list[wave]));
  __syncthreads();

  double e = 0.0, es = 0.0, w = 0.0;
  if (wact) {
    const int hs = __builtin_amdgcn_readfirstlane(cs[B.cell_off + lc]);
    const int hn = __builtin_amdgcn_readfirstlane(cs[B.cell_off + lc + 1]) - hs;
    const Band bd = band_of(cf);
    // one type pair (mixed): forces are summed divided by f6 (see pair_fix)
    const float f12_fold = cf.f12_fold;
    const float fscale = UNI ? kInvFixF * cf.f6[0] : kInvFixF;
    for (int g0 = 0; g0 < hn; g0 += KMAX) {
      const int kc = min(KMAX, hn - g0);
      // The group's homes, one per lane (lane k < kc holds home k), loaded together, with each
      // home's exclusion window (the sorted indices within excl bonds along its chain); then
      // broadcast to wave-uniform values.  A lane past the group holds zeros and a window
      // that excludes every candidate.
      PayT qh{};
      int32_t lo_l = 0, ht_l = 0;
      uint32_t span_l = 0xffffffffu;
      if (ln < kc) {
        qh = pay[hs + g0 + ln];
        const int32_t i = tag_index(pay_tag(qh));
        const int32_t c0 = chain_first(i, ff);
        lo_l = max(i - ff.excl, c0);
        span_l = (uint32_t)(min(i + ff.excl, c0 + ff.chain_len - 1) - lo_l);
        ht_l = tag_type(pay_tag(qh));
      }
      // the homes broadcast to wave-uniform values
      Q hx[KMAX], hy[KMAX], hz[KMAX];
      int32_t lo[KMAX], hti[KMAX];
      uint32_t span[KMAX];
      P ax[KMAX], ay[KMAX], az[KMAX];
#pragma unroll
      for (int k = 0; k < KMAX; ++k) {
        ax[k] = ay[k] = az[k] = (P)0;
        hx[k] = lane_value(qh.x, k);
        hy[k] = lane_value(qh.y, k);
        hz[k] = lane_value(qh.z, k);
        lo[k] = lane_value(lo_l, k);
        span[k] = (uint32_t)lane_value((int32_t)span_l, k);
        hti[k] = lane_value(ht_l, k);
      }
      int nsteps = 0;       // candidate steps with a band pair or a close contact (wave-uniform)
      int32_t bmax = 0;     // bits of the largest r2s counted since the last band check
      for (int c0 = 0; c0 < total; c0 += kListCap) {
        if (c0 != resident) {
          load_list(v, B, lc, c0, list[wave]);
          resident = c0;
        }
        const int cn = min(kListCap, total - c0);
        for (int t0 = 0; t0 < cn; t0 += 64) {
          // the list is padded to whole steps with the sentinel, which lies beyond the cutoff
          const uint32_t ent = list[wave][t0 + ln];
          const PayT q = pay[ent >> 7];
          const Shift<Q> sh = shifts[ent & 127];
          const int32_t jt = pay_tag(q);
          const Q jx = q.x + sh.x, jy = q.y + sh.y, jz = q.z + sh.z;
          const int32_t jidx = tag_index(jt);
          const int jtype = tag_type(jt);
          bool near = false;    // a close contact on this lane in this step (mixed)
          // the group's home count, re-read each step as an opaque scalar: the compiler then
          // tests k < kc with a scalar compare per home instead of holding KMAX lane masks
          int kcs = kc;
          asm volatile("" : "+s"(kcs));
#pragma unroll
          for (int k = 0; k < KMAX; ++k) {
            if (k < kcs) {
              const bool keep = (uint32_t)(jidx - lo[k]) > span[k];
              const int tt = UNI ? 0 : hti[k] * 2 + jtype;
              if constexpr (FP64)
                pair_f64<ENERGY>(hx[k] - jx, hy[k] - jy, hz[k] - jz, keep, ff.rc2, pick(cd.f12, tt),
                                 pick(cd.f6, tt), pick(cd.e12, tt), pick(cd.e6, tt), pick(cd.ecut, tt), ax[k],
                                 ay[k], az[k], e, es, w);
              else
                pair_fix<ENERGY, UNI>(hx[k] - jx, hy[k] - jy, hz[k] - jz, keep, bd,
                                                  UNI ? f12_fold : pick(cf.f12, tt), pick(cf.f6, tt),
                                                  pick(cf.e12, tt), pick(cf.e6, tt), pick(cf.ecut, tt), ax[k],
                                                  ay[k], az[k], e, es, w, bmax, near);
            }
          }
          if constexpr (!FP64) {
            // rare: a lane counted a pair in the cutoff band or met a close contact; note the step
            if (__builtin_amdgcn_ballot_w64(bmax >= __float_as_int(bd.lo) || near) != 0) {
              bmax = 0;
              if (nsteps < kBandSteps && ln == 0) bsteps[wave][nsteps] = c0 + t0;
              ++nsteps;
            }
          }
        }
      }
      // Sum each home atom's partial forces over the 64 lanes in a fixed order, as sum_homes
      // does (written out here: the explicit exchange patterns keep the register allocation
      // tighter): lanes [h * 64/KMAX, (h + 1) * 64/KMAX) then hold home h's sums, and the first
      // of them stores it (and later applies its band and close-contact corrections).
      P* f = static_cast<P*>(v.f_lj);
      {
        constexpr int NV = 3 * KMAX;
        P val[NV];
#pragma unroll
        for (int k = 0; k < KMAX; ++k) {
          val[3 * k] = ax[k];
          val[3 * k + 1] = ay[k];
          val[3 * k + 2] = az[k];
        }
#pragma unroll
        for (int lv = 0; lv < LV; ++lv) {
#pragma unroll
          for (int i = 0; i < (NV >> lv) / 2; ++i) {
            const int h = (NV >> lv) / 2 + i;
            if (lv < 2) {
              val[i] = swap_sum(val[i], val[h], kLevel[lv]);
            } else {
              const bool hi = (ln & (32 >> lv)) != 0;
              const P send = hi ? val[i] : val[h];
              const P keep = hi ? val[h] : val[i];
              val[i] = keep + partner(send, lv == 2 ? Xl::Ror8 : Xl::Mirror8);
            }
          }
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) val[c] = group_sum(val[c], LV);
        P sx = val[0], sy = val[1], sz = val[2];
        if constexpr (!FP64) {
          sx *= fscale;
          sy *= fscale;
          sz *= fscale;
        }
        const int hk = ln >> (6 - LV);
        const int32_t i = tag_index(__shfl(pay_tag(qh), hk));   // home hk's index, from lane hk
        if ((ln & ((64 >> LV) - 1)) == 0 && hk < kc) {
          f[i] = sx;
          f[v.N + i] = sy;
          f[2 * v.N + i] = sz;
        }
      }
      if constexpr (!FP64) {
        if (nsteps > 0) {
          const BandEnergy be = settle_group<ENERGY, UNI, 6 - LV>(v, ff.chain_len, ff.excl, ff.rc2, cf, cd, B, bd,
                                                                       lc, total, list[wave], resident, shifts,
                                                                       bsteps[wave], bq[wave], pay, hs, g0, kc, nsteps);
          if (ENERGY) {
            e += be.e;
            es += be.es;
            w += be.w;
          }
        }
      }
    }
  }
  if (ENERGY) block_energy<kTileWaves>(e, es, w, red, v.part_lj + (int64_t)blk * 3);
}

// ---------------------------------------------------------------------------------
// Cell path, mixed precision (MD_LJ_CELLTILE, MD_LJ_CELLTILE_NB): one wave per home cell.  The cells
// of a stencil row are consecutive in the sorted order, so the (2R + 1)^3 stencil is (2R + 1)^2 runs,
// or two where the box's edge cuts a row; lane r < 32 finds the part of row r inside the box and lane
// 32 + r the part across the edge.  The wave streams the runs 64 candidates at a time (each lane's
// run from a bit mask of run starts); a candidate nearer than rc to the box bounding up to KMAX homes
// goes, in the frame of the cell's first atom, to a list in LDS, which is then taken 64 at a time
// against the homes, held wave-uniform.  The payload is in box coordinates (modulo 128 A).
//
// Bound: VALU instructions (1,419 per cell of 5.1 atoms at R = 2, about half of them pairs: 24 for
// each home and 64 candidates; the rest set-up, 10 windows of 35 and the sums).  The form before listed
// every candidate's index in LDS and gathered the payload twice (1,565 instructions).  LJ pass, event
// timing: 300,000 atoms 159 -> 152 us; a step of 24 boxes of 453,600 atoms 272 -> 262 us, of 3,000 atoms
// 40.0 -> 38.7 us, of 3,000,000 atoms 1,630 -> 1,618 us.  LJ force error as before (12 relaxed
// melts of 3,000 and 15,000 atoms against 80-bit arithmetic: rms 5.16e-7 and 5.17e-7 of the RMS force,
// largest 6.8e-6 and 6.7e-6).  Measured as well: the homes by scalar loads, no change.
// fixed-point coordinates modulo 2^32
__device__ inline int fix_add(int a, int b) { return (int)((uint32_t)a + (uint32_t)b); }
__device__ inline int fix_sub(int a, int b) { return (int)((uint32_t)a - (uint32_t)b); }

constexpr int kRunWindows = 64;   // 64-candidate windows whose run starts are marked at a time
constexpr int kRunBatch = 2;      // windows whose loads are in flight together
constexpr double kFilterGap = 1e-3;   // A added to the filter's reach: the rounding of its FP32 distances
constexpr int kStage = 288;           // candidates held in LDS (16 B each): 24 waves per CU with the rest (at 304, 21)

// Registers: 16 homes, 5 waves per SIMD with 12 spilled 179 us, 4 without 189 (LJ pass, 300,000 atoms, R = 2);
// 8 homes at 6 waves against 5, an evaluation of 300,000 atoms: with energies (12 spilled) 234 against 238 us,
// two types (4 spilled) 186 against 191, two types with energies (22 spilled) 349 against 339.
template <bool ENERGY, bool UNI, int KMAX, bool BRANCHLESS>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(KMAX >= 16 ? (ENERGY ? 4 : 5) : 6)))
void k_lj_cell(Views v, FFDev ff, LjPair<float> cf, LjPair<double> cd) {
  constexpr int LV = KMAX == 16 ? 4 : (KMAX == 8 ? 3 : 2);   // log2(KMAX)
  static_assert((1 << LV) == KMAX, "KMAX must be 4, 8 or 16");
  static_assert(kTileWaves == 1, "one wave per block");
  static_assert((2 * kTileMaxR + 1) * (2 * kTileMaxR + 1) <= 32, "a row per lane of half a wave");
  constexpr int CAP = kStage;
  __shared__ int4 list[CAP];
  __shared__ int4 runs[64];   // x, y, z: added to a payload coordinate; w: to a flat position, in bytes of payload
  __shared__ unsigned long long marks[kRunWindows];
  __shared__ double exact[KMAX][3];   // forces of the pairs evaluated in FP64
  __shared__ dd red[1][3];

  const int ln = lane();
  // Workgroups are dealt to the 8 XCDs round-robin; give each XCD a contiguous run of
  // home cells (a slab of the box) so its L2 holds one neighbourhood of the payload.
  const int per_xcd = (int)gridDim.x / kXcds;
  const int blk = ((int)blockIdx.x % kXcds) * per_xcd + (int)blockIdx.x / kXcds;
  if (blk >= v.n_lj_blocks) return;
  const int b = v.lj_blk_box[blk];
  const BoxDev& B = v.boxes[b];
  const int lc = blk - B.lj_blk_off;   // home cell within the box
  const int32_t* __restrict__ cs = v.cell_start;
  const int4* __restrict__ pay = static_cast<const int4*>(v.payload);
  double e = 0.0, es = 0.0, w = 0.0;

  const int hs = uni(cs[B.cell_off + lc]), hn = uni(cs[B.cell_off + lc + 1]) - hs;
  if (hn > 0) {
    // ---- the runs ----
    const int R = v.R, W = 2 * R + 1;
    const int M0 = B.M[0], M1 = B.M[1], M2 = B.M[2];
    const Cell3 k3 = cell_coords(lc, B);
    const int row = ln & 31;
    const int oz = (int)(((float)row + 0.5f) * rcp_f((float)W)) - R, oy = row - (oz + R) * W - R;
    int ny = k3.y + oy, nz = k3.z + oz;
    const int wy = ny < 0 ? -1 : (ny >= M1 ? 1 : 0), wz = nz < 0 ? -1 : (nz >= M2 ? 1 : 0);
    ny -= wy * M1;
    nz -= wz * M2;
    const int xlo = k3.x - R, xhi = k3.x + R;
    // (M0 >= 2 R + 1: a row crosses at most one edge)
    int a = max(xlo, 0), z = min(xhi, M0 - 1), wx = 0;
    if (ln >= 32) {
      wx = xlo < 0 ? -1 : (xhi >= M0 ? 1 : 0);
      a = wx < 0 ? xlo + M0 : 0;
      z = wx < 0 ? M0 - 1 : (wx > 0 ? xhi - M0 : -1);
    }
    int n = 0, start = 0;
    if (row < W * W && a <= z) {
      const int c = B.cell_off + M0 * (ny + M1 * nz);
      start = cs[c + a];
      n = cs[c + z + 1] - start;
    }
    const int4 q0 = pay[hs];
    const Shift<int> edge = static_cast<const Shift<int>*>(v.shift_tab)[(int64_t)b * kShiftSlots + kBoxCode];
    int total;
    const int f = wave_exclusive_scan(n, total);
    total = uni(total);
    const uint64_t some = __builtin_amdgcn_ballot_w64(n > 0);
    if (n > 0)
      runs[lanes_below(some)] =
          make_int4((int)((uint32_t)wx * (uint32_t)edge.x - (uint32_t)q0.x), (int)((uint32_t)wy * (uint32_t)edge.y - (uint32_t)q0.y),
                    (int)((uint32_t)wz * (uint32_t)edge.z - (uint32_t)q0.z), (start - f) * 16);
    const int mark = n > 0 ? f - 1 : -1;   // a run (but the first) marks the position before it
    const float rc = __builtin_amdgcn_sqrtf((float)ff.rc2) + (float)kFilterGap;
    const float rcf = rc * rc * ((float)kFix * (float)kFix);

    for (int g0 = 0; g0 < hn; g0 += KMAX) {
      const int kc = min(KMAX, hn - g0);
      // The group's homes, one per lane (lane k < kc holds home k), each with its exclusion window
      // (the atoms within excl bonds along its chain, in tag units).  A lane past the group repeats
      // the last home with a window that excludes every candidate.
      const int4 qh = pay[hs + g0 + min(ln, kc - 1)];
      const int hxl = fix_sub(qh.x, q0.x), hyl = fix_sub(qh.y, q0.y), hzl = fix_sub(qh.z, q0.z);
      int32_t lo_l = 0, span_l = -1;
      if (ln < kc) {
        const int32_t i = tag_index(pay_tag(qh));
        const int32_t c0 = chain_first(i, ff), first = max(i - ff.excl, c0);
        lo_l = first << 4;
        span_l = ((min(i + ff.excl, c0 + ff.chain_len - 1) - first) << 4) | 15;
      }
      // the box bounding the homes (in vector registers: the clamp reads both bounds of an axis)
      const float bxl = in_vgpr((float)first_lanes_min<KMAX>(hxl)), bxh = in_vgpr((float)first_lanes_max<KMAX>(hxl));
      const float byl = in_vgpr((float)first_lanes_min<KMAX>(hyl)), byh = in_vgpr((float)first_lanes_max<KMAX>(hyl));
      const float bzl = in_vgpr((float)first_lanes_min<KMAX>(hzl)), bzh = in_vgpr((float)first_lanes_max<KMAX>(hzl));
      uint32_t hx[KMAX], hy[KMAX], hz[KMAX];   // (unsigned: the padding's differences wrap)
      int32_t lo[KMAX], hti[KMAX];
      uint32_t span[KMAX];
      float ax[KMAX], ay[KMAX], az[KMAX];
#pragma unroll
      for (int k = 0; k < KMAX; ++k) {
        ax[k] = ay[k] = az[k] = 0.0f;
        hx[k] = (uint32_t)lane_value(hxl, k);
        hy[k] = (uint32_t)lane_value(hyl, k);
        hz[k] = (uint32_t)lane_value(hzl, k);
        lo[k] = lane_value(lo_l, k);
        span[k] = (uint32_t)lane_value(span_l, k);
        hti[k] = UNI ? 0 : lane_value(tag_type(pay_tag(qh)), k);
      }
      bool settled = false;   // exact[] holds this group's sums
      int m = 0;              // candidates in list[]
      int t0 = -64 * kRunWindows, w0 = 0, nw = 0, before = 0;
      int mlo = 0, mhi = 0;
      bool more = true;
      do {
        // ---- fill the list ----
        while (m <= CAP - 64 * kRunBatch) {
          if (w0 >= nw) {
            t0 += 64 * kRunWindows;
            more = t0 < total;
            if (!more) break;
            marks[ln] = 0ull;
            lds_order();
            const int at = mark - t0;
            if (mark >= 0 && at >= 0 && at < 64 * kRunWindows) atomicOr(&marks[at >> 6], 1ull << (at & 63));
            lds_order();
            const unsigned long long mk = marks[ln];
            mlo = (int)(uint32_t)mk;
            mhi = (int)(uint32_t)(mk >> 32);
            before = __popcll(__builtin_amdgcn_ballot_w64(mark >= 0 && at < 0));
            nw = (min(total - t0, 64 * kRunWindows) + 63) >> 6;
            w0 = 0;
          }
          int4 q[kRunBatch], run[kRunBatch];
          uint64_t in[kRunBatch];
#pragma unroll
          for (int u = 0; u < kRunBatch; ++u) {
            // lanes past the candidates repeat the last one and are dropped below
            const int first = t0 + 64 * (w0 + u), t = first + ln;
            const uint32_t wl = (uint32_t)__builtin_amdgcn_readlane(mlo, w0 + u);
            const uint32_t wh = (uint32_t)__builtin_amdgcn_readlane(mhi, w0 + u);
            const int r = (int)__builtin_amdgcn_mbcnt_hi(wh, __builtin_amdgcn_mbcnt_lo(wl, (uint32_t)before));
            before += __popc(wl) + __popc(wh);
            const int left = total - first;
            in[u] = left >= 64 ? ~0ull : (left > 0 ? (1ull << left) - 1ull : 0ull);
            run[u] = runs[r];
            q[u] = *reinterpret_cast<const int4*>(reinterpret_cast<const char*>(pay) +
                                                  (uint32_t)((min(t, total - 1) << 4) + run[u].w));
          }
#pragma unroll
          for (int u = 0; u < kRunBatch; ++u) {
            asm volatile("" : "+v"(q[u].w));   // (else the tag is loaded by itself once the filter has passed)
            const int cx = fix_add(q[u].x, run[u].x), cy = fix_add(q[u].y, run[u].y), cz = fix_add(q[u].z, run[u].z);
            const float gx = (float)cx, gy = (float)cy, gz = (float)cz;
            const float dx = gx - __builtin_amdgcn_fmed3f(gx, bxl, bxh);
            const float dy = gy - __builtin_amdgcn_fmed3f(gy, byl, byh);
            const float dz = gz - __builtin_amdgcn_fmed3f(gz, bzl, bzh);
            const uint64_t pm = __builtin_amdgcn_ballot_w64(r2_fix(dx, dy, dz) < rcf) & in[u];
            if (__builtin_amdgcn_inverse_ballot_w64(pm))
              list[__builtin_amdgcn_mbcnt_hi((uint32_t)(pm >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)pm, (uint32_t)m))] =
                  make_int4(cx, cy, cz, q[u].w);
            m += __popcll(pm);
          }
          w0 += kRunBatch;
        }
        if (!more) {   // whole steps: padded with candidates 64 A from the cell's first atom
          const int pad = ((m + 63) & ~63) - m;
          if (ln < pad) list[m + ln] = make_int4(INT32_MIN, INT32_MIN, INT32_MIN, 0);
          m += pad;
        }
        lds_order();
        // ---- the whole steps of the list against the homes ----
        const int ns = m >> 6;
#pragma unroll 1
        for (int s = 0; s < ns; ++s) {
          const int4 q = list[64 * s + ln];
          const int32_t jt = pay_tag(q);
          const bool jtype = tag_type(jt) != 0;
          // the pair factors for a home of type 0 and of type 1
          const float f12_0 = UNI ? cf.f12_fold : (jtype ? cf.f12[1] : cf.f12[0]);
          const float f12_1 = UNI ? cf.f12_fold : (jtype ? cf.f12[3] : cf.f12[2]);
          const float f6_0 = UNI ? 1.0f : (jtype ? cf.f6[1] : cf.f6[0]);
          const float f6_1 = UNI ? 1.0f : (jtype ? cf.f6[3] : cf.f6[2]);
          uint64_t rare = 0;   // lanes with a close contact or a pair whose side of the cutoff FP32 cannot tell
          // the group's home count, re-read each step as an opaque scalar: the compiler then
          // tests k < kc with a scalar compare per home instead of holding KMAX lane masks
          int kcs = kc;
          asm volatile("" : "+s"(kcs));
#pragma unroll
          for (int k = 0; k < KMAX; ++k) {
            if (k < kcs) {
              const uint64_t keep = __builtin_amdgcn_ballot_w64((uint32_t)(jt - lo[k]) > span[k]);
              const float dx = (float)(int)(hx[k] - (uint32_t)q.x), dy = (float)(int)(hy[k] - (uint32_t)q.y),
                          dz = (float)(int)(hz[k] - (uint32_t)q.z);
              const float r2s = r2_fix(dx, dy, dz);
              // (lane masks: and-ed by the scalar unit)
              const uint64_t in = keep & __builtin_amdgcn_ballot_w64(r2s < cf.band_hi);
              const uint64_t plain =
                  __builtin_amdgcn_ballot_w64((uint32_t)(__float_as_int(r2s) - __float_as_int(cf.close)) <
                                              (uint32_t)(__float_as_int(cf.band_lo) - __float_as_int(cf.close)));
              const bool hit = __builtin_amdgcn_inverse_ballot_w64(in & plain);
              rare |= in & ~plain;
              if (BRANCHLESS || hit) {
                const float r2i = rcp_f(r2s) * kFix2F;
                const float r4 = r2i * r2i, r6 = r4 * r2i;
                const float t6 = UNI ? __builtin_fmaf(f12_0, r6, -1.0f)
                                     : __builtin_fmaf(hti[k] ? f12_1 : f12_0, r6, -(hti[k] ? f6_1 : f6_0));
                float fs = (r4 * r4) * t6;
                if (BRANCHLESS) fs = hit ? fs : 0.0f;
                ax[k] = __builtin_fmaf(fs, dx, ax[k]);
                ay[k] = __builtin_fmaf(fs, dy, ay[k]);
                az[k] = __builtin_fmaf(fs, dz, az[k]);
                if (ENERGY && hit) {
                  const int tt = UNI ? 0 : hti[k] * 2 + (int)jtype;
                  const float en = r6 * (pick(cf.e12, tt) * r6 - pick(cf.e6, tt));
                  e += (double)en;
                  es += (double)en - (double)pick(cf.ecut, tt);
                  w += (double)(UNI ? r6 * t6 * cf.f6[0] : r6 * t6);
                }
              }
            }
          }
          if (rare != 0) {
            // those pairs from the FP64 positions, summed over the lanes in a fixed order
            if (!settled && ln < KMAX) exact[ln][0] = exact[ln][1] = exact[ln][2] = 0.0;
            settled = true;
            lds_order();
#pragma unroll 1
            for (int k = 0; k < kc; ++k) {
              const int4 h = pay[hs + g0 + k];
              const int32_t i = tag_index(pay_tag(h)), c0 = chain_first(i, ff), first = max(i - ff.excl, c0);
              const uint32_t wide = (uint32_t)(min(i + ff.excl, c0 + ff.chain_len - 1) - first);
              const float r2s = r2_fix((float)fix_sub(fix_sub(h.x, q0.x), q.x), (float)fix_sub(fix_sub(h.y, q0.y), q.y),
                                       (float)fix_sub(fix_sub(h.z, q0.z), q.z));
              const bool exactly = (uint32_t)(tag_index(jt) - first) > wide && r2s < cf.band_hi &&
                                   !(r2s >= cf.close && r2s < cf.band_lo);
              if (__builtin_amdgcn_ballot_w64(exactly) == 0) continue;   // another home's
              double px = 0.0, py = 0.0, pz = 0.0;
              if (exactly) {
                double d[3], r2;
                const int tt = UNI ? 0 : tag_type(pay_tag(h)) * 2 + (int)jtype;
                if (inside_cutoff_f64(v.pos, v.N, B, i, tag_index(jt), ff.rc2, d, r2))
                  add_close_pair<ENERGY>(d, r2, pick(cd.f12, tt), pick(cd.f6, tt), pick(cd.e12, tt), pick(cd.e6, tt),
                                         pick(cd.ecut, tt), px, py, pz, e, es, w);
              }
              px = group_sum(px, 0);
              py = group_sum(py, 0);
              pz = group_sum(pz, 0);
              if (ln == 0) {
                exact[k][0] += px;
                exact[k][1] += py;
                exact[k][2] += pz;
              }
              lds_order();
            }
          }
        }
        if (more) {   // what is left moves to the front (LDS runs a wave's accesses in order)
          const int rest = m & 63;
          if (ln < rest) list[ln] = list[64 * ns + ln];
          m = rest;
          lds_order();
        }
      } while (more);
      // ---- each home's sums over the 64 lanes in a fixed order: lanes [h * 64/KMAX, (h + 1) * 64/KMAX)
      // then hold home h's, and the first of them stores it (sum_homes written out: the explicit
      // exchange patterns keep the register allocation tighter) ----
      constexpr int NV = 3 * KMAX;
      float val[NV];
#pragma unroll
      for (int k = 0; k < KMAX; ++k) {
        val[3 * k] = ax[k];
        val[3 * k + 1] = ay[k];
        val[3 * k + 2] = az[k];
      }
#pragma unroll
      for (int lv = 0; lv < LV; ++lv) {
#pragma unroll
        for (int i = 0; i < (NV >> lv) / 2; ++i) {
          const int h = (NV >> lv) / 2 + i;
          if (lv < 2) {
            val[i] = swap_sum(val[i], val[h], kLevel[lv]);
          } else {
            const bool hi = (ln & (32 >> lv)) != 0;
            const float send = hi ? val[i] : val[h];
            const float keep = hi ? val[h] : val[i];
            val[i] = keep + partner(send, lv == 2 ? Xl::Ror8 : Xl::Mirror8);
          }
        }
      }
#pragma unroll
      for (int c = 0; c < 3; ++c) val[c] = group_sum(val[c], LV);
      const int hk = ln >> (6 - LV);
      const int32_t i = tag_index(__shfl(pay_tag(qh), hk));   // home hk's index, from lane hk
      if ((ln & ((64 >> LV) - 1)) == 0 && hk < kc) {
        const double sc = (double)kInvFixF * (UNI ? cd.f6[0] : 1.0);   // fixed-point units; divided by f6 with one type pair
        double ox = (double)val[0] * sc, oyv = (double)val[1] * sc, ozv = (double)val[2] * sc;
        if (settled) {
          ox += exact[hk][0];
          oyv += exact[hk][1];
          ozv += exact[hk][2];
        }
        float* fo = static_cast<float*>(v.f_lj);
        fo[i] = (float)ox;
        fo[v.N + i] = (float)oyv;
        fo[2 * v.N + i] = (float)ozv;
      }
      lds_order();
    }
  }
  if (ENERGY) block_energy<1>(e, es, w, red, v.part_lj + (int64_t)blk * 3);
}

// ---------------------------------------------------------------------------------
// Newton-3 half shell (MD_LJ_HALFSHELL, opt-in; Section 4.2 names as a cost of its
// thread-per-atom kernels that every pair is computed twice).  Each pair is evaluated once:
// a home cell's wave lists its own atoms and the forward half of its stencil (codes above the
// centre), and takes an in-cell pair only from the lower of the two sorted positions.  The
// force on each candidate (the reaction, summed on its lane over the group's homes) and on
// each home (summed over the lanes) are added to per-atom int64 fixed-point accumulators
// (units of 2^-32 kcal/mol/A) with device atomics.  Integer sums do not depend on the order of
// the additions, so the result is deterministic; k_half_finish turns the accumulators into the
// force array and clears them for the next evaluation.  Band pairs are decided from the FP64
// positions before they are counted.
constexpr double kHalfFix = 4294967296.0;   // accumulator units per kcal/mol/A

// List of home cell lc for the half shell, entries [c0, c0 + kListCap): lane 0 lists the home
// cell (its atoms come first, at positions [0, hn)), lanes 1..(W^3 - 1)/2 the forward cells.
__device__ __forceinline__ int fill_list_half(const Views& v, const BoxDev& B, int lc, int c0, uint32_t* list) {
  const int ln = lane();
  const int R = v.R, W = 2 * R + 1, W3 = W * W * W, ctr = (W3 - 1) / 2;
  const int M0 = B.M[0], M1 = B.M[1], M2 = B.M[2];
  const Cell3 k3 = cell_coords(lc, B);
  const int code = ctr + ln;
  int start = 0, n = 0;
  if (code < W3) {
    const Cell3 o = stencil_offset(code, R);
    int nx = k3.x + o.x, ny = k3.y + o.y, nz = k3.z + o.z;
    nx += nx < 0 ? M0 : 0;
    nx -= nx >= M0 ? M0 : 0;
    ny += ny < 0 ? M1 : 0;
    ny -= ny >= M1 ? M1 : 0;
    nz += nz < 0 ? M2 : 0;
    nz -= nz >= M2 ? M2 : 0;
    const int c = B.cell_off + nx + M0 * (ny + M1 * nz);
    start = v.cell_start[c];
    n = v.cell_start[c + 1] - start;
  }
  int total;
  const int f = wave_exclusive_scan(n, total);
  const int a1 = min(n, c0 + kListCap - f);
  for (int a = max(0, c0 - f); a < a1; ++a) list[f + a - c0] = ((uint32_t)(start + a) << 7) | code;
  return total;
}

// Adds x (in units of 1/scale kcal/mol/A) to an int64 fixed-point accumulator.
__device__ __forceinline__ void deposit(unsigned long long* a, double x) {
  atomicAdd(a, (unsigned long long)__double2ll_rn(x));
}

template <bool FP64, bool ENERGY>
__global__ __launch_bounds__(64 * kTileWaves) void k_lj_half(Views v, FFDev ff, LjPair<float> cf, LjPair<double> cd) {
  using PayT = std::conditional_t<FP64, Pay64, int4>;
  using P = std::conditional_t<FP64, double, float>;
  using Q = std::conditional_t<FP64, double, int>;
  constexpr int KMAX = FP64 ? 4 : 8;
  constexpr int LV = FP64 ? 2 : 3;
  __shared__ uint32_t list[kTileWaves][kListCap];
  __shared__ Shift<Q> shifts[kShiftSlots];
  __shared__ dd red[kTileWaves][3];

  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int ln = lane();
  const int per_xcd = (int)gridDim.x / kXcds;
  const int blk = ((int)blockIdx.x % kXcds) * per_xcd + (int)blockIdx.x / kXcds;
  if (blk >= v.n_lj_blocks) return;
  const BoxDev& B = v.boxes[v.lj_blk_box[blk]];
  const int lc = (blk - B.lj_blk_off) * kTileWaves + wave;
  const bool wact = lc < B.n_cells;
  const PayT* __restrict__ pay = static_cast<const PayT*>(v.payload);
  const int R = v.R, W = 2 * R + 1, ctr = (W * W * W - 1) / 2;
  load_shifts(v, v.lj_blk_box[blk], shifts);
  int total = 0, resident = 0;
  if (wact) total = __builtin_amdgcn_readfirstlane(fill_list_half(v, B, lc, 0, list[wave]));
  __syncthreads();

  double e = 0.0, es = 0.0, w = 0.0;
  if (wact) {
    const int hs = __builtin_amdgcn_readfirstlane(v.cell_start[B.cell_off + lc]);
    const int hn = __builtin_amdgcn_readfirstlane(v.cell_start[B.cell_off + lc + 1]) - hs;
    const Band bd = band_of(cf);
    // accumulator units per unit of the lane sums: mixed sums are in 2^25 (fixed-point) units
    const double scale = FP64 ? kHalfFix : kHalfFix * (double)kInvFixF;
    unsigned long long* __restrict__ acc = v.f_acc;
    const int64_t N = v.N;
    for (int g0 = 0; g0 < hn; g0 += KMAX) {
      const int kc = min(KMAX, hn - g0);
      Q hx[KMAX], hy[KMAX], hz[KMAX];
      int32_t lo[KMAX], hti[KMAX], hidx[KMAX];
      uint32_t span[KMAX];
      P ax[KMAX], ay[KMAX], az[KMAX];
#pragma unroll
      for (int k = 0; k < KMAX; ++k) {
        ax[k] = ay[k] = az[k] = (P)0;
        hx[k] = hy[k] = hz[k] = (Q)0;
        lo[k] = hti[k] = hidx[k] = 0;
        span[k] = 0xffffffffu;   // excludes every candidate
        if (k < kc) {
          const PayT q = pay[hs + g0 + k];
          hx[k] = q.x;
          hy[k] = q.y;
          hz[k] = q.z;
          const int32_t tag = pay_tag(q);
          const int32_t i = tag_index(tag);
          const int32_t c0 = chain_first(i, ff);
          hidx[k] = i;
          lo[k] = max(i - ff.excl, c0);
          span[k] = (uint32_t)(min(i + ff.excl, c0 + ff.chain_len - 1) - lo[k]);
          hti[k] = tag_type(tag);
        }
      }
      for (int c0 = 0; c0 < total; c0 += kListCap) {
        if (c0 != resident) {
          fill_list_half(v, B, lc, c0, list[wave]);
          resident = c0;
        }
        const int cn = min(kListCap, total - c0);
        for (int t0 = 0; t0 < cn; t0 += 64) {
          const bool act = t0 + ln < cn;
          Q jx = (Q)0, jy = (Q)0, jz = (Q)0;
          int32_t jt = 0;
          uint32_t ent = 0;
          if (act) {
            ent = list[wave][t0 + ln];
            const PayT q = pay[ent >> 7];
            const Shift<Q> sh = shifts[ent & 127];
            jt = pay_tag(q);
            jx = q.x + sh.x;
            jy = q.y + sh.y;
            jz = q.z + sh.z;
          }
          const int32_t jidx = tag_index(jt);
          const int jtype = tag_type(jt);
          // in-cell candidates (list positions [0, hn)) pair only with homes at lower positions
          const bool own_cell = c0 + t0 < hn;
          const int jpos = (int)(ent >> 7);
          P cx = (P)0, cy = (P)0, cz = (P)0;   // force on the candidate
#pragma unroll
          for (int k = 0; k < KMAX; ++k) {
            if (k < kc) {
              bool keep = act && (uint32_t)(jidx - lo[k]) > span[k];
              if (own_cell) keep = keep && ((int)(ent & 127) != ctr || jpos > hs + g0 + k);
              const int tt = ff.uniform_lj ? 0 : hti[k] * 2 + jtype;
              if constexpr (FP64) {
                const double dx = hx[k] - jx, dy = hy[k] - jy, dz = hz[k] - jz;
                const double r2 = dx * dx + dy * dy + dz * dz;
                if (keep && r2 < ff.rc2) {
                  const double r2i = 1.0 / r2;
                  const double r6 = r2i * r2i * r2i;
                  const double g = r6 * (pick(cd.f12, tt) * r6 - pick(cd.f6, tt));
                  const double ffs = g * r2i;
                  ax[k] += ffs * dx;
                  ay[k] += ffs * dy;
                  az[k] += ffs * dz;
                  cx -= ffs * dx;
                  cy -= ffs * dy;
                  cz -= ffs * dz;
                  if (ENERGY) {
                    const double en = r6 * (pick(cd.e12, tt) * r6 - pick(cd.e6, tt));
                    e += en;
                    es += en - pick(cd.ecut, tt);
                    w += g;
                  }
                }
              } else {
                const float dx = (float)(hx[k] - jx), dy = (float)(hy[k] - jy), dz = (float)(hz[k] - jz);
                const float r2s = r2_fix(dx, dy, dz);
                bool hit = keep && r2s < bd.hi;
                if (hit && r2s >= bd.lo) {
                  // rare: FP32 cannot tell the side of the cutoff; decide from the FP64 positions
                  double d[3], r2;
                  hit = inside_cutoff_f64(v.pos, N, B, hidx[k], jidx, ff.rc2, d, r2);
                }
                if (is_close(r2s, keep, bd)) {
                  // rare: a close contact, evaluated in FP64 and deposited on both atoms at once
                  double d[3], r2, fx = 0.0, fy = 0.0, fz = 0.0;
                  inside_cutoff_f64(v.pos, N, B, hidx[k], jidx, ff.rc2, d, r2);
                  add_close_pair<ENERGY>(d, r2, pick(cd.f12, tt), pick(cd.f6, tt), pick(cd.e12, tt),
                                         pick(cd.e6, tt), pick(cd.ecut, tt), fx, fy, fz, e, es, w);
                  deposit(acc + hidx[k], fx * kHalfFix);
                  deposit(acc + N + hidx[k], fy * kHalfFix);
                  deposit(acc + 2 * N + hidx[k], fz * kHalfFix);
                  deposit(acc + jidx, -fx * kHalfFix);
                  deposit(acc + N + jidx, -fy * kHalfFix);
                  deposit(acc + 2 * N + jidx, -fz * kHalfFix);
                  hit = false;
                }
                if (hit) {
                  const float r2 = r2s * kInvFix2F;
                  const float r2i = rcp_f(r2);
                  const float r6 = r2i * r2i * r2i;
                  const float g = r6 * (pick(cf.f12, tt) * r6 - pick(cf.f6, tt));
                  const float ffs = g * r2i;
                  ax[k] += ffs * dx;
                  ay[k] += ffs * dy;
                  az[k] += ffs * dz;
                  cx -= ffs * dx;
                  cy -= ffs * dy;
                  cz -= ffs * dz;
                  if (ENERGY) {
                    const float en = r6 * (pick(cf.e12, tt) * r6 - pick(cf.e6, tt));
                    e += (double)en;
                    es += (double)en - (double)pick(cf.ecut, tt);
                    w += (double)g;
                  }
                }
              }
            }
          }
          if (act && (cx != (P)0 || cy != (P)0 || cz != (P)0)) {
            deposit(acc + jidx, (double)cx * scale);
            deposit(acc + N + jidx, (double)cy * scale);
            deposit(acc + 2 * N + jidx, (double)cz * scale);
          }
        }
      }
      P sx, sy, sz;
      sum_homes<P, KMAX>(ln, ax, ay, az, sx, sy, sz);
      const int hk = ln >> (6 - LV);
      if ((ln & ((64 >> LV) - 1)) == 0 && hk < kc) {
        const int32_t i = tag_index(pay_tag(pay[hs + g0 + hk]));
        deposit(acc + i, (double)sx * scale);
        deposit(acc + N + i, (double)sy * scale);
        deposit(acc + 2 * N + i, (double)sz * scale);
      }
    }
  }
  // each pair counted once: the block sums halve, so pass twice the pair sums
  if (ENERGY) block_energy<kTileWaves>(2.0 * e, 2.0 * es, 2.0 * w, red, v.part_lj + (int64_t)blk * 3);
}

// Accumulators -> force array (FP32 or FP64), and back to zero for the next evaluation.
template <typename P>
__global__ __launch_bounds__(256) void k_half_finish(Views v) {
  const int64_t n3 = 3 * v.N;
  P* f = static_cast<P*>(v.f_lj);
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < n3; e += (int64_t)gridDim.x * 256) {
    const long long a = (long long)v.f_acc[e];
    f[e] = (P)((double)a * (1.0 / kHalfFix));
    v.f_acc[e] = 0ull;
  }
}

// ---------------------------------------------------------------------------------
// Neighbour-list mode (Sections 3.1-3.2: the paper's list, rebuilt every few steps).
//
// Build: one wave per home cell, exactly as the cell tile streams its candidates, but a
// pair closer than rc + skin (and not excluded) appends the candidate's list entry to the
// home atom's list instead of computing a force.  Lists are stored per 64 atoms of
// sorted order, entry-major ([nl_cap][64]), so that the force kernel's 64 lanes read 64
// consecutive words per step.
template <bool FP64, int KMAX>
__global__ __launch_bounds__(64 * kTileWaves) void k_nl_build(Views v, FFDev ff, const int32_t* __restrict__ gate) {
  if (gate && *gate == 0) return;   // no rebuild this step
  using PayT = std::conditional_t<FP64, Pay64, int4>;
  using Q = std::conditional_t<FP64, double, int>;
  __shared__ uint32_t list[kTileWaves][kListCap];
  __shared__ Shift<Q> shifts[kShiftSlots];

  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int ln = lane();
  const int per_xcd = (int)gridDim.x / kXcds;
  const int blk = ((int)blockIdx.x % kXcds) * per_xcd + (int)blockIdx.x / kXcds;
  if (blk >= v.n_cell_blocks) return;
  const BoxDev& B = v.boxes[v.cell_blk_box[blk]];
  const int lc = (blk - B.cell_blk_off) * kTileWaves + wave;
  const bool wact = lc < B.n_cells;
  const PayT* __restrict__ pay = static_cast<const PayT*>(v.payload);
  load_shifts(v, v.cell_blk_box[blk], shifts);
  int total = 0, resident = 0;
  if (wact) total = __builtin_amdgcn_readfirstlane(fill_list(v, B, lc, 0, list[wave]));
  __syncthreads();
  if (!wact) return;
  const int hs = __builtin_amdgcn_readfirstlane(v.cell_start[B.cell_off + lc]);
  const int hn = __builtin_amdgcn_readfirstlane(v.cell_start[B.cell_off + lc + 1]) - hs;
  // list radius in the payload's units, widened a little: the list may hold extra pairs,
  // never miss one
  const double rl2 = v.nl_rl2 * (1.0 + 1e-5);
  const float rl2s = (float)(rl2 * kFix * kFix);
  const int cap = v.nl_cap;
  for (int g0 = 0; g0 < hn; g0 += KMAX) {
    const int kc = min(KMAX, hn - g0);
    Q hx[KMAX], hy[KMAX], hz[KMAX];
    int32_t lo[KMAX], cnt[KMAX];
    uint32_t span[KMAX];
#pragma unroll
    for (int k = 0; k < KMAX; ++k) {
      cnt[k] = 0;
      if (k < kc) {
        const PayT q = pay[hs + g0 + k];
        hx[k] = uni(q.x);
        hy[k] = uni(q.y);
        hz[k] = uni(q.z);
        const int32_t i = tag_index(uni(pay_tag(q)));
        const int32_t c0 = chain_first(i, ff);
        lo[k] = max(i - ff.excl, c0);
        span[k] = (uint32_t)(min(i + ff.excl, c0 + ff.chain_len - 1) - lo[k]);
      } else {
        hx[k] = hy[k] = hz[k] = (Q)0;
        lo[k] = 0;
        span[k] = 0xffffffffu;
      }
    }
    for (int c0 = 0; c0 < total; c0 += kListCap) {
      if (c0 != resident) {
        fill_list(v, B, lc, c0, list[wave]);
        resident = c0;
      }
      const int cn = min(kListCap, total - c0);
      for (int t0 = 0; t0 < cn; t0 += 64) {
        const bool act = t0 + ln < cn;
        uint32_t ent = 0;
        Q jx = (Q)0, jy = (Q)0, jz = (Q)0;
        int32_t jt = 0;
        if (act) {
          ent = list[wave][t0 + ln];
          const PayT q = pay[ent >> 7];
          const Shift<Q> sh = shifts[ent & 127];
          jt = pay_tag(q);
          jx = q.x + sh.x;
          jy = q.y + sh.y;
          jz = q.z + sh.z;
        }
        const int32_t jidx = tag_index(jt);
#pragma unroll
        for (int k = 0; k < KMAX; ++k) {
          if (k < kc) {
            bool hit;
            if constexpr (FP64) {
              const double dx = hx[k] - jx, dy = hy[k] - jy, dz = hz[k] - jz;
              hit = dx * dx + dy * dy + dz * dz < rl2;
            } else {
              const float dx = (float)(hx[k] - jx), dy = (float)(hy[k] - jy), dz = (float)(hz[k] - jz);
              hit = r2_fix(dx, dy, dz) < rl2s;
            }
            hit = hit && act && (uint32_t)(jidx - lo[k]) > span[k];
            const uint64_t m = __builtin_amdgcn_ballot_w64(hit);
            const int at = cnt[k] + lanes_below(m);
            if (hit && at < cap) {
              const int ls = hs + g0 + k - B.atom_off;   // box-local sorted slot of the home
              v.nl_list[B.nl_off + (int64_t)(ls >> 6) * 64 * cap + (int64_t)at * 64 + (ls & 63)] = ent;
            }
            cnt[k] += __popcll(m);
          }
        }
      }
    }
    // the full count: above cap the force kernel walks this atom's stencil instead
#pragma unroll
    for (int k = 0; k < KMAX; ++k)
      if (k < kc && ln == 0) v.nl_count[hs + g0 + k] = cnt[k];
  }
}

// Build with per-cell lists: one wave per home cell streams its stencil as the cell tile
// does and keeps every candidate within rc + skin of ANY atom of the cell (the union of
// their Verlet spheres, in stencil order), so the force kernel can stream it exactly like
// the stencil (k_lj_tile): fewer candidates, the same coalesced loads.  Home atoms
// and excluded partners stay in the list (the force kernel tests exclusions per pair).
template <bool FP64>
__global__ __launch_bounds__(64 * kTileWaves) void k_nl_build_tile(Views v, FFDev ff, const int32_t* __restrict__ gate) {
  if (gate && *gate == 0) return;   // no rebuild this step
  using PayT = std::conditional_t<FP64, Pay64, int4>;
  using Q = std::conditional_t<FP64, double, int>;
  __shared__ uint32_t list[kTileWaves][kListCap];
  __shared__ Shift<Q> shifts[kShiftSlots];

  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int ln = lane();
  const int per_xcd = (int)gridDim.x / kXcds;
  const int blk = ((int)blockIdx.x % kXcds) * per_xcd + (int)blockIdx.x / kXcds;
  if (blk >= v.n_cell_blocks) return;
  const BoxDev& B = v.boxes[v.cell_blk_box[blk]];
  const int lc = (blk - B.cell_blk_off) * kTileWaves + wave;
  const bool wact = lc < B.n_cells;
  const PayT* __restrict__ pay = static_cast<const PayT*>(v.payload);
  load_shifts(v, v.cell_blk_box[blk], shifts);
  int total = 0, resident = 0;
  if (wact) total = __builtin_amdgcn_readfirstlane(fill_list(v, B, lc, 0, list[wave]));
  __syncthreads();
  if (!wact) return;
  const int hs = __builtin_amdgcn_readfirstlane(v.cell_start[B.cell_off + lc]);
  const int hn = __builtin_amdgcn_readfirstlane(v.cell_start[B.cell_off + lc + 1]) - hs;
  // list radius, widened a little: the list may hold extra pairs, never miss one
  const double rl2 = v.nl_rl2 * (1.0 + 1e-5);
  const float rl2s = (float)(rl2 * kFix * kFix);
  const int cap = v.nl_cap;
  uint32_t* __restrict__ out = v.nl_list + B.nl_off + (int64_t)lc * cap;
  constexpr int KB = FP64 ? 4 : 8;   // homes held in registers at a time
  int cnt = 0;
  for (int c0 = 0; c0 < total; c0 += kListCap) {
    if (c0 != resident) {
      fill_list(v, B, lc, c0, list[wave]);
      resident = c0;
    }
    const int cn = min(kListCap, total - c0);
    // bit s: the candidate of step s (list position c0 + 64 s + lane) is within reach of a home
    uint32_t hits = 0;
    for (int g0 = 0; g0 < hn; g0 += KB) {
      const int kc = min(KB, hn - g0);
      Q hx[KB], hy[KB], hz[KB];
#pragma unroll
      for (int k = 0; k < KB; ++k) {
        hx[k] = hy[k] = hz[k] = (Q)0;
        if (k < kc) {
          const PayT q = pay[hs + g0 + k];
          hx[k] = q.x;
          hy[k] = q.y;
          hz[k] = q.z;
        }
      }
      for (int t0 = 0, s = 0; t0 < cn; t0 += 64, ++s) {
        if (t0 + ln >= cn) continue;
        const uint32_t ent = list[wave][t0 + ln];
        const PayT q = pay[ent >> 7];
        const Shift<Q> sh = shifts[ent & 127];
        const Q jx = q.x + sh.x, jy = q.y + sh.y, jz = q.z + sh.z;
        bool hit = false;
#pragma unroll
        for (int k = 0; k < KB; ++k) {
          if (k < kc) {
            if constexpr (FP64) {
              const double dx = hx[k] - jx, dy = hy[k] - jy, dz = hz[k] - jz;
              hit = hit || dx * dx + dy * dy + dz * dz < rl2;
            } else {
              hit = hit || r2_fix((float)(hx[k] - jx), (float)(hy[k] - jy), (float)(hz[k] - jz)) < rl2s;
            }
          }
        }
        if (hit) hits |= 1u << s;
      }
    }
    // compaction in list order
    for (int t0 = 0, s = 0; t0 < cn; t0 += 64, ++s) {
      const bool hit = (hits >> s) & 1u;
      const uint64_t m = __builtin_amdgcn_ballot_w64(hit);
      const int at = cnt + lanes_below(m);
      if (hit && at < cap) out[at] = list[wave][t0 + ln];
      cnt += __popcll(m);
    }
  }
  // the full count: above cap the force kernel streams this cell's stencil instead
  if (ln == 0) v.nl_count[B.cell_off + lc] = cnt;
}

// LJ force from the lists: one lane per atom of sorted order, walking its list; the
// candidate comes from the current payload plus the stencil shift recorded at the
// build.  Mixed form: FP32 on exact int32 differences, with the cutoff band decided in
// FP64 (inline: about one list entry in 10^6).
template <bool FP64, bool ENERGY, bool UNI>
__global__ __launch_bounds__(kLjNlBlock) void k_lj_nl(Views v, FFDev ff, LjPair<float> cf, LjPair<double> cd,
                                                    const void* payv) {
  using PayT = std::conditional_t<FP64, Pay64, int4>;
  using P = std::conditional_t<FP64, double, float>;
  using Q = std::conditional_t<FP64, double, int>;
  __shared__ Shift<Q> shifts[kShiftSlots];
  __shared__ dd red[kLjNlBlock / 64][3];
  const BoxDev& B = v.boxes[v.lj_blk_box[blockIdx.x]];
  const int local = ((int)blockIdx.x - B.lj_blk_off) * kLjNlBlock + (int)threadIdx.x;
  load_shifts(v, v.lj_blk_box[blockIdx.x], shifts);
  __syncthreads();
  double e = 0.0, es = 0.0, w = 0.0;
  if (local < B.n_atoms) {
    const PayT* __restrict__ pay = static_cast<const PayT*>(payv);
    const int32_t s = B.atom_off + local;
    const PayT hq = pay[s];
    const int32_t i = tag_index(pay_tag(hq));
    const int ti = tag_type(pay_tag(hq));
    const int n = v.nl_count[s];
    const uint32_t* __restrict__ row =
        v.nl_list + B.nl_off + (int64_t)(local >> 6) * 64 * v.nl_cap + (local & 63);
    const Band bd = band_of(cf);
    const float f12_fold = cf.f12[0] / cf.f6[0];
    // kNlSums interleaved partial sums: shorter FP32 summation chains, and that many list
    // entries in flight per lane
    constexpr int kNlSums = FP64 ? 4 : 8;
    P ax[kNlSums], ay[kNlSums], az[kNlSums];
#pragma unroll
    for (int u = 0; u < kNlSums; ++u) ax[u] = ay[u] = az[u] = (P)0;
    double cx = 0.0, cy = 0.0, cz = 0.0;   // close contacts (mixed), FP64
    int32_t bmax = 0;
    // one candidate (payload q at stencil shift sh) into partial sum u
    auto one = [&](const PayT& q, const Shift<Q>& sh, bool keep, int u) {
      const int32_t tj = pay_tag(q);
      const int tt = UNI ? 0 : ti * 2 + tag_type(tj);
      if constexpr (FP64) {
        pair_f64<ENERGY>(hq.x - (q.x + sh.x), hq.y - (q.y + sh.y), hq.z - (q.z + sh.z), keep, ff.rc2,
                         pick(cd.f12, tt), pick(cd.f6, tt), pick(cd.e12, tt), pick(cd.e6, tt), pick(cd.ecut, tt),
                         ax[u], ay[u], az[u], e, es, w);
      } else {
        const int dqx = hq.x - (q.x + sh.x), dqy = hq.y - (q.y + sh.y), dqz = hq.z - (q.z + sh.z);
        bool near = false;
        const float r2s = pair_fix<ENERGY, UNI>(dqx, dqy, dqz, keep, bd, UNI ? f12_fold : pick(cf.f12, tt),
                                                       pick(cf.f6, tt), pick(cf.e12, tt), pick(cf.e6, tt),
                                                       pick(cf.ecut, tt), ax[u], ay[u], az[u], e, es, w, bmax, near);
        double d[3], r2;
        if (near) {   // rare: a close contact, in FP64
          inside_cutoff_f64(v.pos, v.N, B, i, tag_index(tj), ff.rc2, d, r2);
          add_close_pair<ENERGY>(d, r2, pick(cd.f12, tt), pick(cd.f6, tt), pick(cd.e12, tt), pick(cd.e6, tt),
                                 pick(cd.ecut, tt), cx, cy, cz, e, es, w);
        }
        if (in_band(r2s, keep, bd) && !inside_cutoff_f64(v.pos, v.N, B, i, tag_index(tj), ff.rc2, d, r2)) {
          // counted above as inside; in the folded form the sums are divided by f6
          float bx = 0.0f, by = 0.0f, bz = 0.0f;
          remove_band_pair<ENERGY>(d, r2, pick(cf.f12, tt), pick(cf.f6, tt), pick(cf.e12, tt), pick(cf.e6, tt),
                                   pick(cf.ecut, tt), bx, by, bz, e, es, w);
          const float sc = UNI ? 1.0f / cf.f6[0] : 1.0f;
          ax[u] += bx * sc;
          ay[u] += by * sc;
          az[u] += bz * sc;
        }
      }
    };
    if (n <= v.nl_cap) {
      for (int t0 = 0; t0 < n; t0 += kNlSums) {
#pragma unroll
        for (int u = 0; u < kNlSums; ++u) {
          const int t = t0 + u;
          if (t < n) {
            const uint32_t ent = row[(int64_t)t * 64];
            one(pay[ent >> 7], shifts[ent & 127], true, u);
          }
        }
      }
    } else {
      // the list outgrew its capacity: walk the stencil of the build's bins (every atom has moved
      // less than half the skin since, and the stencil covers rc + skin), excluding 1-2/1-3 here
      const int32_t c0 = chain_first(i, ff);
      const int32_t lo = max(i - ff.excl, c0);
      const uint32_t span = (uint32_t)(min(i + ff.excl, c0 + ff.chain_len - 1) - lo);
      const int R = v.R, W = 2 * R + 1;
      const Cell3 k3 = cell_coords(v.scell[s] - B.cell_off, B);
      for (int code = 0; code < W * W * W; ++code) {
        const Cell3 o = stencil_offset(code, R);
        int nx = k3.x + o.x, ny = k3.y + o.y, nz = k3.z + o.z;
        nx += nx < 0 ? B.M[0] : 0;
        nx -= nx >= B.M[0] ? B.M[0] : 0;
        ny += ny < 0 ? B.M[1] : 0;
        ny -= ny >= B.M[1] ? B.M[1] : 0;
        nz += nz < 0 ? B.M[2] : 0;
        nz -= nz >= B.M[2] ? B.M[2] : 0;
        const int c = B.cell_off + nx + B.M[0] * (ny + B.M[1] * nz);
        for (int t = v.cell_start[c]; t < v.cell_start[c + 1]; ++t) {
          const PayT q = pay[t];
          one(q, shifts[code], (uint32_t)(tag_index(pay_tag(q)) - lo) > span, 0);
        }
      }
    }
    for (int h = kNlSums / 2; h > 0; h >>= 1)   // pairwise
#pragma unroll
      for (int u = 0; u < h; ++u) {
        ax[u] += ax[u + h];
        ay[u] += ay[u + h];
        az[u] += az[u + h];
      }
    P fx = ax[0], fy = ay[0], fz = az[0];
    if constexpr (!FP64) {
      const float sc = UNI ? kInvFixF * cf.f6[0] : kInvFixF;
      fx = (float)((double)(fx * sc) + cx);
      fy = (float)((double)(fy * sc) + cy);
      fz = (float)((double)(fz * sc) + cz);
    }
    P* f = static_cast<P*>(v.f_lj);
    f[i] = fx;
    f[v.N + i] = fy;
    f[2 * v.N + i] = fz;
  }
  if (ENERGY) block_energy<kLjNlBlock / 64>(e, es, w, red, v.part_lj + (int64_t)blockIdx.x * 3);
}

template <bool FP64, bool ENERGY, int K>
void launch_tile_k(const Views& v, const FFDev& ff, const LjPair<float>& cf, const LjPair<double>& cd, hipStream_t s) {
  const dim3 g((v.n_lj_blocks + kXcds - 1) / kXcds * kXcds), b(64 * kTileWaves);
  if (ff.uniform_lj) hipLaunchKernelGGL((k_lj_tile<FP64, ENERGY, true, K>), g, b, 0, s, v, ff, cf, cd);
  else hipLaunchKernelGGL((k_lj_tile<FP64, ENERGY, false, K>), g, b, 0, s, v, ff, cf, cd);
}

// homes: home atoms per pass of a wave (4, 8 or 16; the FP64 form holds 4 in scalar registers).
template <bool FP64, bool ENERGY>
void launch_tile(const Views& v, const FFDev& ff, const LjPair<float>& cf, const LjPair<double>& cd, int homes,
                 hipStream_t s) {
  if constexpr (FP64) {
    launch_tile_k<FP64, ENERGY, 4>(v, ff, cf, cd, s);
  } else {
    if (homes == 4) launch_tile_k<FP64, ENERGY, 4>(v, ff, cf, cd, s);
    else if (homes == 16) launch_tile_k<FP64, ENERGY, 16>(v, ff, cf, cd, s);
    else launch_tile_k<FP64, ENERGY, 8>(v, ff, cf, cd, s);
  }
}

template <bool ENERGY, int K>
void launch_cell_k(const Views& v, const FFDev& ff, const LjPair<float>& cf, const LjPair<double>& cd,
                   bool branchless, hipStream_t s) {
  const dim3 g((v.n_lj_blocks + kXcds - 1) / kXcds * kXcds), b(64);
  if (ff.uniform_lj) {
    if (branchless) hipLaunchKernelGGL((k_lj_cell<ENERGY, true, K, true>), g, b, 0, s, v, ff, cf, cd);
    else hipLaunchKernelGGL((k_lj_cell<ENERGY, true, K, false>), g, b, 0, s, v, ff, cf, cd);
  } else {
    hipLaunchKernelGGL((k_lj_cell<ENERGY, false, K, false>), g, b, 0, s, v, ff, cf, cd);
  }
}

template <bool ENERGY>
void launch_cell(const Views& v, const FFDev& ff, const LjPair<float>& cf, const LjPair<double>& cd, bool branchless,
                 int homes, hipStream_t s) {
  if (homes == 4) launch_cell_k<ENERGY, 4>(v, ff, cf, cd, branchless, s);
  else if (homes == 16) launch_cell_k<ENERGY, 16>(v, ff, cf, cd, branchless, s);
  else launch_cell_k<ENERGY, 8>(v, ff, cf, cd, branchless, s);
}

}  // namespace

int64_t lj_blocks_for_box(int kernel, int64_t n_atoms, int64_t n_cells) {
  if (kernel == 4) return (n_atoms + kLjNlBlock - 1) / kLjNlBlock;
  return (n_cells + kTileWaves - 1) / kTileWaves;
}

void launch_nl_build(const Views& v, const FFDev& ff, bool fp32, int kernel, hipStream_t s, const int32_t* gate) {
  dim3 g((v.n_cell_blocks + kXcds - 1) / kXcds * kXcds), b(64 * kTileWaves);
  if (kernel == 5) {
    if (fp32)
      hipLaunchKernelGGL((k_nl_build_tile<false>), g, b, 0, s, v, ff, gate);
    else
      hipLaunchKernelGGL((k_nl_build_tile<true>), g, b, 0, s, v, ff, gate);
    return;
  }
  if (fp32)
    hipLaunchKernelGGL((k_nl_build<false, kTileHomesMixed>), g, b, 0, s, v, ff, gate);
  else
    hipLaunchKernelGGL((k_nl_build<true, 4>), g, b, 0, s, v, ff, gate);
}

// Neighbour-list forces always read the current payload (the build's right after a rebuild).
void launch_lj_nl(const Views& v, const FFDev& ff, bool fp32, int kernel, bool energy, int homes, hipStream_t s) {
  const LjPair<float> cf = make_pair<float>(ff);
  const LjPair<double> cd = make_pair<double>(ff);
  const void* pay = v.pay_cur;
  if (kernel == 5) {   // per-cell lists through the cell tile, reading the current payload
    Views w = v;
    w.payload = const_cast<void*>(pay);
    if (fp32) {
      if (energy) launch_tile<false, true>(w, ff, cf, cd, homes, s);
      else launch_tile<false, false>(w, ff, cf, cd, homes, s);
    } else {
      if (energy) launch_tile<true, true>(w, ff, cf, cd, homes, s);
      else launch_tile<true, false>(w, ff, cf, cd, homes, s);
    }
    return;
  }
  dim3 g(v.n_lj_blocks), b(kLjNlBlock);
#define MDK_NL(F64, E, U) hipLaunchKernelGGL((k_lj_nl<F64, E, U>), g, b, 0, s, v, ff, cf, cd, pay)
  if (fp32) {
    if (ff.uniform_lj) { if (energy) MDK_NL(false, true, true); else MDK_NL(false, false, true); }
    else { if (energy) MDK_NL(false, true, false); else MDK_NL(false, false, false); }
  } else {
    if (ff.uniform_lj) { if (energy) MDK_NL(true, true, true); else MDK_NL(true, false, true); }
    else { if (energy) MDK_NL(true, true, false); else MDK_NL(true, false, false); }
  }
#undef MDK_NL
}

void launch_lj(const Views& v, const FFDev& ff, bool fp32, int kernel, bool energy, int homes, hipStream_t s) {
  const LjPair<float> cf = make_pair<float>(ff);
  const LjPair<double> cd = make_pair<double>(ff);
  if (kernel == 6) {
    dim3 g((v.n_lj_blocks + kXcds - 1) / kXcds * kXcds), b(64 * kTileWaves);
    if (fp32) {
      if (energy) hipLaunchKernelGGL((k_lj_half<false, true>), g, b, 0, s, v, ff, cf, cd);
      else hipLaunchKernelGGL((k_lj_half<false, false>), g, b, 0, s, v, ff, cf, cd);
    } else {
      if (energy) hipLaunchKernelGGL((k_lj_half<true, true>), g, b, 0, s, v, ff, cf, cd);
      else hipLaunchKernelGGL((k_lj_half<true, false>), g, b, 0, s, v, ff, cf, cd);
    }
    const int fg = (int)std::min<int64_t>((3 * v.N + 255) / 256, 4096);
    if (fp32) hipLaunchKernelGGL(k_half_finish<float>, dim3(fg), dim3(256), 0, s, v);
    else hipLaunchKernelGGL(k_half_finish<double>, dim3(fg), dim3(256), 0, s, v);
    return;
  }
  const bool nb = kernel == 3;   // (FP64 goes to the group kernel)
  if (energy) launch_cell<true>(v, ff, cf, cd, nb, homes, s);
  else launch_cell<false>(v, ff, cf, cd, nb, homes, s);
}

}  // namespace mdk
