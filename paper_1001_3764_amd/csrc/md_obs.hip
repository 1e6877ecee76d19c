// Structural observables of Section 5 for gfx950: the pair-distance histogram behind the
// radial distribution function (Fig. 10), the dihedral-angle distribution and trans /
// gauche fractions (Figs. 9, 15), and per-chain radius of gyration and end-to-end vector
// (Figs. 8, 12).
//
//   k_obs_pairs      one wavefront per cell: its atoms against the forward half of the current
//                    grid's stencil (with at least 2R + 1 cells per dimension no pair of cells is
//                    reached from both sides), so every unordered non-excluded pair is counted
//                    once; the bin is decided in FP64 on r^2 against squared edges, so the
//                    counts are exact integers; a block histogram in LDS (integer atomics: the
//                    counts do not depend on their order), one row of block partials per block
//   k_obs_dihedrals  one lane per dihedral: the IUPAC angle, its bin and its class
//   k_obs_reduce     per bin, the block partials in block order (64-bit)
//   k_obs_chains     one wavefront per chain: the chain unwrapped bond by bond (a wave
//                    prefix sum per 64 atoms), centre of mass, then R_g^2 and R_ee
//   k_ree,           the end-to-end vector autocorrelation (Fig. 8): each chain's R_ee
//   k_ree_reduce     against the one stored at the reference time, summed per box
#include "md_internal.h"

namespace mdk {
namespace {

__device__ inline int lane() { return (int)(threadIdx.x & 63); }

// minimum image of one coordinate difference, no fused multiply-add
__device__ inline double mi_rn(double t, double L, double invL) {
  return __dadd_rn(t, -__dmul_rn(L, rint(__dmul_rn(t, invL))));
}

// The largest k < n_bins with edge2[k] <= r2 (r2 below edge2[n_bins]; edge2[k] = (k dr)^2): a guess
// from FP32 (rarely off, and then by one bin for any but absurdly small distances), then the
// exact comparison.
__device__ inline int distance_bin(double r2, float inv_dr, const double* edge2, int n_bins) {
  int k = min((int)(__builtin_amdgcn_sqrtf((float)r2) * inv_dr), n_bins - 1);
  const double lo = edge2[k], hi = edge2[k + 1];
  if (r2 < lo || r2 >= hi) {
    while (k > 0 && r2 < edge2[k]) --k;
    while (k + 1 < n_bins && r2 >= edge2[k + 1]) ++k;
  }
  return k;
}

// Exclusive prefix sum over the wave.
__device__ inline int wave_scan(int x, int& total) {
  const int ln = lane();
  int s = x;
  for (int d = 1; d < 64; d <<= 1) {
    const int y = __shfl_up(s, d);
    if (ln >= d) s += y;
  }
  total = __builtin_amdgcn_readlane(s, 63);
  return s - x;
}

// LDS is shared within one wavefront here, which executes its LDS accesses in order: only the
// compiler has to keep them so.
__device__ __forceinline__ void lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

struct alignas(16) ObsAtom {
  double x, y, z;
  int32_t idx, flat;   // atom; its place in the wave's candidate list (homes: in the cell)
};

// One wavefront per home cell (grid stride).  The candidates of a cell are its own atoms, then
// the forward half of the stencil: the cells after it in its row, the rows after it in its layer
// and the layers after it, each row one or two contiguous runs of the cell lists.  64 of them at a
// time go to LDS with their FP64 positions (read once per cell, where a lane per atom read
// them once per pair), and the lanes take the home-candidate pairs 64 at a time.  The
// minimum image is evaluated only where some difference of the wave's pairs reaches 0.499 L (below
// that it is the difference itself).  Bound: LDS (the pairs' operands, the edges and the histogram's
// atomics) and FP64 issue, about equally.  300,000 atoms, 210 bins, R = 2: 1,200 us with a lane per
// atom, 245 us here (12 waves per block; 8, 10 and 16: 275, 270, 310).
constexpr int kObsWaves = 12;
__global__ __launch_bounds__(64 * kObsWaves) void k_obs_pairs(Views v, int b, int chain_len, int excl, double dr,
                                                            int n_bins, uint32_t* part) {
  extern __shared__ double obs_lds[];   // edge2[n_bins + 1], hist[n_bins]
  double* const edge2 = obs_lds;
  uint32_t* const hist = (uint32_t*)(obs_lds + n_bins + 1);
  __shared__ ObsAtom cands[kObsWaves][64], homes_[kObsWaves][64];
  __shared__ int2 window_[kObsWaves][64];
  __shared__ int32_t runs[kObsWaves][64];
  __shared__ unsigned long long marks[kObsWaves][64];
  for (int k = (int)threadIdx.x; k <= n_bins; k += 64 * kObsWaves) {
    if (k < n_bins) hist[k] = 0;
    edge2[k] = __dmul_rn(__dmul_rn((double)k, dr), __dmul_rn((double)k, dr));
  }
  __syncthreads();
  const BoxDev& B = v.boxes[b];
  const double rmax2 = __dmul_rn(__dmul_rn((double)n_bins, dr), __dmul_rn((double)n_bins, dr));
  const float inv_dr = (float)(1.0 / dr);
  const int64_t N = v.N;
  const int R = v.R, W = 2 * R + 1;
  const int M0 = B.M[0], M1 = B.M[1], M2 = B.M[2];
  const int ln = lane(), wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  ObsAtom* const cand = cands[wave];
  ObsAtom* const homes = homes_[wave];
  int2* const window = window_[wave];
  const double hx = 0.499 * B.L[0], hy = 0.499 * B.L[1], hz = 0.499 * B.L[2];
  // this lane's run: 0 the home cell, 1 and 2 the rest of its row, then two per forward row (the
  // part inside the box and the part wrapped around it); 3 + 2 (R + R W) <= 51 lanes
  const int fr = ln < 3 ? 0 : (ln - 3) / 2, wrapped = ln < 3 ? ln == 2 : (ln - 3) & 1;
  const int oy = ln < 3 ? 0 : (fr < R ? fr + 1 : (fr - R) % W - R), oz = ln < 3 || fr < R ? 0 : (fr - R) / W + 1;
  const bool used = ln < 3 + 2 * (R + R * W);
  for (int lc = (int)blockIdx.x * kObsWaves + wave; lc < B.n_cells; lc += (int)gridDim.x * kObsWaves) {
    const int hs = v.cell_start[B.cell_off + lc], hn = v.cell_start[B.cell_off + lc + 1] - hs;
    if (hn == 0) continue;
    const Cell3 k3 = cell_coords(lc, B);
    int n = 0, start = 0;
    if (used) {
      int ny = k3.y + oy, nz = k3.z + oz;
      ny += ny < 0 ? M1 : 0;
      ny -= ny >= M1 ? M1 : 0;
      nz -= nz >= M2 ? M2 : 0;
      const int row = B.cell_off + M0 * (ny + M1 * nz);
      int lo = ln < 3 ? k3.x + 1 : k3.x - R, hi = k3.x + R;   // unwrapped cells of the run's row
      if (ln == 0) lo = hi = k3.x;
      int a = max(lo, 0), z = min(hi, M0 - 1);
      if (wrapped) {   // (M0 >= W: at most one side leaves the box)
        a = lo < 0 ? lo + M0 : max(lo - M0, 0);
        z = lo < 0 ? M0 - 1 : hi - M0;
      }
      if (a <= z) {
        start = v.cell_start[row + a];
        n = v.cell_start[row + z + 1] - start;
      }
    }
    int total;
    const int f = wave_scan(n, total);
    const uint64_t some = __builtin_amdgcn_ballot_w64(n > 0);
    if (n > 0) runs[wave][__popcll(some & ((1ull << ln) - 1ull))] = start - f;
    const int mark = n > 0 ? f - 1 : -1;   // a run (but the first) marks the position before it
    for (int g0 = 0; g0 < hn; g0 += 64) {
      const int hc = min(64, hn - g0);
      const float inv_hc = __builtin_amdgcn_rcpf((float)hc);
      if (ln < hc) {
        const int32_t i = v.cell_atoms[hs + g0 + ln];
        homes[ln] = ObsAtom{v.pos[i], v.pos[N + i], v.pos[2 * N + i], i, g0 + ln};
        const int32_t c0 = i - i % chain_len;
        const int32_t lo = max(i - excl, c0);
        window[ln] = make_int2(lo, min(i + excl, c0 + chain_len - 1) - lo);
      }
      for (int t0 = 0; t0 < total; t0 += 64 * 64) {
        marks[wave][ln] = 0ull;
        lds_order();
        const int at = mark - t0;
        if (mark >= 0 && at >= 0 && at < 64 * 64) atomicOr(&marks[wave][at >> 6], 1ull << (at & 63));
        lds_order();
        const unsigned long long mk = marks[wave][ln];
        const int end = min(total, t0 + 64 * 64);
        for (int w0 = t0; w0 < end; w0 += 64) {
          const int win = (w0 - t0) >> 6;
          const int before = __popcll(__builtin_amdgcn_ballot_w64(mark >= 0 && mark < w0));
          const int ml = __builtin_amdgcn_readlane((int)(uint32_t)mk, win);
          const int mh = __builtin_amdgcn_readlane((int)(uint32_t)(mk >> 32), win);
          const int r = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)mh, __builtin_amdgcn_mbcnt_lo((uint32_t)ml, (uint32_t)before));
          const int t = w0 + ln;
          if (t < end) {
            const int32_t j = v.cell_atoms[t + runs[wave][r]];
            cand[ln] = ObsAtom{v.pos[j], v.pos[N + j], v.pos[2 * N + j], j, t};
          }
          lds_order();
          const int wc = min(64, end - w0);
          // all pairs (candidate p / hc, home p % hc), 64 at a time: p < 4096, so the FP32 quotient
          // is exact
          for (int p0 = 0; p0 < hc * wc; p0 += 64) {
            const int p = min(p0 + ln, hc * wc - 1);
            const int c = (int)(((float)p + 0.5f) * inv_hc);
            const ObsAtom h = homes[p - c * hc], q = cand[c];
            const int2 ex = window[p - c * hc];
            // of two atoms of the home cell, the later one is the candidate
            const bool on = p0 + ln < hc * wc && (q.flat >= hn || q.flat > h.flat) &&
                            (uint32_t)(q.idx - ex.x) > (uint32_t)ex.y;
            double dx = __dadd_rn(h.x, -q.x), dy = __dadd_rn(h.y, -q.y), dz = __dadd_rn(h.z, -q.z);
            if (__builtin_amdgcn_ballot_w64(fabs(dx) > hx || fabs(dy) > hy || fabs(dz) > hz) != 0) {
              dx = mi_rn(dx, B.L[0], B.invL[0]);
              dy = mi_rn(dy, B.L[1], B.invL[1]);
              dz = mi_rn(dz, B.L[2], B.invL[2]);
            }
            const double r2 = __dadd_rn(__dadd_rn(__dmul_rn(dx, dx), __dmul_rn(dy, dy)), __dmul_rn(dz, dz));
            if (on && r2 < rmax2) atomicAdd(&hist[distance_bin(r2, inv_dr, edge2, n_bins)], 1u);
          }
          lds_order();
        }
      }
    }
  }
  __syncthreads();
  for (int k = (int)threadIdx.x; k < n_bins; k += 64 * kObsWaves) part[(int64_t)blockIdx.x * kMaxObsBins + k] = hist[k];
}

// IUPAC dihedral angle of sites (p, p+1, p+2, p+3), bonds minimum-imaged
__device__ inline double dihedral_phi(const Views& v, const BoxDev& B, int64_t p) {
  const int64_t N = v.N;
  double s[4][3];
  for (int q = 0; q < 3; ++q) s[0][q] = v.pos[q * N + p];
  for (int a = 1; a < 4; ++a)
    for (int q = 0; q < 3; ++q)
      s[a][q] = s[a - 1][q] + mi_rn(v.pos[q * N + p + a] - v.pos[q * N + p + a - 1], B.L[q], B.invL[q]);
  double F[3], G[3], H[3];
  for (int q = 0; q < 3; ++q) {
    F[q] = s[0][q] - s[1][q];
    G[q] = s[1][q] - s[2][q];
    H[q] = s[3][q] - s[2][q];
  }
  const double A[3] = {F[1] * G[2] - F[2] * G[1], F[2] * G[0] - F[0] * G[2], F[0] * G[1] - F[1] * G[0]};
  const double Bv[3] = {H[1] * G[2] - H[2] * G[1], H[2] * G[0] - H[0] * G[2], H[0] * G[1] - H[1] * G[0]};
  const double BA[3] = {Bv[1] * A[2] - Bv[2] * A[1], Bv[2] * A[0] - Bv[0] * A[2], Bv[0] * A[1] - Bv[1] * A[0]};
  const double lA = sqrt(A[0] * A[0] + A[1] * A[1] + A[2] * A[2]);
  const double lB = sqrt(Bv[0] * Bv[0] + Bv[1] * Bv[1] + Bv[2] * Bv[2]);
  const double lG = sqrt(G[0] * G[0] + G[1] * G[1] + G[2] * G[2]);
  const double c = (A[0] * Bv[0] + A[1] * Bv[1] + A[2] * Bv[2]) / (lA * lB);
  const double sn = (BA[0] * G[0] + BA[1] * G[1] + BA[2] * G[2]) / (lA * lB * lG);
  return atan2(sn, c);
}

// bins [0, n_bins): the angle histogram; n_bins, n_bins + 1, n_bins + 2: trans, gauche+, gauche-
__global__ __launch_bounds__(kAtomBlock) void k_obs_dihedrals(Views v, int b, int chain_len, int n_bins,
                                                            uint32_t* part) {
  __shared__ uint32_t hist[kMaxObsBins];
  const int nb = n_bins + 3;
  for (int k = (int)threadIdx.x; k < nb; k += kAtomBlock) hist[k] = 0;
  __syncthreads();
  const BoxDev& B = v.boxes[b];
  const double pi = 3.141592653589793, two_pi = 2.0 * pi, third = two_pi / 3.0, scale = n_bins / two_pi;
  for (int64_t t = (int64_t)blockIdx.x * kAtomBlock + threadIdx.x; t < B.n_atoms; t += (int64_t)gridDim.x * kAtomBlock) {
    if (t % chain_len + 3 >= chain_len) continue;
    const double phi = dihedral_phi(v, B, B.atom_off + t);
    if (n_bins > 0) {
      int k = (int)floor((phi + pi) * scale);
      k = k > n_bins - 1 ? n_bins - 1 : (k < 0 ? 0 : k);
      atomicAdd(&hist[k], 1u);
    }
    atomicAdd(&hist[n_bins + (fabs(phi) > third ? 0 : (phi >= 0.0 ? 1 : 2))], 1u);
  }
  __syncthreads();
  for (int k = (int)threadIdx.x; k < nb; k += kAtomBlock) part[(int64_t)blockIdx.x * kMaxObsBins + k] = hist[k];
}

// 64 bins per block: wave w adds the rows w, w + 16, ... of its bins (their loads in flight
// together), then the waves in order.  One thread per bin adding 512 rows one after the other took
// 114 us for 210 bins.
constexpr int kObsReduceWaves = 16;
__global__ __launch_bounds__(64 * kObsReduceWaves) void k_obs_reduce(const uint32_t* part, int n_blocks, int n_bins,
                                                                   unsigned long long* out) {
  __shared__ unsigned long long sh[kObsReduceWaves][64];
  const int w = (int)threadIdx.x >> 6;
  const int k = (int)blockIdx.x * 64 + lane();
  unsigned long long s = 0;
  if (k < n_bins) {
#pragma unroll 8
    for (int q = w; q < n_blocks; q += kObsReduceWaves) s += part[(int64_t)q * kMaxObsBins + k];
  }
  sh[w][lane()] = s;
  __syncthreads();
  if (w != 0 || k >= n_bins) return;
  for (int u = 1; u < kObsReduceWaves; ++u) s += sh[u][lane()];
  out[k] = s;
}

__device__ inline double wave_sum(double x) {
  for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off);
  return x;
}

__device__ inline double wave_inclusive_scan(double x) {
  const int ln = lane();
  for (int d = 1; d < 64; d <<= 1) {
    const double y = __shfl_up(x, d);
    if (ln >= d) x += y;
  }
  return x;
}

// One wavefront per chain of box b.  Pass 1: unwrapped positions u_p = x_0 + sum of the
// minimum-imaged bonds up to p, mass-weighted sums; pass 2: sum m |u - u_cm|^2.
__global__ __launch_bounds__(256) void k_obs_chains(Views v, FFDev ff, int b, int chain_len, double* out) {
  const BoxDev& B = v.boxes[b];
  const int n_chains = B.n_atoms / chain_len;
  const int ch = (int)((blockIdx.x * blockDim.x + threadIdx.x) >> 6);
  if (ch >= n_chains) return;
  const int ln = lane();
  const int64_t N = v.N;
  const int64_t a0 = (int64_t)B.atom_off + (int64_t)ch * chain_len;
  double x0[3];
  for (int q = 0; q < 3; ++q) x0[q] = v.pos[q * N + a0];
  double cm[3] = {0.0, 0.0, 0.0}, msum = 0.0, rg = 0.0, ree[3] = {0.0, 0.0, 0.0};
  for (int pass = 0; pass < 2; ++pass) {
    double carry[3] = {0.0, 0.0, 0.0};
    double acc[3] = {0.0, 0.0, 0.0}, macc = 0.0, racc = 0.0;
    for (int p0 = 0; p0 < chain_len; p0 += 64) {
      const int p = p0 + ln;
      const bool in = p < chain_len;
      double u[3];
      for (int q = 0; q < 3; ++q) {
        double d = 0.0;
        if (in && p > 0) d = mi_rn(v.pos[q * N + a0 + p] - v.pos[q * N + a0 + p - 1], B.L[q], B.invL[q]);
        const double sc = wave_inclusive_scan(d);
        u[q] = x0[q] + (carry[q] + sc);
        carry[q] += __shfl(sc, 63);
      }
      if (in) {
        const double m = ff.mass[v.type[a0 + p]];
        if (pass == 0) {
          macc += m;
          for (int q = 0; q < 3; ++q) acc[q] += m * u[q];
        } else {
          double d2 = 0.0;
          for (int q = 0; q < 3; ++q) d2 += (u[q] - cm[q]) * (u[q] - cm[q]);
          racc += m * d2;
        }
      }
    }
    if (pass == 0) {
      msum = wave_sum(macc);
      for (int q = 0; q < 3; ++q) {
        cm[q] = wave_sum(acc[q]) / msum;
        ree[q] = carry[q];
      }
    } else {
      rg = wave_sum(racc) / msum;
    }
  }
  if (ln == 0) {
    const int64_t c = (int64_t)B.atom_off / chain_len + ch;
    out[4 * c] = rg;
    for (int q = 0; q < 3; ++q) out[4 * c + 1 + q] = ree[q];
  }
}

// End-to-end vector autocorrelation (Fig. 8).  One wavefront per chain of box b: R, the sum
// of the chain's minimum-imaged bonds (each lane sums every 64th bond, then a fixed-order wave
// sum).  REF: store R as the reference ree0[c]; otherwise write the chain's terms
// part[2 c] = R . ree0[c] and part[2 c + 1] = |ree0[c]|^2.
template <bool REF>
__global__ __launch_bounds__(256) void k_ree(Views v, int b, int chain_len, double* ree0, double* part) {
  const BoxDev& B = v.boxes[b];
  const int n_chains = B.n_atoms / chain_len;
  const int ch = (int)((blockIdx.x * blockDim.x + threadIdx.x) >> 6);
  if (ch >= n_chains) return;
  const int ln = lane();
  const int64_t N = v.N;
  const int64_t a0 = (int64_t)B.atom_off + (int64_t)ch * chain_len;
  double r[3] = {0.0, 0.0, 0.0};
  for (int p = 1 + ln; p < chain_len; p += 64)
    for (int q = 0; q < 3; ++q)
      r[q] += mi_rn(__dadd_rn(v.pos[q * N + a0 + p], -v.pos[q * N + a0 + p - 1]), B.L[q], B.invL[q]);
  for (int q = 0; q < 3; ++q) r[q] = wave_sum(r[q]);
  if (ln != 0) return;
  const int64_t c = (int64_t)B.atom_off / chain_len + ch;
  if (REF) {
    for (int q = 0; q < 3; ++q) ree0[3 * c + q] = r[q];
  } else {
    const double* r0 = ree0 + 3 * c;
    part[2 * c] = r[0] * r0[0] + r[1] * r0[1] + r[2] * r0[2];
    part[2 * c + 1] = r0[0] * r0[0] + r0[1] * r0[1] + r0[2] * r0[2];
  }
}

// Box b's autocorrelation: the chain terms of k_ree summed as double-double in a fixed order (each
// thread every 256th chain, a butterfly over the wave, then the waves), out[b] = num / den.
__global__ __launch_bounds__(256) void k_ree_reduce(Views v, int b, int chain_len, const double* part,
                                                    double* out) {
  __shared__ dd sh[4][2];
  const BoxDev& B = v.boxes[b];
  const int64_t c0 = (int64_t)B.atom_off / chain_len;
  const int64_t n = B.n_atoms / chain_len;
  dd s[2] = {dd_from(0.0), dd_from(0.0)};
#pragma unroll 4
  for (int64_t c = threadIdx.x; c < n; c += 256)
    for (int k = 0; k < 2; ++k) s[k] = dd_add(s[k], dd_from(part[2 * (c0 + c) + k]));
  for (int k = 0; k < 2; ++k)
    for (int off = 32; off > 0; off >>= 1) s[k] = dd_add(s[k], dd{__shfl_xor(s[k].hi, off), __shfl_xor(s[k].lo, off)});
  if (lane() == 0)
    for (int k = 0; k < 2; ++k) sh[threadIdx.x >> 6][k] = s[k];
  __syncthreads();
  if (threadIdx.x == 0) {
    dd num = sh[0][0], den = sh[0][1];
    for (int w = 1; w < 4; ++w) {
      num = dd_add(num, sh[w][0]);
      den = dd_add(den, sh[w][1]);
    }
    out[b] = (num.hi + num.lo) / (den.hi + den.lo);
  }
}

int obs_blocks(int64_t n) {
  const int64_t g = (n + kAtomBlock - 1) / kAtomBlock;
  return (int)(g < 1 ? 1 : (g > kObsBlocks ? kObsBlocks : g));
}

}  // namespace

void launch_obs_pairs(const Views& v, int b, int64_t n_cells, int chain_len, int excl, double dr, int n_bins,
                      unsigned long long* out, hipStream_t s) {
  const int64_t want = (n_cells + kObsWaves - 1) / kObsWaves;
  const int g = (int)(want > kObsBlocks ? kObsBlocks : want);
  hipLaunchKernelGGL(k_obs_pairs, dim3(g), dim3(64 * kObsWaves),
                     12 * (size_t)n_bins + 8, s, v, b, chain_len, excl, dr, n_bins, v.obs_part);
  hipLaunchKernelGGL(k_obs_reduce, dim3((n_bins + 63) / 64), dim3(64 * kObsReduceWaves), 0, s,
                     (const uint32_t*)v.obs_part, g, n_bins, out);
}

void launch_obs_dihedrals(const Views& v, int b, int64_t n_atoms, int chain_len, int n_bins,
                          unsigned long long* out, hipStream_t s) {
  const int g = obs_blocks(n_atoms);
  hipLaunchKernelGGL(k_obs_dihedrals, dim3(g), dim3(kAtomBlock), 0, s, v, b, chain_len, n_bins, v.obs_part);
  hipLaunchKernelGGL(k_obs_reduce, dim3((n_bins + 3 + 63) / 64), dim3(64 * kObsReduceWaves), 0, s,
                     (const uint32_t*)v.obs_part, g, n_bins + 3, out);
}

void launch_obs_chains(const Views& v, const FFDev& ff, int b, int64_t n_chains, int chain_len, double* out,
                       hipStream_t s) {
  const int64_t threads = n_chains * 64;
  hipLaunchKernelGGL(k_obs_chains, dim3((int)((threads + 255) / 256)), dim3(256), 0, s, v, ff, b, chain_len, out);
}

void launch_ree(const Views& v, int b, int64_t n_chains, int chain_len, bool reference, double* out, hipStream_t s) {
  const dim3 g((unsigned)((n_chains * 64 + 255) / 256)), blk(256);
  if (reference) {
    hipLaunchKernelGGL(k_ree<true>, g, blk, 0, s, v, b, chain_len, v.ree0, v.ree_part);
  } else {
    hipLaunchKernelGGL(k_ree<false>, g, blk, 0, s, v, b, chain_len, v.ree0, v.ree_part);
    hipLaunchKernelGGL(k_ree_reduce, dim3(1), dim3(256), 0, s, v, b, chain_len, (const double*)v.ree_part, out);
  }
}

}  // namespace mdk
