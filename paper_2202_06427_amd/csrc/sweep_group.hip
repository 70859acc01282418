// sweep_group.hip -- the cell-pair sweep for the reduced maps (counts, sums,
// energies, histograms) and the force gather in groups of 16 particles (paper
// section 2.8: a cell and half of its neighbour cells, all of them for the
// gather; sections 2.3/2.7: a function of every pair within the cutoff,
// reduced).
//
// Work decomposition: one block of four waves per tile (<= 64 consecutive
// sorted particles of a cell row), one wave per group of 16 of them; a tile
// of one or two groups spreads their neighbour rows over the waves instead.
// A wave scans the candidates of its stencil 64 at a time, keeps those within
// the cutoff of the group's bounding box (the paper's section 2.8 pruning by
// position, applied to 16 particles at a time) in an LDS list, and pairs 16
// of them with the group at a time: lane (q, c) = (lane / 16, lane % 16)
// holds candidate c and the group's particles 4q .. 4q + 3, so a block of 256
// pairs is four steps of 64.
//
// What bounds it: the vector ALU.  One particle per lane against every
// candidate of the stencil spent its instructions on pairs out of range (18 %
// in range at lcell 2); the boxes of 16 particles keep 43 %.  For the maps
// that need d^2 only to classify a pair (counts, distance histograms, the
// membership of speed histograms), d^2 of a block is one matrix instruction,
//   d^2 = |x_i|^2 + [x_j, y_j, z_j, |x_j|^2] . [-2x_i, -2y_i, -2z_i, 1],
// FP32 in and out, whose larger rounding error only widens the band of pairs
// that FP64 decides; the integers stay exact.  Sums and energies take d^2
// from coordinate differences on the vector ALU, as accurate as before.
//
// Measured (MI355X, whole pass with the cell-list build; before: one particle
// per lane): 10^6 particles, cutoff 12, lcell 2: 128-bin distance histogram
// 3.13 -> 0.74 ms (kernel 3.07 -> 0.60 ms, 3.1 10^8 instead of 1.55 10^9
// vector instructions: 0.51 ms of issue), sum of w_i w_j / d 1.34 -> 0.70 ms,
// count 1.16 -> 0.39 ms, LJ energy 1.40 -> 0.65 ms; distance-binned speeds of
// 2 10^6 clustered points in 2D 19.0 -> 5.5 ms; 10^4 particles in the FP64
// form, 128 bins, 0.16 -> 0.064 ms.  Force gather (both ends of every pair,
// both forms): 10^6 particles, cutoff 12 3.3 -> 1.85 ms in FP32 and 4.1 ->
// 2.15 ms in FP64, 8 requests of a served batch 1.79 -> 0.72 ms.
//
// Precision, FP32 form.  Maps that classify: FP32 coordinates relative to the
// centre of the group's bounding box (formed in FP64, rounded once).  With
// S = 2 max|x_i| + 1.01 rc every coordinate of a pair near the cutoff is at
// most S, and
//   |d2_32 - d2| <= 2 (1.01 rc) (u S) + 2 u S^2 (coordinates)
//                 + 3 u S^2 (|x_j|^2) + 3 u S^2 (|x_i|^2) + 8 u S^2 (products)
// is below 20 u S^2 (u = 2^-24); the band is 24 u S^2 (room for the roundings
// of rc and of the thresholds) plus the FP64 roundings, the host's term.
// Sums, energies and forces: 32-bit fixed-point coordinates about the same
// centre, whose differences are exact (quanta).  Pairs within the band of rc^2
// (histograms: of a bin edge; LJ: closer than the near threshold) are queued
// in LDS and recomputed in canonical FP64, 64 at a time.  The box test uses
// the FP32 coordinates: rounding is monotone, so a candidate's distance to the
// box is at most its distance to any particle of it.
//
// FP64 form: canonical d^2 of every pair of a block on the FP64 vector ALU; FP32
// only in the box test, and in lists, where matrix products leave out what is
// certainly beyond the cutoff and FP64 decides the rest.
//
// Sorted neighbour lists: the rows of a group (all partners of its particles;
// of a single set those of larger index) are counted by one sweep and written
// by a second to the ranges that the counts give (nl_rows.hip orders them).
// Both classify by matrix instructions; the second stages what may be in
// range, 8 bits a pair, and forms the distances of 64 staged pairs at a time
// with the arithmetic of the unsorted list.  2 10^5 particles, 30.5 10^6
// pairs: 152 + 433 us where the half-shell sweeps took 267 + 493 us and the
// radix sort behind them 3250; 10^4 against 10^6 particles 28 + 83 us.
#include <algorithm>
#include <type_traits>

#include "clmap_internal.h"
#include "device_util.h"
#include "hist_bins.h"

namespace clm {

namespace {

constexpr int kGrp = 16;      // particles of a group, candidates of a block
constexpr int kGCap = 80;     // candidate ring (a multiple of 16, >= 15 + 64)
constexpr int kGQCap = 320;   // FP64 queue (>= 63 + 4 * 64)
constexpr int kGWaves = 4;
constexpr int kFoldBlocks = 16; // blocks whose FP32 sums (16 terms a row and lane) enter FP64 together;
                                // a gather's energy and virial (4 terms a lane) do so after every block
constexpr int kFlatRun = 48;  // runs shorter than this on average are scanned together
constexpr int kFarQ = 1 << 30;  // an empty row (-) or column (+) in quanta: out of reach of any other
constexpr float kFar = 1e30f; // d^2 of an empty row or column
constexpr unsigned long long kCutRow = 1ull << 63;  // offset of the row that the capacity cuts
// Copies of a wave's forces of queued pairs in LDS, by lane: the 64 lanes of a
// batch add to 16 rows (2 10^6 clustered points in 2D, 9 % of the pairs in the
// queue: 16.9 ms with one copy, 14.5 with four or eight).
constexpr int kGaCopies = 4;

typedef float f32x4 __attribute__((ext_vector_type(4)));

template <int K>
__device__ __forceinline__ float ror16(float v) {
  return __builtin_bit_cast(float,
                            __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x120 + K, 0xF, 0xF, true));
}
__device__ __forceinline__ float min16(float v) {
  v = fminf(v, ror16<8>(v));
  v = fminf(v, ror16<4>(v));
  v = fminf(v, ror16<2>(v));
  return fminf(v, ror16<1>(v));
}
__device__ __forceinline__ float max16(float v) {
  v = fmaxf(v, ror16<8>(v));
  v = fmaxf(v, ror16<4>(v));
  v = fmaxf(v, ror16<2>(v));
  return fmaxf(v, ror16<1>(v));
}
__device__ __forceinline__ int min16i(int v) {
  v = min(v, ror16i<8>(v));
  v = min(v, ror16i<4>(v));
  v = min(v, ror16i<2>(v));
  return min(v, ror16i<1>(v));
}
__device__ __forceinline__ int max16i(int v) {
  v = max(v, ror16i<8>(v));
  v = max(v, ror16i<4>(v));
  v = max(v, ror16i<2>(v));
  return max(v, ror16i<1>(v));
}
__device__ __forceinline__ float uniform_f(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, v)));
}
__device__ __forceinline__ double uniform_d(double v) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)b);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(b >> 32));
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ float from_lane(float v, int src) {
  return __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(src << 2, __builtin_bit_cast(int, v)));
}

// Square root of a non-negative FP32 value, correctly rounded: the corrected
// reciprocal root equals the library's function for each of the 1.6 10^9 FP32
// values in [2^-96, 2^96] (compared one by one on gfx950); the others (zero,
// infinities and NaN among them) take the library's.
__device__ __forceinline__ float sqrt_fast(float q, unsigned long long m) {
  const float r = __builtin_amdgcn_rsqf(q);
  float s = q * r;
  s = __builtin_fmaf(__builtin_fmaf(-s, s, q), 0.5f * r, s);
  const uint32_t b = __builtin_bit_cast(uint32_t, q) - 0x0f800000u;  // 2^-96
  if (__builtin_expect((__builtin_amdgcn_ballot_w64(b > 0x6f800000u - 0x0f800000u) & m) != 0, 0)) {
    asm volatile("" : "+v"(q));  // keep the branch (the library's sequence is three times as long)
    s = __builtin_sqrtf(q);
  }
  return s;
}

constexpr bool group_ljf(int kind) { return kind == K_LJ_F || kind == K_LJ_FV; }
constexpr bool group_rows(int kind) { return kind == K_ROW_COUNT || kind == K_ROW_LIST || kind == K_VLIST; }
constexpr bool group_lists(int kind) { return kind == K_ROW_LIST || kind == K_VLIST; }
// maps that need d^2 only to classify a pair, in the FP32 form; lists of the
// FP64 form leave out what is certainly beyond the cutoff in this way and
// decide the other pairs in FP64
constexpr bool group_mfma(int kind, bool f64) {
  return group_lists(kind) || (!f64 && (kind == K_COUNT || kind == K_HIST_DIST || kind == K_HIST_REL ||
                                        kind == K_HIST_DV || kind == K_ROW_COUNT));
}

// LDS of one wave (5 KB: with the block's own the CU holds six or seven blocks).
// Runs: consecutive sorted particles of one row and image, at positions
// [.., end) of the wave's candidate sequence; particle = position + delta.
template <int KIND, bool F64>
struct GroupLds {
  static constexpr bool kVel = KIND == K_HIST_REL || KIND == K_HIST_DV;
  static constexpr bool kLJF = group_ljf(KIND);
  static constexpr bool kMfma = group_mfma(KIND, F64);
  float4 lst[kMfma ? kGCap : 1];           // x, y, z and |x|^2
  int4 lsti[!F64 && !kMfma ? kGCap : 1];   // x, y, z in quanta, and the weight (float bits)
  double4 lst64[F64 && !kMfma ? kGCap : 1];  // wrapped position and weight
  uint2 who[kGCap];                  // sorted index, image code (FP32 lists: and the row)
  float4 vel[kVel ? kGCap : 1];
  static constexpr bool kRows = group_rows(KIND), kList = group_lists(KIND);
  uint2 q[(F64 && !kMfma) || kList ? 1 : kGQCap];  // FP64 queue
  // row lists: the candidates' caller indices and, as the group's, positions;
  // (FP32 form) offsets in their cells, with the cell along the row
  uint32_t jdx[kRows && KIND != K_VLIST ? kGCap : 1];
  double rj[kList ? kGCap : 1][3], ri[kList ? kGrp : 1][3];
  float4 posj[kList && !F64 ? kGCap : 1], posi[kList && !F64 ? kGrp : 1];
  uint8_t stage[kList ? 4 * kWave : 4];  // pairs of the block: row | column << 4
  uint32_t cols[2];                      // Verlet lists: lanes in range
  double ga[kLJF && !F64 ? kGaCopies : 1][kLJF && !F64 ? kGrp * 3 : 1];  // forces of queued pairs, by row
  uint32_t run_end[kWave], run_delta[kWave];
  uint8_t run_kc[kWave];  // (FP32 lists: the lane that holds the run)
};

// F64: the plain FP64 form.
template <int DIM, int KIND, bool F64>
struct Group {
  static constexpr bool kLJF = group_ljf(KIND);   // forces: the full shell
  static constexpr bool kVir = KIND == K_LJ_FV;
  static constexpr bool kLJ = kLJF || KIND == K_LJ_E;
  static constexpr bool kDV = KIND == K_HIST_DV;
  static constexpr bool kRel = KIND == K_HIST_REL;
  static constexpr bool kVel = kDV || kRel;
  static constexpr bool kHist = KIND == K_HIST_DIST || kVel;
  static constexpr bool kW = KIND == K_SUM_W;
  static constexpr bool kSum = KIND == K_SUM_D || KIND == K_SUM_INV_D || kW || KIND == K_LJ_E;
  static constexpr bool kMfma = group_mfma(KIND, F64);
  static constexpr bool kRows = group_rows(KIND);
  static constexpr bool kList = group_lists(KIND);
  static constexpr bool kVL = KIND == K_VLIST;   // both ends list a pair
  // candidates' indices read with their positions (the registers are there in
  // 2D forces; elsewhere few steps queue a pair)
  static constexpr bool kWhoFirst = kLJF && DIM == 2;
  // the sweep itself is canonical FP64 (of a list only its distances are)
  static constexpr bool kF64 = F64 && !kMfma;
  using Real = typename std::conditional<F64, double, int>::type;

  const JobDesc* J;
  GroupLds<KIND, F64>* L;
  const double* tks;       // LDS: image shifts, 3 per code
  // row lists: LDS counters of the block's rows (this group's 16), the rows'
  // output offsets, and this lane's rows
  uint32_t* rcnt;
  uint32_t* vslot;         // Verlet lists: LDS, particles of the group's rows
  uint32_t* gcnt;          // Verlet lists: LDS counters of the candidates of four rows
  const unsigned long long* roff;
  bool with_cut;           // the group has the row that the capacity cuts
  uint32_t ir[kRows ? 4 : 1], cr[kRows ? 4 : 1];
  // lists: staged pairs, the group's row, FP32 thresholds of cell offsets and,
  // per lane, the run's first cell (unwrapped ux; linear) and cells
  uint32_t nst;
  int gcy, gcz;
  int l_ux, l_cell, l_nc;
  const uint32_t* OFFJ;
  // Which end of a pair the half shell visits it from: the group's (kAhead),
  // the candidate's, or that of the smaller sorted index (the own row).
  static constexpr int kAhead = 0, kBehind = 1, kByIndex = 2;
  static constexpr int kRowBias = 128;
  // image code of the runs of row (dy, dz); FP32 lists: with that end and the row
  __device__ __forceinline__ int row_code(int kc, int dy, int dz) const {
    if constexpr (!kList || F64) return kc;
    const int px = kc % 3 - 1;
    const int z = cross ? 1 : (dz != 0 ? dz : (dy != 0 ? dy : px));
    return kc | ((z == 0 ? kByIndex : (z > 0 ? kAhead : kBehind)) << 5) | ((dy + kRowBias) << 8) |
           ((dz + kRowBias) << 16);
  }
  uint32_t* hist;          // [nbins + 1][C] counters of the block, from this lane's copy on
  double* hsum;            // [nbins + 1][C] sums (the last bin's is not used)
  int lane, c, q;
  int lgC;
  uint32_t gs;             // first particle of the group
  int gc;                  // its particles
  int cross;
  double rc2, s2;
  double O[3];             // origin of the FP32 coordinates
  double scale;
  float bl[3], bh[3];      // the group's box
  float lo, hi;            // membership thresholds
  float test_hi;           // of the box test (FP32 coordinates)
  float near2;
  // FP32 sums: coordinates in quanta of 1 / (iq scale), iq a power of two;
  // unit: what a sum of d, of 1/d or of force terms is worth
  double iq, unit;
  float sig2;              // LJ: sigma^2 in quanta
  float ih2;               // speed histograms: (1 / bin width)^2
  int nbins;
  // histogram: the bin of u = sqrt(v) (bin widths) is certain when
  // |fract(u) - 1/2| < c3 - c1 / sqrt(v), or u > over, or v < first (bin 0,
  // zero and coincident values among it)
  float c1, c3, over, first;
  double inv_h64;
  float inv_h32;
  const double* E64;       // (FP64 form: in LDS)
  const double4* R;
  const uint32_t* IDXJ;
  const double* VJ64;
  int want_sums;
  // per lane
  f32x4 cn;                // |x_i|^2 of rows 4q .. 4q + 3
  float a_op;              // matrix operand A: component q of [-2x, -2y, -2z, 1] of row c
  Real xr[4][3];            // coordinates of rows 4q .. 4q + 3
  float vr[4][3];          // velocities
  float acc[4];            // FP32 sums of the rows since the last fold
  double wr[4];            // weights of the rows
  double accE;
  // forces: sums of the rows (FP32 form: f32 since the last fold), unscaled
  float f32[kLJF && !F64 ? 4 : 1][3];
  double fr[kLJF ? 4 : 1][3];
  double wunit;            // FP32 form: virial terms
  double B[9];             // image part of the box gradient
  double W[6];
  unsigned long long cnt_wave;
  uint32_t qband, qnear;   // the wave's re-evaluations: in the band, others
  uint32_t qtail;
  uint32_t head, fill;     // the ring: first slot (a multiple of 16), candidates
  int img;                 // candidates up to the last periodic image
  int unfolded;            // blocks since the last fold

  __device__ __forceinline__ void hist_add(int k) {
    atomicAdd((uint32_t*)((char*)hist + ((uint32_t)k << (lgC + 2))), 1u);
  }
  __device__ __forceinline__ void hsum_add(int k, double v) {
    atomicAdd((double*)((char*)hsum + ((uint32_t)k << (lgC + 3))), v);
  }

  static constexpr int kHere = 13;  // image code of K = (0, 0, 0)
  // box gradient: half of f D K^T (every pair is visited from both ends)
  __device__ __forceinline__ void image_term(const double* fD, int kc) {
    const double p[3] = {0.5 * (double)(kc % 3 - 1), 0.5 * (double)((kc / 3) % 3 - 1),
                         0.5 * (double)(kc / 9 - 1)};
#pragma unroll
    for (int a = 0; a < DIM; ++a)
#pragma unroll
      for (int b = 0; b < DIM; ++b) B[a * 3 + b] += fD[a] * p[b];
  }

  __device__ __forceinline__ void virial_term(const double* fD, const double* D, double c) {
    W[0] += c * fD[0] * D[0];
    W[1] += c * fD[0] * D[1];
    W[3] += c * fD[1] * D[1];
    if (DIM == 3) {
      W[2] += c * fD[0] * D[2];
      W[4] += c * fD[1] * D[2];
      W[5] += c * fD[2] * D[2];
    }
  }

  // ------------------------------------------------------------ row lists
  // Entry p of row `row` of the group: partner jo at distance d.
  __device__ __forceinline__ void row_store(int row, uint32_t p, uint32_t jo, double d) {
    const unsigned long long o = roff[row], g = o + p;
    if (g < (unsigned long long)ldu(&J->capacity)) {
      ldu(&J->row_j)[g] = jo;
      double* rd = ldu(&J->row_d);
      if (rd) rd[g] = d;
    }
    // (a branch of the wave: asked of every entry it took 5 % of the kernel, so 3 %)
    if (__builtin_expect(with_cut, 0)) {
      if (o == kCutRow) {  // which of its entries are written is decided later (nl_rows.hip)
        atomicOr(&ldu(&J->row_bits)[jo >> 5], 1u << (jo & 31u));
        double* dj = ldu(&J->row_dj);
        if (dj) dj[jo] = d;
      }
    }
  }

  // Verlet lists: the particle of this lane's row where the group's are ordered
  // so that every four are close: halves by y, then by z.  (Along x the 16 are
  // close already: consecutive particles of a row of cells, which are ordered
  // by x.)  At 29 particles a cell the force kernel takes 199 us instead of 217.
  __device__ __forceinline__ uint32_t vl_order(const double4& r, uint32_t sl) {
    const int n = gc, me = (int)c;
    const float y = (float)(r.y - uniform_d(r.y)), z = DIM == 3 ? (float)(r.z - uniform_d(r.z)) : 0.0f;
    int ry = 0;
    for (int k = 0; k < n; ++k) {
      const float v = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, y), k));
      ry += v < y || (v == y && k < me) ? 1 : 0;
    }
    const int half = ry >= 8 ? 1 : 0;
    int rz = 0;
    for (int k = 0; k < n; ++k) {
      const float v = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, z), k));
      rz += __builtin_amdgcn_readlane(half, k) == half && (v < z || (v == z && k < me)) ? 1 : 0;
    }
    const int row = 8 * half + rz;  // of particle c; not finite: any order would do, but one it must be
    const unsigned long long ok = __builtin_amdgcn_ballot_w64(lane < n && y - y == 0.0f && z - z == 0.0f);
    if (ok != (n < kWave ? (1ull << n) - 1ull : ~0ull)) return sl;
    int p = 0;
    for (int k = 0; k < n; ++k) p = __builtin_amdgcn_readlane(row, k) == min(me, n - 1) ? k : p;
    return (uint32_t)p;
  }

  // Verlet lists: the lanes (q, c) with a staged pair in range of a row of q (a
  // block with a pair in the band of the list's cutoff but beyond it).
  __device__ __forceinline__ unsigned long long vl_columns(uint32_t pos, uint32_t n) {
    if (lane < 2) L->cols[lane] = 0u;
    __builtin_amdgcn_wave_barrier();
    for (uint32_t b = (uint32_t)lane; b < n; b += kWave) {
      const uint32_t e = L->stage[b], s = pos + (e >> 4);
      const double* t = &tks[L->who[s].y * 3];
      double D[3] = {0.0, 0.0, 0.0};
#pragma unroll
      for (int a = 0; a < DIM; ++a) D[a] = (L->rj[s][a] - L->ri[e & 15u][a]) + t[a];
      double d2 = D[0] * D[0] + D[1] * D[1];
      if (DIM == 3) d2 = d2 + D[2] * D[2];
      const uint32_t bit = 16u * ((e & 15u) >> 2) + (e >> 4);
      if (d2 <= rc2) atomicOr(&L->cols[bit >> 5], 1u << (bit & 31u));
    }
    __builtin_amdgcn_wave_barrier();
    return (unsigned long long)L->cols[0] | ((unsigned long long)L->cols[1] << 32);
  }

  // Verlet lists of the four rows of every q: the lanes' candidates are appended.
  __device__ __forceinline__ void vl_append(uint32_t pos, unsigned long long lanes) {
    const uint32_t mine = (uint32_t)(lanes >> (16 * q)) & 0xffffu;
    uint32_t p = 0u;
    if (c == 0 && mine) p = atomicAdd(&gcnt[q], (uint32_t)__popc(mine));
    p = (uint32_t)__shfl((int)p, 16 * q, kWave);
    if ((mine >> c) & 1u) {
      const size_t cap = (size_t)ldu(&J->vl_cap);
      const uint32_t k = p + (uint32_t)__popc(mine & ((1u << c) - 1u));
      const uint2 w = L->who[pos + (uint32_t)c];
      if (k < (uint32_t)min(gc - 4 * q, kVlRows) * (uint32_t)cap)
        ldu(&J->vl_list)[(size_t)(gs + 4u * (uint32_t)q) * cap + k] = (w.x << 5) | w.y;
    }
    __builtin_amdgcn_wave_barrier();
  }

  // The block's staged pairs, 64 at a time (about a quarter of a block's pairs
  // are within reach and of larger index, so they are evaluated densely).  The
  // values are those of the unsorted list: in the FP32 form the half-shell
  // owner's position relative to the other end's cell, canonical FP64 where
  // that is within the band of the cutoff.
  // Returns whether a staged pair was out of range (Verlet lists).
  __device__ __forceinline__ bool row_flush(uint32_t pos) {
    bool out = false;
    __builtin_amdgcn_wave_barrier();
    for (uint32_t b = 0; b < nst; b += kWave) {
      if (b + (uint32_t)lane < nst) {
        const uint32_t e = L->stage[b + (uint32_t)lane];
        const int row = (int)(e & 15u);
        const uint32_t s = pos + (e >> 4);
        const uint2 w = L->who[s];
        bool in, exact = true;
        double d = 0.0;
        if constexpr (!F64) {
          const int side = (int)((w.y >> 5) & 3u), kc = (int)(w.y & 31u);
          const bool ahead = side == kAhead || (side == kByIndex && w.x > gs + (uint32_t)row);
          // the group's particle seen from the candidate: the opposite image
          const float4 p = ahead ? L->posj[s] : L->posi[row];
          const int ux = __builtin_bit_cast(int, p.w);
          const double u0 = (double)(ahead ? ux : ux - (kc % 3 - 1) * ldu(&J->n[0]));
          const double u1 = (double)(ahead ? gcy + (int)((w.y >> 8) & 255u) - kRowBias
                                           : gcy - ((kc / 3) % 3 - 1) * ldu(&J->n[1]));
          const double u2 = DIM == 3 ? (double)(ahead ? gcz + (int)((w.y >> 16) & 255u) - kRowBias
                                                      : gcz - (kc / 9 - 1) * ldu(&J->n[2])) : 0.0;
          const double* o = ahead ? L->ri[row] : L->rj[s];
          const float pa[3] = {p.x, p.y, p.z};
          float D[3] = {0.0f, 0.0f, 0.0f};
#pragma unroll
          for (int a = 0; a < DIM; ++a) {
            const double org = (ldu(&J->Hn[a * 3 + 1]) * u1 + ldu(&J->Hn[a * 3 + 2]) * u2) + ldu(&J->Hn[a * 3]) * u0;
            D[a] = pa[a] - (float)(o[a] - org);
          }
          const float d2 = DIM == 3 ? __builtin_fmaf(D[2], D[2], __builtin_fmaf(D[1], D[1], D[0] * D[0]))
                                    : __builtin_fmaf(D[1], D[1], D[0] * D[0]);
          in = d2 <= ldu(&J->lo32);
          exact = !in && d2 <= ldu(&J->hi32);
          d = (double)__builtin_sqrtf(d2);
        }
        if (exact) {
          const double* t = &tks[(w.y & 31u) * 3];
          double D[3] = {0.0, 0.0, 0.0};
#pragma unroll
          for (int a = 0; a < DIM; ++a) D[a] = (L->rj[s][a] - L->ri[row][a]) + t[a];
          double d2 = D[0] * D[0] + D[1] * D[1];
          if (DIM == 3) d2 = d2 + D[2] * D[2];
          in = d2 <= rc2;
          d = sqrt(d2);
        }
        out = out || !in;
        if (in) {
          const uint32_t p = atomicAdd(&rcnt[row], 1u);
          if constexpr (!kVL) row_store(row, p, L->jdx[s], d);
        }
      }
    }
    nst = 0;
    __builtin_amdgcn_wave_barrier();
    return kVL && __builtin_amdgcn_ballot_w64(out) != 0ull;
  }

  // ------------------------------------------------------------ FP64 queue
  __device__ __forceinline__ double speed64(uint32_t io, uint32_t jo) const {
    const double* vi = ldu(&J->vel64_x);
    double dv[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int a = 0; a < DIM; ++a) dv[a] = VJ64[(size_t)jo * DIM + a] - vi[(size_t)io * DIM + a];
    double qq = dv[0] * dv[0] + dv[1] * dv[1];
    if (DIM == 3) qq = qq + dv[2] * dv[2];
    return qq;
  }

  // canonical FP64 evaluation of one queued pair; returns whether it is in range
  // and not counted yet (counts are the wave's, in scalar registers)
  __device__ __forceinline__ bool process(const uint2 e) {
    const uint32_t j = e.x, i = gs + (e.y & 15u);
    const double4 rI = ldu(&J->r64_x)[i];
    const double4 rJ = R[j];
    const double* tk = &tks[((e.y >> 8) & 31u) * 3];
    double D[3];
    D[0] = (rJ.x - rI.x) + tk[0];
    D[1] = (rJ.y - rI.y) + tk[1];
    double d2 = D[0] * D[0] + D[1] * D[1];
    if (DIM == 3) {
      D[2] = (rJ.z - rI.z) + tk[2];
      d2 = d2 + D[2] * D[2];
    }
    if (!(d2 <= rc2)) return false;
    if constexpr (KIND == K_SUM_D) accE += sqrt(d2);
    if constexpr (KIND == K_SUM_INV_D) accE += 1.0 / sqrt(d2);
    if constexpr (kW) accE += (rI.w * rJ.w) / sqrt(d2);
    if constexpr (kLJ) {
      const double r = rcp64(d2);
      const double x = s2 * r;
      const double x3 = x * x * x;
      const double u = x3 * x3 - x3;
      accE += kLJF ? 0.5 * u : u;
      if constexpr (kLJF) {
        const double f = (2.0 * x3 * x3 - x3) * r;
        const int kc = (int)((e.y >> 8) & 31u);
        double fD[3] = {0.0, 0.0, 0.0};
#pragma unroll
        for (int a = 0; a < DIM; ++a) {
          fD[a] = f * D[a];
          atomicAdd(&L->ga[lane & (kGaCopies - 1)][(e.y & 15u) * 3 + a], fD[a]);
        }
        if (kc != kHere) image_term(fD, kc);
        if constexpr (kVir) virial_term(fD, D, 0.5);
      }
    }
    if constexpr (kRows) atomicAdd(&rcnt[e.y & 15u], 1u);
    if constexpr (KIND == K_HIST_DIST) hist_add(bin64(E64, nbins, inv_h64, d2));
    if constexpr (kDV) {
      const int k = bin64(E64, nbins, inv_h64, d2);
      hist_add(k);
      if (k < nbins) hsum_add(k, sqrt(speed64(ldu(&J->idx_x)[i], IDXJ[j])));
    }
    if constexpr (kRel) {
      const double qq = speed64(ldu(&J->idx_x)[i], IDXJ[j]);
      const int k = bin64(E64, nbins, inv_h64, qq);
      hist_add(k);
      if (want_sums && k < nbins) hsum_add(k, sqrt(qq));
    }
    return ((e.y >> 16) & 1u) != 0u;
  }

  __device__ __forceinline__ void drain(bool all) {
    uint32_t h = 0;
    const uint32_t tl = (uint32_t)uniform((int)qtail);
    while (tl - h >= (uint32_t)kWave || (all && tl != h)) {
      const uint32_t nb = min(tl - h, (uint32_t)kWave);
      bool counted = false;
      if ((uint32_t)lane < nb) counted = process(L->q[h + (uint32_t)lane]);
      cnt_wave += (unsigned long long)__popcll(__builtin_amdgcn_ballot_w64(counted));
      h = (uint32_t)uniform((int)(h + nb));
    }
    const uint32_t left = tl - h;  // fewer than 64: to the front
    if (h != 0u && left != 0u) {
      uint2 e = make_uint2(0u, 0u);
      if ((uint32_t)lane < left) e = L->q[h + (uint32_t)lane];
      __builtin_amdgcn_wave_barrier();
      if ((uint32_t)lane < left) L->q[lane] = e;
      __builtin_amdgcn_wave_barrier();
    }
    qtail = left;
  }

  __device__ __forceinline__ void enqueue(unsigned long long m, unsigned long long band, int r, uint2 w) {
    if (__builtin_amdgcn_inverse_ballot_w64(m)) {
      const bool b = __builtin_amdgcn_inverse_ballot_w64(band);
      L->q[qtail + (uint32_t)lane_rank(m)] =
          make_uint2(w.x, (uint32_t)(4 * q + r) | (w.y << 8) | (b ? (1u << 16) : 0u));
    }
    const uint32_t all = (uint32_t)__popcll(m), b = (uint32_t)__popcll(band);
    qtail += all;
    qband += b;
    qnear += all - b;
  }

  // ------------------------------------------------------------ one block
  // Ring slots [pos, pos + nv) (nv <= 16) against the
  // group; SELF: the group against itself, pairs column > row (half shell) or
  // column != row (forces).  IMG: some candidate is a periodic image.
  template <bool SELF>
  __device__ __forceinline__ unsigned long long self_mask(int r) const {
    if constexpr (!SELF || (kRows && !kVL)) return ~0ull;  // (row lists compare indices)
    return kLJF || kVL ? __builtin_amdgcn_ballot_w64(c != 4 * q + r) : __builtin_amdgcn_ballot_w64(c > 4 * q + r);
  }

  template <bool SELF, bool IMG>
  __device__ __forceinline__ void block(uint32_t pos, int nv) {
    if constexpr (kF64)
      block64<SELF, IMG>(pos, nv);
    else
      block32<SELF, IMG>(pos, nv);
  }

  template <bool SELF, bool IMG>
  __device__ __forceinline__ void block32(uint32_t pos, int nv) {
    const uint32_t s = pos + (uint32_t)c;
    const bool have = c < nv;
    f32x4 d;
    int4 xi = make_int4(0, 0, 0, 0);
    if constexpr (kMfma) {
      // operand B of lane (q, c): component q of [x, y, z, |x|^2] of candidate c
      const float b = ((const float*)&L->lst[s])[q];
      const float bb = have ? b : (q == 3 ? kFar : 0.0f);
      d = __builtin_amdgcn_mfma_f32_16x16x4f32(a_op, bb, cn, 0, 0, 0);
    } else {
      xi = L->lsti[s];
      if (!have) xi = make_int4(kFarQ, 0, 0, 0);
    }
    float4 vj = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if constexpr (kVel) vj = L->vel[s];
    uint2 wj = make_uint2(0u, 0u);  // (of a column that is there: others are out of range)
    if constexpr (kWhoFirst) wj = L->who[s];
    uint32_t jo = 0u;
    if constexpr (kRows && !kVL) jo = L->jdx[s];
    float tj[3] = {0.0f, 0.0f, 0.0f};
    float e32 = 0.0f, w32[6] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};  // forces: energy and virial of the block
    unsigned long long any = 0ull;  // lists: pairs staged
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float d2, D[3] = {0.0f, 0.0f, 0.0f};
      if constexpr (kMfma) {
        d2 = d[r];
      } else {
        D[0] = (float)(xi.x - (int)xr[r][0]);
        D[1] = (float)(xi.y - (int)xr[r][1]);
        if (DIM == 3) D[2] = (float)(xi.z - (int)xr[r][2]);
        d2 = DIM == 3 ? __builtin_fmaf(D[2], D[2], __builtin_fmaf(D[1], D[1], D[0] * D[0]))
                      : __builtin_fmaf(D[1], D[1], D[0] * D[0]);
      }
      unsigned long long ok = self_mask<SELF>(r);
      // a single set lists a pair at the particle of smaller index
      if constexpr (kRows && !kVL)
        if (!cross) ok = __builtin_amdgcn_ballot_w64(jo > ir[r]);
      const unsigned long long mlo = __builtin_amdgcn_ballot_w64(d2 <= lo) & ok;
      const unsigned long long mhi = __builtin_amdgcn_ballot_w64(d2 <= hi) & ok;
      unsigned long long spec = mhi & ~mlo;
      const unsigned long long band = spec;
      cnt_wave += (unsigned long long)__popcll(mlo);
      if constexpr (KIND == K_ROW_COUNT) cr[r] += __builtin_amdgcn_inverse_ballot_w64(mlo) ? 1u : 0u;
      if constexpr (kList) {  // classified when written
        if (__builtin_amdgcn_inverse_ballot_w64(mhi))
          L->stage[nst + (uint32_t)lane_rank(mhi)] = (uint8_t)((4 * q + r) | (c << 4));
        nst += (uint32_t)__popcll(mhi);
        spec = 0ull;
        any |= mhi;
      }
      if constexpr (KIND == K_SUM_D || KIND == K_SUM_INV_D || kW) {
        const bool in = __builtin_amdgcn_inverse_ballot_w64(mlo);
        // (coincident particles: d = 0, not 0 times infinity)
        const float rs = __builtin_amdgcn_rsqf(KIND == K_SUM_D ? fmaxf(d2, 1e-37f) : d2);
        const float t = KIND == K_SUM_D ? d2 * rs : (kW ? __builtin_bit_cast(float, xi.w) * rs : rs);
        acc[r] += in ? t : 0.0f;
      }
      if constexpr (kLJ) {  // x = sigma^2 / d^2
        // (of the pairs that may be in range: the threshold can be beyond any d^2,
        // that of empty rows and columns among them)
        const unsigned long long near = __builtin_amdgcn_ballot_w64(d2 < near2) & mhi;
        spec |= near;
        const bool fast = __builtin_amdgcn_inverse_ballot_w64(mlo & ~near);
        const float x = fast ? sig2 * __builtin_amdgcn_rcpf(d2) : 0.0f;
        const float x3 = x * x * x;
        const float u = __builtin_fmaf(x3, x3, -x3);
        if constexpr (!kLJF) {
          acc[r] += u;
        } else {
          e32 += u;
          const float f = __builtin_fmaf(2.0f, u, x3) * x;
#pragma unroll
          for (int a = 0; a < DIM; ++a) {
            f32[r][a] = __builtin_fmaf(f, D[a], f32[r][a]);
            if constexpr (IMG) tj[a] = __builtin_fmaf(f, D[a], tj[a]);
          }
          if constexpr (kVir) {
            const float tx = f * D[0], ty = f * D[1];
            w32[0] = __builtin_fmaf(tx, D[0], w32[0]);
            w32[1] = __builtin_fmaf(tx, D[1], w32[1]);
            w32[3] = __builtin_fmaf(ty, D[1], w32[3]);
            if (DIM == 3) {
              w32[2] = __builtin_fmaf(tx, D[2], w32[2]);
              w32[4] = __builtin_fmaf(ty, D[2], w32[4]);
              w32[5] = __builtin_fmaf(f * D[2], D[2], w32[5]);
            }
          }
          // finish this step's sums before the next step's (left free, the
          // scheduler interleaves the four steps and spills)
          asm volatile("" : "+v"(f32[r][0]), "+v"(f32[r][1]), "+v"(f32[r][2]), "+v"(e32));
        }
      }
      if constexpr (kHist) {
        float v = d2;
        float qq = 0.0f;
        if constexpr (kVel) {
          const float ex = vj.x - vr[r][0], ey = vj.y - vr[r][1];
          const float ez = DIM == 3 ? vj.z - vr[r][2] : 0.0f;
          qq = DIM == 3 ? __builtin_fmaf(ez, ez, __builtin_fmaf(ey, ey, ex * ex))
                        : __builtin_fmaf(ey, ey, ex * ex);
          if constexpr (kRel) v = qq * ih2;
        }
        const float rs = __builtin_amdgcn_rsqf(v);
        const float u = v * rs;  // in bin widths
        const float w = __builtin_amdgcn_fractf(u) - 0.5f;
        const unsigned long long put =
            (__builtin_amdgcn_ballot_w64(__builtin_fabsf(w) < __builtin_fmaf(-c1, rs, c3)) |
             __builtin_amdgcn_ballot_w64(u > over) | __builtin_amdgcn_ballot_w64(v < first)) & mlo;
        spec = mhi & ~put;
        if (__builtin_amdgcn_inverse_ballot_w64(put)) {
          const int k = min((int)u, nbins);
          hist_add(k);
          if constexpr (kVel) {
            if (kDV || want_sums) hsum_add(k, (double)sqrt_fast(qq, put));
          }
        }
      }
      if (!kList && spec) enqueue(spec, band, r, kWhoFirst ? wj : L->who[s]);
    }
    if constexpr (kVL) {
      const uint32_t n = nst;
      if (row_flush(pos)) any = vl_columns(pos, n);
      if (any) vl_append(pos, any);
    } else if constexpr (kList) {
      row_flush(pos);
    }
    if constexpr (kLJF) {
      accE += 0.5 * (double)e32;
      if constexpr (kVir) {
#pragma unroll
        for (int k = 0; k < 6; ++k) W[k] += wunit * (double)w32[k];
      }
    }
    if constexpr (kLJF && IMG) {
      const int kc = have ? (int)L->who[s].y : kHere;
      if (kc != kHere) {
        const double fD[3] = {(double)tj[0] * unit, (double)tj[1] * unit, (double)tj[2] * unit};
        image_term(fD, kc);
      }
    }
  }

  // Canonical FP64: D = (r_j - r_i) + H K, every operation rounded on its own.
  template <bool SELF, bool IMG>
  __device__ __forceinline__ void block64(uint32_t pos, int nv) {
    const uint32_t s = pos + (uint32_t)c;
    const bool have = c < nv;
    double4 rj = L->lst64[s];
    if (!have) rj = make_double4(1e100, 0.0, 0.0, 0.0);  // (unwritten slots may hold NaN)
    int kc = kHere;
    double t[3] = {0.0, 0.0, 0.0};
    if constexpr (IMG) {
      kc = have ? (int)L->who[s].y : kHere;
#pragma unroll
      for (int a = 0; a < DIM; ++a) t[a] = tks[kc * 3 + a];
    }
    uint32_t jo = 0u;
    if constexpr (kRows) jo = L->jdx[s];
    double tj[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      double D[3] = {rj.x - xr[r][0], rj.y - xr[r][1], DIM == 3 ? rj.z - xr[r][2] : 0.0};
      if constexpr (IMG) {
#pragma unroll
        for (int a = 0; a < DIM; ++a) D[a] = D[a] + t[a];
      }
      double d2 = D[0] * D[0] + D[1] * D[1];
      if (DIM == 3) d2 = d2 + D[2] * D[2];
      unsigned long long ok = self_mask<SELF>(r);
      if constexpr (kRows)
        if (!cross) ok = __builtin_amdgcn_ballot_w64(jo > ir[r]);
      const unsigned long long min = __builtin_amdgcn_ballot_w64(d2 <= rc2) & ok;
      const bool in = __builtin_amdgcn_inverse_ballot_w64(min);
      cnt_wave += (unsigned long long)__popcll(min);
      if constexpr (KIND == K_ROW_COUNT) cr[r] += in ? 1u : 0u;
      if constexpr (kLJ) {
        const double ri = in ? rcp64(d2) : 0.0;
        const double x = s2 * ri;
        const double x3 = x * x * x;
        const double u = x3 * x3 - x3;
        accE += u;
        if constexpr (kLJF) {
          const double f = (2.0 * x3 * x3 - x3) * ri;
          double fD[3] = {0.0, 0.0, 0.0};
#pragma unroll
          for (int a = 0; a < DIM; ++a) {
            fr[r][a] = __builtin_fma(f, D[a], fr[r][a]);
            if constexpr (IMG) tj[a] = __builtin_fma(f, D[a], tj[a]);
            fD[a] = f * D[a];
          }
          if constexpr (kVir) virial_term(fD, D, 0.5);
          asm volatile("" : "+v"(fr[r][0]), "+v"(fr[r][1]), "+v"(fr[r][2]), "+v"(accE));
        }
      } else if constexpr (KIND != K_COUNT && !kRows) {
        if (in) {
          if constexpr (KIND == K_HIST_DIST) hist_add(bin64_near(E64, nbins, inv_h32, inv_h64, d2));
          if constexpr (KIND == K_SUM_D) accE += sqrt(d2);
          if constexpr (KIND == K_SUM_INV_D) accE += 1.0 / sqrt(d2);
          if constexpr (kW) accE += (wr[r] * rj.w) / sqrt(d2);
        }
      }
    }
    if constexpr (kLJF && IMG) {
      if (kc != kHere) image_term(tj, kc);
    }
  }

  // FP32 sums into FP64
  __device__ __forceinline__ void fold() {
    if constexpr (kSum && !F64) {
      const double un = KIND == K_LJ_E ? 1.0 : unit;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        accE += kW ? wr[r] * ((double)acc[r] * un) : (double)acc[r] * un;
        acc[r] = 0.0f;
      }
    }
    if constexpr (kLJF && !F64) {
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int a = 0; a < DIM; ++a) {
          fr[r][a] += (double)f32[r][a];
          f32[r][a] = 0.0f;
        }
    }
    unfolded = 0;
  }

  // FP32 coordinates of a position: scale r + o, o = scale (image shift - origin)
  __device__ __forceinline__ float4 rel(const double4& r, const double* o) const {
    float4 x;
    x.x = (float)__builtin_fma(r.x, scale, o[0]);
    x.y = (float)__builtin_fma(r.y, scale, o[1]);
    x.z = DIM == 3 ? (float)__builtin_fma(r.z, scale, o[2]) : 0.0f;
    x.w = DIM == 3 ? __builtin_fmaf(x.z, x.z, __builtin_fmaf(x.y, x.y, x.x * x.x))
                   : __builtin_fmaf(x.y, x.y, x.x * x.x);
    return x;
  }

  // The same in quanta.  Differences of these are exact, so a pair's D carries
  // one rounding to FP32 and the quantum (2^-29 of the pair's reach or less)
  // however long the group's box is: FP32 coordinates about the box centre
  // lose the close pairs of a sparse row, whose 16 particles span many cells
  // (worst force error 1.5 times that of cell-relative coordinates at 0.55
  // particles a unit length).
  __device__ __forceinline__ int4 quanta(const double4& r, const double* o) const {
    return make_int4((int)rint(__builtin_fma(r.x, scale, o[0]) * iq), (int)rint(__builtin_fma(r.y, scale, o[1]) * iq),
                     DIM == 3 ? (int)rint(__builtin_fma(r.z, scale, o[2]) * iq) : 0, 0);
  }

  // lanes with keep append candidate j (FP32 coordinates x, position r, image
  // code kc) to the ring
  __device__ __forceinline__ void push(bool keep, const float4& x, const double4& r, const double* o, uint32_t j,
                                       int kc, int ux = 0) {
    const unsigned long long m = __builtin_amdgcn_ballot_w64(keep);
    if (keep) {
      uint32_t s = head + fill + (uint32_t)lane_rank(m);
      s = min(s, s - (uint32_t)kGCap);  // the ring's slot (smaller than twice its size)
      if constexpr (kF64) {
        L->lst64[s] = r;
        if constexpr (kRows) L->jdx[s] = IDXJ[j];
      } else if constexpr (kMfma) {
        L->lst[s] = x;
        if constexpr (kRows && !kVL) L->jdx[s] = IDXJ[j];
        if constexpr (kList) {
          if constexpr (!F64) {
            float4 p = (cross ? ldu(&J->pos_y) : ldu(&J->pos_x))[j];
            p.w = __builtin_bit_cast(float, ux);
            L->posj[s] = p;
          }
          L->rj[s][0] = r.x;
          L->rj[s][1] = r.y;
          L->rj[s][2] = r.z;
        }
      } else {
        int4 v = quanta(r, o);
        if constexpr (kW) v.w = __builtin_bit_cast(int, (float)r.w);
        L->lsti[s] = v;
      }
      L->who[s] = make_uint2(j, (uint32_t)kc);
      if constexpr (kVel) L->vel[s] = (cross ? ldu(&J->vel32_y) : ldu(&J->vel32_x))[j];
    }
    fill += (uint32_t)__popcll(m);
    if constexpr (kLJF || kF64) {
      if (__builtin_amdgcn_ballot_w64(keep && kc != kHere)) img = (int)fill;
    }
    __builtin_amdgcn_wave_barrier();
  }

  // 64 candidates (one per lane, valid: j, image code kc, coordinates
  // fma(scale, r, o)): those within the cutoff of the group's box to the ring,
  // then the ring's full blocks.
  __device__ __forceinline__ void test(bool valid, uint32_t j, int kc, const double* o,
                                       int ux = 0) {
    const double4 r = R[j];
    const float4 x = rel(r, o);
    const float ex = fmaxf(fmaxf(bl[0] - x.x, x.x - bh[0]), 0.0f);
    const float ey = fmaxf(fmaxf(bl[1] - x.y, x.y - bh[1]), 0.0f);
    float dd = __builtin_fmaf(ey, ey, ex * ex);
    if (DIM == 3) {
      const float ez = fmaxf(fmaxf(bl[2] - x.z, x.z - bh[2]), 0.0f);
      dd = __builtin_fmaf(ez, ez, dd);
    }
    push(valid && dd <= test_hi, x, r, o, j, kc, ux);
    while (fill >= (uint32_t)kGrp) {
      if constexpr (!kF64 && !kList) {
        if (qtail >= (uint32_t)kWave) drain(false);
      }
      if ((kLJF || kF64) && img > 0)
        block<false, kLJF || kF64>(head, kGrp);
      else
        block<false, false>(head, kGrp);
      head = head + kGrp == kGCap ? 0u : head + (uint32_t)kGrp;
      fill -= (uint32_t)kGrp;
      img -= kGrp;
      if (++unfolded >= kFoldBlocks) fold();
    }
  }

  // Candidates of a batch's runs (lanes of the mask: [jb, je) with image code
  // kcs), one run after the other.
  __device__ __forceinline__ void scan(unsigned long long runs, uint32_t jb, uint32_t je, int kcs) {
    while (runs) {
      const int s = (int)__builtin_ctzll(runs);
      runs &= runs - 1ull;
      const uint32_t rb = (uint32_t)__builtin_amdgcn_readlane((int)jb, s);
      const uint32_t re = (uint32_t)__builtin_amdgcn_readlane((int)je, s);
      const int kc = __builtin_amdgcn_readlane(kcs, s);
      double o[3] = {0.0, 0.0, 0.0};
#pragma unroll
      for (int a = 0; a < DIM; ++a) o[a] = (ldu(&J->tK[(kList ? kc & 31 : kc) * 4 + a]) - O[a]) * scale;
      // FP32 lists need every candidate's cell: the ends of the run's cells,
      // one per lane, and for each candidate the number of ends up to it (long
      // runs: a search)
      uint32_t cend = 0u;
      int ncell = 0, cell0 = 0, ux0 = 0;
      if constexpr (kList && !F64) {
        ux0 = __builtin_amdgcn_readlane(l_ux, s);
        ncell = __builtin_amdgcn_readlane(l_nc, s);
        cell0 = __builtin_amdgcn_readlane(l_cell, s);
        if (lane < ncell) cend = OFFJ[cell0 + lane + 1];
      }
      for (uint32_t cb = rb; cb < re; cb += kWave) {
        const uint32_t j = cb + (uint32_t)lane;
        const bool valid = j < re;
        const uint32_t jj = valid ? j : re - 1u;
        if constexpr (kList && !F64) {
          int k = 0;
          if (ncell <= kWave) {
            for (int i = 0; i < ncell; ++i) k += jj >= (uint32_t)__builtin_amdgcn_readlane((int)cend, i) ? 1 : 0;
          } else {
            for (int e = ncell - 1; k < e;) {
              const int m = (k + e) / 2;
              if (jj >= OFFJ[cell0 + m + 1]) k = m + 1;
              else e = m;
            }
          }
          test(valid, jj, kc, o, ux0 + k);
        } else {
          test(valid, jj, kc, o);
        }
      }
    }
  }

  // The same where the runs are short (few particles in a cell): 64 candidates
  // from as many runs as it takes (the runs in L->run_*, total candidates in
  // all), for an LDS look-up each.
  __device__ __forceinline__ void scan_flat(uint32_t total, int kcs) {
    double o0[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int a = 0; a < DIM; ++a) o0[a] = -O[a] * scale;
    int n = 0;  // this lane's run
    for (uint32_t cb = 0; cb < total; cb += kWave) {
      const bool valid = cb + (uint32_t)lane < total;
      const uint32_t p = valid ? cb + (uint32_t)lane : total - 1u;
      while (p >= L->run_end[n]) ++n;
      int kc = L->run_kc[n], ux = 0;
      if constexpr (kList && !F64) {
        // the candidate's cell: the first of the run's that ends beyond it
        const int src = kc;
        kc = __shfl(kcs, src, kWave);
        const int cell0 = __shfl(l_cell, src, kWave);
        int k = 0;
        for (int e = __shfl(l_nc, src, kWave) - 1; k < e;) {
          const int m = (k + e) / 2;
          if (p + L->run_delta[n] >= OFFJ[cell0 + m + 1]) k = m + 1;
          else e = m;
        }
        ux = __shfl(l_ux, src, kWave) + k;
      }
      double o[3] = {o0[0], o0[1], o0[2]};
      const int im = kList ? kc & 31 : kc;
      if (__builtin_amdgcn_ballot_w64(im != kHere)) {
#pragma unroll
        for (int a = 0; a < DIM; ++a) o[a] = (tks[im * 3 + a] - O[a]) * scale;
      }
      test(valid, p + L->run_delta[n], kc, o, ux);
    }
  }

  // ------------------------------------------------------------ the group
  // Rows r (in visiting order) with r % ngrp == grp.  Cross sets and forces
  // visit the whole stencil, the other maps its half shell.
  __device__ __forceinline__ void run(const Tile& T, int g, int grp, int ngrp) {
    cross = ldu(&J->cross);
    const int l = ldu(&J->lcell), lx = ldu(&J->lcell_x);
    const int nx = ldu(&J->n[0]), ny = ldu(&J->n[1]), nz = ldu(&J->n[2]);
    gs = T.start + (uint32_t)(kGrp * g);
    gc = min((int)T.count - kGrp * g, kGrp);
    c = lane & 15;
    q = lane >> 4;
    rc2 = ldu(&J->rc2);
    scale = ldu(&J->grp_scale);
    R = cross ? ldu(&J->r64_y) : ldu(&J->r64_x);
    IDXJ = cross ? ldu(&J->idx_y) : ldu(&J->idx_x);
    if constexpr (kVel) VJ64 = cross ? ldu(&J->vel64_y) : ldu(&J->vel64_x);
    const uint32_t* OFF = cross ? ldu(&J->off_y) : ldu(&J->off_x);

    // the group's origin (box centre) and box; lane (q, c) works on particle c
    const bool act = c < gc;
    uint32_t sl = (uint32_t)min(c, gc - 1);  // the lane's particle in the group
    if constexpr (kVL) {
      sl = vl_order(ldu(&J->r64_x)[gs + sl], sl);
      if (lane < kGrp) vslot[lane] = sl;
    }
    const double4 ri = ldu(&J->r64_x)[gs + sl];
    const double4 r0 = ldu(&J->r64_x)[gs];
    {
      const double d[3] = {ri.x - r0.x, ri.y - r0.y, ri.z - r0.z};
      const double o[3] = {r0.x, r0.y, r0.z};
#pragma unroll
      for (int a = 0; a < DIM; ++a) {
        const float y = (float)d[a];
        O[a] = o[a] + 0.5 * ((double)uniform_f(min16(y)) + (double)uniform_f(max16(y)));
      }
    }
    double o0[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int a = 0; a < DIM; ++a) o0[a] = -O[a] * scale;
    const float4 xi = rel(ri, o0);
    const bool full = kLJF || kRows || cross;
    bl[0] = uniform_f(min16(xi.x)); bh[0] = uniform_f(max16(xi.x));
    bl[1] = uniform_f(min16(xi.y)); bh[1] = uniform_f(max16(xi.y));
    if (DIM == 3) { bl[2] = uniform_f(min16(xi.z)); bh[2] = uniform_f(max16(xi.z)); }
    {
      const float rcs = ldu(&J->grp_rc), e64 = ldu(&J->grp_e64);
      const float S = 2.0f * __builtin_sqrtf(uniform_f(max16(xi.w))) * 1.000001f + 1.01f * rcs;
      const float band = 24.0f * 5.9604645e-8f * S * S + e64;
      const float rcs2 = rcs * rcs;
      lo = uniform_f(rcs2 - band);
      hi = uniform_f(rcs2 + band);
      test_hi = hi;
      if constexpr (!kMfma && !F64) {
        // quanta: S < 2^e, so coordinates stay below 2^29 and differences
        // below 2^30 for every pair of the box test
        // (the cutoff is at least 2^-30 units: iq^2 and the thresholds are FP32
        // numbers whatever the caller's unit)
        const int e = (int)((__builtin_bit_cast(uint32_t, S) >> 23) & 255u) - 126;
        iq = uniform_d(__builtin_ldexp(1.0, 29 - e));
        const float iq2 = (float)(iq * iq);
        unit = KIND == K_SUM_D ? 1.0 / (iq * scale) : iq * scale;
        if constexpr (kLJ) {
          const double s2q = ldu(&J->s2) * (scale * scale) * (iq * iq);
          sig2 = uniform_f((float)s2q);
          near2 = ldu(&J->half_near2) * sig2;
          unit = 1.0 / (ldu(&J->s2) * (iq * scale));
          wunit = 0.5 / (ldu(&J->s2) * (iq * scale) * (iq * scale));
        }
        // u = 2^-24: a component's difference is off by a quantum, at most u S / 16
        // (2 sqrt(3) u S rc / 16 = 0.217 u S rc in d^2), and rounded once (2 u
        // rc^2), d^2 three times (3 u rc^2), the cutoff in this unit, its square
        // and the threshold once each (2 + 1 + 1 u rc^2): 9 u rc^2 and 0.217 u S rc
        const float b = 5.9604645e-8f * (10.0f * rcs2 + 0.25f * S * rcs) + e64;
        lo = uniform_f((rcs2 - b) * iq2);
        hi = uniform_f((rcs2 + b) * iq2);
      }
      if constexpr (kHist) {
        nbins = ldu(&J->nbins);
        if constexpr (!kF64) E64 = ldu(&J->E64);
        inv_h64 = (double)nbins / ldu(&J->hist_hi);
        inv_h32 = (float)inv_h64;
        want_sums = ldu(&J->want_sums);
        // v is within bv of the true value, so u is within bv / sqrt(v)
        // (|sqrt(v) - sqrt(v')| = |v - v'| / (sqrt(v) + sqrt(v'))) and a few
        // units of its own; beyond the last bin the error of a speed grows
        // with the speed: E bounds it in bin widths
        float bv = band;
        if constexpr (kRel) {
          const double ih = inv_h64 * inv_h64;
          ih2 = (float)ih;
          bv = (float)(ldu(ldu(&J->bandq)) * ih * 1.0001);
        }
        const float nf = (float)nbins;
        const float E = fminf(bv / (4.04f * nf), __builtin_sqrtf(0.5f * bv));
        c1 = uniform_f(1.0001f * bv);
        c3 = 0.5f - 1e-6f * (nf + 2.0f);
        first = uniform_f(0.98f - bv);
        over = uniform_f(1.0001f * (E + __builtin_sqrtf(nf * nf + bv + 2.0f * E * E)) + 0.5f);
      }
    }
    // matrix operand and rows
    if constexpr (kMfma) {
      const float v = q == 0 ? -2.0f * xi.x : (q == 1 ? -2.0f * xi.y : (q == 2 ? -2.0f * xi.z : 1.0f));
      a_op = act ? v : 0.0f;
      const float n2 = act ? xi.w : kFar;
#pragma unroll
      for (int r = 0; r < 4; ++r) cn[r] = from_lane(n2, 4 * q + r);
    } else {
      Real x0, y0, z0;
      if constexpr (F64) {
        x0 = act ? ri.x : -1e100;
        y0 = ri.y;
        z0 = ri.z;
      } else {
        const int4 v = quanta(ri, o0);
        x0 = act ? v.x : -kFarQ;
        y0 = v.y;
        z0 = v.z;
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        xr[r][0] = __shfl(x0, 4 * q + r, kWave);
        xr[r][1] = __shfl(y0, 4 * q + r, kWave);
        xr[r][2] = DIM == 3 ? __shfl(z0, 4 * q + r, kWave) : (Real)0;
        acc[r] = 0.0f;
      }
      if constexpr (kW) {
#pragma unroll
        for (int r = 0; r < 4; ++r) wr[r] = __shfl(ri.w, 4 * q + r, kWave);
      }
    }
    if constexpr (kLJ) s2 = ldu(&J->s2);
    if constexpr (kLJF) {
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          if constexpr (!F64) f32[r][a] = 0.0f;
          fr[r][a] = 0.0;
        }
      if constexpr (!F64) {
        if (lane < kGrp * 3)
#pragma unroll
          for (int z = 0; z < kGaCopies; ++z) L->ga[z][lane] = 0.0;
        __builtin_amdgcn_wave_barrier();
      }
    }
    if constexpr (kVel) {
      const float4 v = ldu(&J->vel32_x)[gs + (uint32_t)min(c, gc - 1)];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        vr[r][0] = from_lane(v.x, 4 * q + r);
        vr[r][1] = from_lane(v.y, 4 * q + r);
        vr[r][2] = DIM == 3 ? from_lane(v.z, 4 * q + r) : 0.0f;
      }
    }
    if constexpr (kRows && !kVL) {
      const uint32_t io = ldu(&J->idx_x)[gs + (uint32_t)min(c, gc - 1)];
      // (no candidate's index is larger than that of an empty row)
      const uint32_t iv = act ? io : 0xffffffffu;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        ir[r] = (uint32_t)__shfl((int)iv, 4 * q + r, kWave);
        cr[r] = 0u;
      }
    }
    const int cy = (int)(T.row % (uint32_t)ny);
    const int cz = DIM == 3 ? (int)(T.row / (uint32_t)ny) : 0;
    int cxi = 0;  // this lane's particle's cell along the row
    if constexpr (kList) {
      nst = 0;
      OFFJ = OFF;
      gcy = cy;
      gcz = cz;
      if constexpr (!F64) {
        cxi = T.cx0;
        const uint32_t* ends = ldu(&J->off_x) + (size_t)T.row * nx + 1;
        for (int k = T.cx0; k < T.cx1; ++k) cxi += gs + (uint32_t)min(c, gc - 1) >= ends[k] ? 1 : 0;
      }
      if constexpr (KIND == K_ROW_LIST)
        with_cut = __builtin_amdgcn_ballot_w64(roff[lane & (kGrp - 1)] == kCutRow) != 0ull;
      if (lane < kGrp) {
        L->ri[lane][0] = ri.x;
        L->ri[lane][1] = ri.y;
        L->ri[lane][2] = ri.z;
        if constexpr (!F64) {
          float4 p = ldu(&J->pos_x)[gs + (uint32_t)min(c, gc - 1)];
          p.w = __builtin_bit_cast(float, cxi);
          L->posi[lane] = p;
        }
      }
      __builtin_amdgcn_wave_barrier();
    }
    qtail = 0;
    head = 0;
    fill = 0;
    img = 0;
    unfolded = 0;

    // the group's cells along the row: from its fractional coordinates, one
    // cell wider where rounding could matter, within the tile's cells
    int gx0, gx1;
    {
      double f = ldu(&J->hinv0[0]) * ri.x + ldu(&J->hinv0[1]) * ri.y;
      if (DIM == 3) f = f + ldu(&J->hinv0[2]) * ri.z;
      f *= (double)nx;
      gx0 = max((int)T.cx0, uniform(min16i((int)floor(f - 1e-6))));
      gx1 = min((int)T.cx1, uniform(max16i((int)floor(f + 1e-6))));
      if (gx0 > gx1) { gx0 = T.cx0; gx1 = T.cx1; }
    }
    // neighbour rows in visiting order: half shell (home row first, then
    // (dz, dy) > 0) or all; each row's stencil is at most two runs of cells
    // (the range is no longer than the row), and the own row of a full stencil
    // leaves out the group: three
    const int side = 2 * l + 1;
    const int nrow = full ? (DIM == 3 ? side * side : side) : half_rows(DIM, l);
    const int own = cross ? -1 : (full ? nrow / 2 : 0);
    const int mine = nrow > grp ? (nrow - grp + ngrp - 1) / ngrp : 0;  // rows grp, grp + ngrp, ...
    if (!cross && own % ngrp == grp) {  // the group against itself
      push(lane < gc, xi, ri, o0, gs + (kVL ? sl : (uint32_t)lane), row_code(kHere, 0, 0), cxi);
      block<true, false>(0, gc);
      fill = 0;
      unfolded = 1;
    }
    constexpr int kPer = kLJF || kRows ? 3 : 2;  // runs of a row
    constexpr int kBatch = kWave / kPer;
    for (int base = 0; base < mine; base += kBatch) {
      // lane kPer k + p: run p of row grp + (base + k) ngrp
      uint32_t jb = 0, je = 0;
      int kc = kHere;
      if constexpr (kList && !F64) l_ux = l_cell = l_nc = 0;
      {
        const int k = base + lane / kPer, p = lane % kPer;
        if (k < mine && lane < kBatch * kPer) {
          const int r = grp + k * ngrp;
          int dy, dz;
          if (full) {
            dy = r % side - l;
            dz = DIM == 3 ? r / side - l : 0;
          } else if (r <= l) {
            dy = r;
            dz = 0;
          } else {
            dz = 1 + (r - l - 1) / side;
            dy = (r - l - 1) % side - l;
          }
          int uy = cy + dy, uz = cz + dz, py = 0, pz = 0;
          if (uy < 0) { uy += ny; py = -1; } else if (uy >= ny) { uy -= ny; py = 1; }
          if (DIM == 3) {
            if (uz < 0) { uz += nz; pz = -1; } else if (uz >= nz) { uz -= nz; pz = 1; }
          }
          const int rowbase = (uy + ny * uz) * nx;
          const bool home = r == own;
          const int xlo = home && !full ? gx0 : gx0 - lx, xhi = gx1 + lx;
          // p = 0: the cells of the row itself; p = 1: what wraps around; of
          // the own row p = 0 is the part after the group, p = 2 that before
          int a0, a1, px;
          if (p != 1) { a0 = max(xlo, 0); a1 = min(xhi, nx - 1); px = 0; }
          else if (xlo < 0) { a0 = xlo; a1 = min(xhi, -1); px = -1; }
          else { a0 = max(xlo, nx); a1 = xhi; px = 1; }
          if (a0 <= a1 && (p != 2 || home)) {
            jb = OFF[rowbase + a0 - px * nx];
            je = OFF[rowbase + a1 - px * nx + 1];
            if constexpr (kList && !F64) {
              l_ux = a0;
              l_cell = rowbase + a0 - px * nx;
              l_nc = a1 - a0 + 1;
            }
            if (home && p == 0) jb = gs + (uint32_t)gc;
            if (home && p == 2) je = gs;
            kc = row_code(kcode(px, py, pz), dy, dz);
          }
        }
      }
      const uint32_t len = jb < je ? je - jb : 0u;
      uint32_t end = len;
#pragma unroll
      for (int d = 1; d < kWave; d <<= 1) {
        const uint32_t v = __shfl_up(end, d, kWave);
        if (lane >= d) end += v;
      }
      const unsigned long long runs = __builtin_amdgcn_ballot_w64(len != 0u);
      const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)end, kWave - 1);
      // (forces: one copy of the blocks' code, for the registers' sake)
      if (kLJF || total < (uint32_t)(kFlatRun * __popcll(runs))) {
        if (len != 0u) {
          const int k = lane_rank(runs);
          L->run_end[k] = end;
          L->run_delta[k] = jb - (end - len);
          L->run_kc[k] = (uint8_t)(kList && !F64 ? lane : kc);
        }
        __builtin_amdgcn_wave_barrier();
        scan_flat(total, kc);
        __builtin_amdgcn_wave_barrier();
      } else {
        scan(runs, jb, je, kc);
      }
    }
    if constexpr (!kF64 && !kList) {
      if (qtail >= (uint32_t)kWave) drain(false);
    }
    if (fill != 0u) block<false, kLJF || kF64>(head, (int)fill);
    fold();
    if constexpr (!kF64 && !kList) drain(true);
  }
};

// Forces of the block's groups (ng groups of nsub waves): the lanes' sums of
// every row, then the waves', in a fixed order; the wrap term of the box
// gradient; the block's box gradient and virial into its partial slot Pp.
template <int DIM, int KIND, bool F64>
__device__ __forceinline__ void finish_forces(Group<DIM, KIND, F64>& S, uint32_t start, int count, int ng,
                                              int nsub, bool ran, double (*sF)[kGrp * 3], double (*sP)[18],
                                              double* Pp) {
  const JobDesc* J = S.J;
  const int lane = S.lane, wid = (int)threadIdx.x / kWave, c = lane & 15, q = lane >> 4;
  if (ran) {
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        double v = 0.0;
        if (a < DIM) {
          v = sum16(S.fr[r][a]);
          if constexpr (!F64) {
            v *= S.unit;
#pragma unroll
            for (int z = 0; z < kGaCopies; ++z) v += S.L->ga[z][(4 * q + r) * 3 + a];
          }
        }
        if (c == 0) sF[wid][(4 * q + r) * 3 + a] = v;
      }
  }
  __syncthreads();
  if (wid == 0 && lane < kGrp * ng && lane < count) {
    const int g = lane / kGrp;
    double G[3] = {0.0, 0.0, 0.0};
    for (int z = 0; z < nsub; ++z)
#pragma unroll
      for (int a = 0; a < DIM; ++a) G[a] += sF[g + ng * z][(lane % kGrp) * 3 + a];
    const uint32_t i = start + (uint32_t)lane;
    const double* up = ldu(&J->upstream);
    const double sc = (up ? ldu(up) : ldu(&J->scale)) * 24.0 * ldu(&J->eps);
    double* out = ldu(&J->forces) + (size_t)ldu(&J->idx_x)[i] * DIM;
#pragma unroll
    for (int a = 0; a < DIM; ++a) out[a] = sc * G[a];
    const int4 w = ldu(&J->wrap_x)[i];
    const double wv[3] = {(double)w.x, (double)w.y, (double)w.z};
#pragma unroll
    for (int a = 0; a < DIM; ++a)
#pragma unroll
      for (int b = 0; b < DIM; ++b) S.B[a * 3 + b] += G[a] * wv[b];
  }
  bool some = false;  // most groups touch no image and no wrapped particle
#pragma unroll
  for (int k = 0; k < 9; ++k) some = some || S.B[k] != 0.0;
  const bool any = __builtin_amdgcn_ballot_w64(some) != 0ull;
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    const double v = any ? wave_sum_d(S.B[k]) : 0.0;
    if (lane == 0) sP[wid][k] = v;
  }
  if constexpr (KIND == K_LJ_FV) {
    constexpr int map[9] = {0, 1, 2, 1, 3, 4, 2, 4, 5};
    double ws[6];
#pragma unroll
    for (int k = 0; k < 6; ++k) ws[k] = wave_sum_d(S.W[k]);
#pragma unroll
    for (int k = 0; k < 9; ++k)
      if (lane == 0) sP[wid][9 + k] = ws[map[k]];
  }
  __syncthreads();
  if (threadIdx.x < 9) {
    const int k = (int)threadIdx.x;
    Pp[P_BOX + k] = ((sP[0][k] + sP[1][k]) + sP[2][k]) + sP[3][k];
    if constexpr (KIND == K_LJ_FV)
      if (k < 3 || (k > 3 && k != 6 && k != 7))  // the upper triangle: the others hold counts
        Pp[P_VIR + k] = ((sP[0][9 + k] + sP[1][9 + k]) + sP[2][9 + k]) + sP[3][9 + k];
  }
}

// The same for a wave's group: its rows' forces and the wrap term.
template <int DIM, int KIND, bool F64>
__device__ __forceinline__ void write_forces(Group<DIM, KIND, F64>& S, uint32_t start, int count) {
  const JobDesc* J = S.J;
  const int c = S.lane & 15, q = S.lane >> 4;
  double G[3] = {0.0, 0.0, 0.0};  // lane (q, c < 4): of row 4q + c
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int a = 0; a < DIM; ++a) {
      double v = sum16(S.fr[r][a]);
      if constexpr (!F64) {
        v *= S.unit;
#pragma unroll
        for (int z = 0; z < kGaCopies; ++z) v += S.L->ga[z][(4 * q + r) * 3 + a];
      }
      G[a] = c == r ? v : G[a];
    }
  if (c < 4 && 4 * q + c < count) {
    const uint32_t i = start + (uint32_t)(4 * q + c);
    const double* up = ldu(&J->upstream);
    const double sc = (up ? ldu(up) : ldu(&J->scale)) * 24.0 * ldu(&J->eps);
    double* out = ldu(&J->forces) + (size_t)ldu(&J->idx_x)[i] * DIM;
    const int4 w = ldu(&J->wrap_x)[i];
    const double wv[3] = {(double)w.x, (double)w.y, (double)w.z};
#pragma unroll
    for (int a = 0; a < DIM; ++a) {
      out[a] = sc * G[a];
#pragma unroll
      for (int b = 0; b < DIM; ++b) S.B[a * 3 + b] += G[a] * wv[b];
    }
  }
  __builtin_amdgcn_wave_barrier();
}

// And its box gradient and virial, summed over the wave, into the slot Pp.
template <int DIM, int KIND, bool F64>
__device__ __forceinline__ void write_tensors(const Group<DIM, KIND, F64>& S, double* Pp) {
  bool some = false;
#pragma unroll
  for (int k = 0; k < 9; ++k) some = some || S.B[k] != 0.0;
  const bool any = __builtin_amdgcn_ballot_w64(some) != 0ull;
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    const double v = any ? wave_sum_d(S.B[k]) : 0.0;
    if (S.lane == 0) Pp[P_BOX + k] = v;
  }
  if constexpr (KIND == K_LJ_FV) {
    constexpr int slot[6] = {0, 1, 2, 4, 5, 8};  // (the upper triangle)
#pragma unroll
    for (int k = 0; k < 6; ++k) {
      const double v = wave_sum_d(S.W[k]);
      if (S.lane == 0) Pp[P_VIR + slot[k]] = v;
    }
  }
}

}  // namespace

// Sparse boxes: tiles end after kMaxSpan cells, however few particles they
// hold, and four waves of a block have no work to share.  10^6 particles at
// 0.3 a unit volume, count, block / wave per tile: cutoff 1 (1.2 neighbours)
// 2516 / 1387 us, 2 907 / 490, 3 (33 neighbours, above kSoloParticles a tile)
// 390 / 450.  (Without the blocks that find no item, as below: 810, 380, 360.)
// FP64 forces of 10^6 particles at cutoff 1 5302 / 2556 us, at 2 1911 / 1137.
__device__ __forceinline__ bool sparse_tiles(const Tile* tiles, int ntiles) {
  const Tile z = ldu(&tiles[ntiles - 1]);
  return (long long)z.start + (long long)z.count <= (long long)kSoloParticles * ntiles;
}

// What the list's readers find of four rows: candidates and the rows' particles
// of the group (an integer below 2^53).
__device__ __forceinline__ double vl_word(uint32_t candidates, const uint32_t* slots) {
  uint64_t w = (uint64_t)candidates << 16;
  for (int r = 0; r < kVlRows; ++r) w |= (uint64_t)(slots[r] & 15u) << (4 * r);
  return (double)w;
}

// Blocks per CU the registers are budgeted for (= waves per SIMD).  2D forces of
// the FP32 form have the registers for one more (14 spilled outside the loop):
// 10^6 points at 2000 neighbours 2.64 -> 2.33 ms, with the virial 3.52 -> 2.95.
constexpr int group_blocks(int dim, int kind, bool f64) {
  const int flat = dim == 2 && !f64 ? 1 : 0;
  return kind == K_LJ_FV ? 3 + flat : (kind == K_LJ_F ? 4 + flat
                                                      : (kind == K_COUNT || (kind == K_HIST_DIST && !f64) ? 6 : 5));
}

// solo: the sparse form, an item to each wave of a block instead of one to the
// block (a kernel of its own: the loop over a tile's groups costs the blocks'
// form registers).  maybe_sparse: both forms are launched, and one returns.
template <int DIM, int KIND, bool F64, bool solo>
__global__ void __launch_bounds__(kGWaves * kWave, group_blocks(DIM, KIND, F64)) group_kernel(const JobDesc* __restrict__ jobs,
                                                                const Tile* __restrict__ tiles,
                                                                const uint32_t* __restrict__ ntiles_dev,
                                                                int split_rows, int cap, bool maybe_sparse,
                                                                const uint32_t* __restrict__ gate) {
  if constexpr (KIND == K_VLIST)
    if (ldu(gate) == 0u) return;
  constexpr bool kHist = KIND == K_HIST_DIST || KIND == K_HIST_REL || KIND == K_HIST_DV;
  constexpr bool kLJF = group_ljf(KIND), kRows = group_rows(KIND);
  constexpr bool kOwn = kLJF || kRows;  // the block writes per-particle results
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ GroupLds<KIND, F64> lds[kGWaves];
  __shared__ double tks[27 * 3];
  __shared__ double red_e[kGWaves];
  __shared__ unsigned long long red_c[kGWaves];
  __shared__ uint32_t red_g[kGWaves][2];
  const int lane = (int)__lane_id();
  const int wid = uniform((int)(threadIdx.x / kWave));
  const int ntiles = min((int)ldu(ntiles_dev), cap);
  // items: a tile, a tile and every G-th of its neighbour rows, or (forces of
  // few tiles) one of the four groups of a tile
  const int G = item_split(ntiles, cap, split_rows);
  const int nitems = ntiles * G;
  if (maybe_sparse && (nitems >= kSoloItems && sparse_tiles(tiles, ntiles) && (!kOwn || G == 1)) != solo) return;
  const int nblocks = solo ? (nitems + kGWaves - 1) / kGWaves : nitems;
  int b = blockIdx.x;
  if (b >= nblocks) return;
  if (nblocks >= 8) {  // each XCD (block mod 8) a contiguous range of items
    const int per = nblocks / 8, rem = nblocks % 8;
    const int xcd = b % 8, k = b / 8;
    b = (xcd < rem ? xcd * (per + 1) : rem * (per + 1) + (xcd - rem) * per) + k;
  }
  const int item = solo ? min(b * kGWaves + wid, nitems - 1) : b;
  const bool mine = !solo || b * kGWaves + wid < nitems;
  const int tile_id = item / G, part = item - tile_id * G;
  const Tile T = ldu(&tiles[tile_id]);

  Group<DIM, KIND, F64> S;
  S.J = &jobs[T.job];
  S.L = &lds[wid];
  S.tks = tks;
  S.lane = lane;
  S.accE = 0.0;
  S.cnt_wave = 0;
  S.qband = 0;
  S.qnear = 0;
#pragma unroll
  for (int k = 0; k < 9; ++k) S.B[k] = 0.0;
#pragma unroll
  for (int k = 0; k < 6; ++k) S.W[k] = 0.0;
  for (int k = threadIdx.x; k < 27 * 3; k += kGWaves * kWave) tks[k] = S.J->tK[(k / 3) * 4 + k % 3];
  int nb = 0, lgC = 0;
  uint32_t* hist = nullptr;
  double* hsum = nullptr;
  if constexpr (kHist) {
    nb = ldu(&S.J->nbins);
    lgC = hist_lgC(KIND, nb);
    const int nh = (nb + 1) << lgC;
    unsigned char* base = smem;
    if constexpr (F64) {  // the edges
      double* E = (double*)base;
      const double* Eg = ldu(&S.J->E64);
      for (int k = threadIdx.x; k <= nb; k += kGWaves * kWave) E[k] = Eg[k];
      S.E64 = E;
      base += (size_t)(nb + 1) * 8;
    }
    hsum = (double*)base;
    hist = (uint32_t*)(base + (hist_has_sums(KIND) ? (size_t)nh * 8 : 0));
    for (int k = threadIdx.x; k < nh; k += kGWaves * kWave) {
      hist[k] = 0u;
      if constexpr (hist_has_sums(KIND)) hsum[k] = 0.0;
    }
    const int copy = (int)threadIdx.x & ((1 << lgC) - 1);
    S.hist = hist + copy;
    S.hsum = hsum + copy;
    S.lgC = lgC;
  }
  __syncthreads();
  // group of this wave; where the block has fewer groups than waves, several
  // waves share the neighbour rows of one
  const int first = kOwn && G > 1 ? part : 0;  // the block's first group
  const int ngt = ((int)T.count + kGrp - 1) / kGrp;
  const int ng = kOwn && G > 1 ? (first < ngt ? 1 : 0) : ngt;
  // (large Verlet lists: a wave a group, whose order does not vary)
  const bool single = solo || (KIND == K_VLIST && ldu(&S.J->nx) >= kVlOrdered);
  const int nsub = single ? 1 : (ng == 1 ? 4 : (ng == 2 ? 2 : 1));
  int g = ng == 0 || solo ? 0 : (nsub == 1 ? wid : wid % ng);
  const int sub = nsub == 1 ? 0 : wid / max(ng, 1);
  const bool ran = mine && g < ng;
  __shared__ uint32_t rcnt[kRows ? kTileMax : 1];
  __shared__ uint32_t gcnt[KIND == K_VLIST ? 4 * kGWaves : 1], vslot[KIND == K_VLIST ? kTileMax : 1];
  __shared__ unsigned long long roff[KIND == K_ROW_LIST ? kTileMax : 1];
  uint32_t cut = 0u;
  if constexpr (KIND == K_ROW_LIST) cut = ldu(ldu(&S.J->row_cut));
  const auto offset_of = [&](int i) -> unsigned long long {  // of the row of particle i of the tile
    if (i >= (int)T.count) return 0ull;
    const uint32_t io = ldu(&S.J->idx_x)[T.start + (uint32_t)i];
    return io == cut ? kCutRow : ldu(&S.J->row_off)[io];
  };
  if constexpr (kRows) {
    // the counters of group g of the block, or of the wave's group
    S.rcnt = rcnt + kGrp * (solo ? wid : g);
    S.gcnt = gcnt + 4 * (solo ? wid : g);
    S.vslot = vslot + kGrp * (solo ? wid : g);
    if constexpr (KIND == K_ROW_LIST) S.roff = roff + kGrp * (solo ? wid : g);
    if (!solo) {
      const int t = (int)threadIdx.x, i = kGrp * first + t;  // row t of the block's groups
      if (t < kTileMax) {
        rcnt[t] = 0u;
        if (KIND == K_VLIST && t < 4 * kGWaves) gcnt[t] = 0u;
        if constexpr (KIND == K_ROW_LIST) roff[t] = offset_of(i);
      }
      __syncthreads();
    }
  }
  if (ran) {
    do {
      const int i = kGrp * (first + g) + lane;
      if constexpr (kRows) {
        if (solo && lane < kGrp) {
          S.rcnt[lane] = 0u;
          if (KIND == K_VLIST && lane < 4) S.gcnt[lane] = 0u;
          if constexpr (KIND == K_ROW_LIST) roff[kGrp * wid + lane] = offset_of(i);
        }
        __builtin_amdgcn_wave_barrier();
      }
      S.run(T, first + g, kOwn ? sub : part + G * sub, kOwn ? nsub : G * nsub);
      if constexpr (kLJF && solo) write_forces(S, T.start + (uint32_t)(kGrp * g), (int)T.count - kGrp * g);
      if constexpr (KIND == K_ROW_COUNT) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          uint32_t v = S.cr[r];
#pragma unroll
          for (int d = 8; d > 0; d >>= 1) v += __shfl_xor((int)v, d, kWave);
          if ((lane & 15) == 0 && v) atomicAdd(&S.rcnt[4 * (lane >> 4) + r], v);
        }
        __builtin_amdgcn_wave_barrier();
        if (solo && lane < kGrp && i < (int)T.count)
          ldu(&S.J->row_cnt)[ldu(&S.J->idx_x)[T.start + (uint32_t)i]] = S.rcnt[lane];
        __builtin_amdgcn_wave_barrier();
      }
      if constexpr (KIND == K_VLIST) {
        __builtin_amdgcn_wave_barrier();
        if (solo && lane < kGrp && i < (int)T.count) {
          ldu(&S.J->vl_cnt)[T.start + (uint32_t)(i - lane) + S.vslot[lane]] = S.rcnt[lane];
          if (lane % kVlRows == 0)
            ldu(&S.J->vl_pf)[T.start + (uint32_t)i].w = vl_word(S.gcnt[lane / kVlRows], S.vslot + lane);
        }
        __builtin_amdgcn_wave_barrier();
      }
    } while (solo && ++g < ng);
  }
  if constexpr (KIND == K_ROW_COUNT) {
    if (!solo) {
      __syncthreads();
      const int t = (int)threadIdx.x, i = kGrp * first + t;
      if (t < kGrp * ng && i < (int)T.count)
        ldu(&S.J->row_cnt)[ldu(&S.J->idx_x)[T.start + (uint32_t)i]] = rcnt[t];
    }
  }
  if constexpr (KIND == K_VLIST) {
    if (!solo) {
      __syncthreads();
      const int t = (int)threadIdx.x, i = kGrp * first + t;
      if (t < kGrp * ng && i < (int)T.count) {
        ldu(&S.J->vl_cnt)[T.start + (uint32_t)(i - t % kGrp) + vslot[t]] = rcnt[t];
        if (t % kVlRows == 0) ldu(&S.J->vl_pf)[T.start + (uint32_t)i].w = vl_word(gcnt[t / kVlRows], vslot + t);
      }
    }
  }
  if constexpr (KIND == K_ROW_LIST || KIND == K_VLIST) return;  // (pairs: the counting pass)
  const unsigned long long cnt = S.cnt_wave;
  const double e = wave_sum_d(S.accE) * (kLJF && F64 ? 0.5 : 1.0);
  const uint32_t gb = S.qband, gn = S.qnear;
  if (lane == 0) {
    red_c[wid] = cnt;
    red_e[wid] = e;
    red_g[wid][0] = gb;
    red_g[wid][1] = gn;
  }
  const int local = (tile_id - ldu(&S.J->tile_begin)) * G + part;
  double* Pp = ldu(&S.J->partials) + (size_t)local * kPartialD;
  if constexpr (kLJF && !solo) {
    __shared__ double sF[kGWaves][kGrp * 3];
    __shared__ double sP[kGWaves][18];
    finish_forces<DIM, KIND, F64>(S, T.start + (uint32_t)(kGrp * first), (int)T.count - kGrp * first, ng, nsub, ran,
                                  sF, sP, Pp);
  } else {
    __syncthreads();
  }
  if (solo) {
    if constexpr (kLJF && solo)
      if (mine) write_tensors(S, Pp);
    if (lane == 0 && mine) {
      ldu(&S.J->pcount)[local] = cnt;
      Pp[P_SUM] = e;
      Pp[P_STAT0] = (double)gb;
      Pp[P_STAT1] = (double)gn;
      if constexpr (kLJF) {
        Pp[P_STAT2] = 0.0;
        Pp[P_STAT3] = 0.0;
      }
    }
  } else if (threadIdx.x == 0) {
    ldu(&S.J->pcount)[local] = ((red_c[0] + red_c[1]) + red_c[2]) + red_c[3];
    Pp[P_SUM] = ((red_e[0] + red_e[1]) + red_e[2]) + red_e[3];
    // the re-evaluation counts go through the finalize, too: adds of every
    // wave to one address took as long as the sweep
    Pp[P_STAT0] = (double)(red_g[0][0] + red_g[1][0] + red_g[2][0] + red_g[3][0]);
    Pp[P_STAT1] = (double)(red_g[0][1] + red_g[1][1] + red_g[2][1] + red_g[3][1]);
    if constexpr (kLJF) {
      Pp[P_STAT2] = 0.0;
      Pp[P_STAT3] = 0.0;
    }
  }
  if constexpr (kHist) {
    // into one of the job's copies (hist_reduce_kernel adds them up): with
    // one, thousands of blocks' adds to the same addresses took longer than
    // the sweep
    const int rep = (int)(blockIdx.x % (unsigned)ldu(&S.J->hist_reps));
    unsigned long long* gh = ldu(&S.J->hist_rep) + (size_t)rep * (nb + 1);
    double* gsum = ldu(&S.J->hsum_rep) + (size_t)rep * nb;
    const bool sums = KIND == K_HIST_DV || (KIND == K_HIST_REL && ldu(&S.J->want_sums) != 0);
    for (int k = threadIdx.x; k <= nb; k += kGWaves * kWave) {
      uint32_t t = 0u;
      for (int z = 0; z < (1 << lgC); ++z) t += hist[(k << lgC) + z];
      if (t) atomicAdd(&gh[k], (unsigned long long)t);
      if (hist_has_sums(KIND) && sums && k < nb) {
        double sm = 0.0;
        for (int z = 0; z < (1 << lgC); ++z) sm += hsum[(k << lgC) + z];
        if (sm != 0.0) atomicAdd(&gsum[k], sm);
      }
    }
  }
}

// The job's copies of a histogram (and its sums) into its outputs: one wave
// per bin, a copy per lane; block (x, y): bins 4 x .. of job y.
__global__ void __launch_bounds__(256) hist_reduce_kernel(const JobDesc* __restrict__ jobs) {
  const JobDesc& J = jobs[blockIdx.y];
  const int k = (int)(blockIdx.x * 4 + threadIdx.x / kWave), nb = J.nbins;
  const int r = (int)threadIdx.x & (kWave - 1);
  static_assert(kHistReps <= kWave, "one lane per copy");
  if (k > nb) return;
  const bool on = r < J.hist_reps, sums = J.want_sums && k < nb;
  const unsigned long long t = wave_sum_u64(on ? J.hist_rep[(size_t)r * (nb + 1) + k] : 0ull);
  const double sm = wave_sum_d(on && sums ? J.hsum_rep[(size_t)r * nb + k] : 0.0);
  if (r == 0) {
    J.hist[k] = t;
    if (sums) J.hist_sums[k] = sm;
  }
}

template <int DIM, bool F64, bool SOLO>
static hipError_t group_dispatch(int kind, unsigned grid, size_t lds, const JobDesc* jobs, const Tile* tiles,
                                 const uint32_t* nt, int split, int cap, bool sparse, const uint32_t* gate,
                                 hipStream_t s) {
  constexpr int kT = kGWaves * kWave;
#define CLM_GROUP(K, D) group_kernel<DIM, K, D, SOLO><<<grid, kT, lds, s>>>(jobs, tiles, nt, split, cap, sparse, gate)
  switch (kind) {
    case K_SUM_D: CLM_GROUP(K_SUM_D, F64); break;
    case K_SUM_INV_D: CLM_GROUP(K_SUM_INV_D, F64); break;
    case K_SUM_W: CLM_GROUP(K_SUM_W, F64); break;
    case K_LJ_E: CLM_GROUP(K_LJ_E, F64); break;
    case K_LJ_F: CLM_GROUP(K_LJ_F, F64); break;
    case K_LJ_FV: CLM_GROUP(K_LJ_FV, F64); break;
    case K_ROW_LIST: CLM_GROUP(K_ROW_LIST, F64); break;
    case K_VLIST: CLM_GROUP(K_VLIST, true); break;  // canonical FP64 in both forms
    case K_ROW_COUNT: CLM_GROUP(K_ROW_COUNT, F64); break;
    case K_COUNT: CLM_GROUP(K_COUNT, F64); break;
    case K_HIST_DIST: CLM_GROUP(K_HIST_DIST, F64); break;
    case K_HIST_REL:
      if (F64) return hipErrorInvalidValue;
      CLM_GROUP(K_HIST_REL, false);
      break;
    case K_HIST_DV:
      if (F64) return hipErrorInvalidValue;
      CLM_GROUP(K_HIST_DV, false);
      break;
    default: return hipErrorInvalidValue;
  }
#undef CLM_GROUP
  return hipGetLastError();
}

template <bool SOLO>
static hipError_t group_form(int dim, bool fp32, int kind, const JobDesc* jobs, const Tile* tiles,
                             const uint32_t* nt, unsigned g, size_t lds, hipStream_t s, int split, int cap, bool sparse,
                             const uint32_t* gate) {
  if (dim == 3)
    return fp32 ? group_dispatch<3, false, SOLO>(kind, g, lds, jobs, tiles, nt, split, cap, sparse, gate, s)
                : group_dispatch<3, true, SOLO>(kind, g, lds, jobs, tiles, nt, split, cap, sparse, gate, s);
  return fp32 ? group_dispatch<2, false, SOLO>(kind, g, lds, jobs, tiles, nt, split, cap, sparse, gate, s)
              : group_dispatch<2, true, SOLO>(kind, g, lds, jobs, tiles, nt, split, cap, sparse, gate, s);
}

hipError_t launch_group(int dim, bool fp32, int kind, const JobDesc* jobs, const Tile* tiles,
                        const uint32_t* ntiles_dev, int max_tiles, int64_t tile_bound, int nbins, hipStream_t s,
                        int split_rows, int64_t sparse_n, const uint32_t* gate) {
  if (max_tiles <= 0) return hipSuccess;
  const bool hist = kind == K_HIST_DIST || kind == K_HIST_REL || kind == K_HIST_DV;
  const size_t lds = hist ? hist_group_bytes(kind, nbins) + (fp32 ? 0 : sizeof(double) * (size_t)(nbins + 1)) : 0;
  const bool sparse = sparse_n > 0;
  // Blocks for the items there can be (item_split makes more than one of a
  // tile up to kSplitTarget or kSplitGroupBlocks in all): 2 10^5 blocks that find nothing to do take
  // 110 us.
  const auto blocks = [&](int64_t tiles_most) {
    return std::min<int64_t>(max_tiles, std::max<int64_t>(tiles_most, split_rows == kSplitGroups ? kSplitGroupBlocks
                                                                                                 : kSplitTarget));
  };
  const int64_t most = std::min(tile_bound, sparse ? sparse_n / kSoloParticles : tile_bound);
  hipError_t e = group_form<false>(dim, fp32, kind, jobs, tiles, ntiles_dev, (unsigned)blocks(most), lds, s,
                                   split_rows, max_tiles, sparse, gate);
  if (e == hipSuccess && sparse)
    e = group_form<true>(dim, fp32, kind, jobs, tiles, ntiles_dev,
                         (unsigned)((blocks(tile_bound) + kGWaves - 1) / kGWaves), lds, s, split_rows, max_tiles, true, gate);
  return e;
}

hipError_t launch_hist_reduce(const JobDesc* jobs, int njobs, int nbins, hipStream_t s) {
  hist_reduce_kernel<<<dim3((nbins + 4) / 4, njobs), 256, 0, s>>>(jobs);
  return hipGetLastError();
}

}  // namespace clm
