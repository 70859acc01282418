// sweep_group.hip -- the cell-pair sweep for the reduced maps (counts, sums,
// energies, histograms) in groups of 16 particles (paper section 2.8: a cell
// and half of its neighbour cells; sections 2.3/2.7: a function of every pair
// within the cutoff, reduced).
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
// 3.13 -> 0.75 ms (kernel 3.07 -> 0.68 ms, 3.4 10^8 instead of 1.55 10^9
// vector instructions: 0.56 ms of issue), sum of w_i w_j / d 1.34 -> 0.65 ms,
// count 1.16 -> 0.41 ms, LJ energy 1.41 -> 0.60 ms; distance-binned speeds of
// 2 10^6 clustered points in 2D 19.0 -> 7.5 ms; 10^4 particles in the FP64
// form, 128 bins, 0.16 -> 0.10 ms.
//
// Precision: FP32 coordinates are relative to the centre of the group's
// bounding box (formed in FP64, rounded once).  With S = 2 max|x_i| + 1.01 rc
// every coordinate of a pair near the cutoff is at most S, and
//   |d2_32 - d2| <= 2 (1.01 rc) (u S) + 2 u S^2 (coordinates)
//                 + 3 u S^2 (|x_j|^2) + 3 u S^2 (|x_i|^2) + 8 u S^2 (products)
// is below 20 u S^2 (u = 2^-24); the band is 24 u S^2 (room for the roundings
// of rc and of the thresholds) plus the FP64 roundings, the host's term.
// Pairs within that band of rc^2 (histograms: of a bin edge; LJ: closer than
// the near threshold) are queued in LDS and recomputed in canonical FP64, 64
// at a time.  The box test uses the same FP32 coordinates: rounding is
// monotone, so a candidate's distance to the box is at most its distance to
// any particle of it.
#include "clmap_internal.h"
#include "device_util.h"
#include "hist_bins.h"

namespace clm {

namespace {

constexpr int kGrp = 16;      // particles of a group, candidates of a block
constexpr int kGCap = 128;    // candidate ring (power of two, >= 15 + 64)
constexpr int kGQCap = 320;   // FP64 queue (>= 63 + 4 * 64)
constexpr int kGWaves = 4;
constexpr float kFar = 1e30f; // d^2 of an empty row or column

typedef float f32x4 __attribute__((ext_vector_type(4)));

template <int K>
__device__ __forceinline__ float ror16(float v) {
  return __builtin_bit_cast(float,
                            __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x120 + K, 0xF, 0xF, true));
}
template <int K>
__device__ __forceinline__ int ror16i(int v) {
  return __builtin_amdgcn_mov_dpp(v, 0x120 + K, 0xF, 0xF, true);
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
__device__ __forceinline__ float from_lane(float v, int src) {
  return __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(src << 2, __builtin_bit_cast(int, v)));
}

// Square root of a non-negative FP32 value, rounded as by the correctly
// rounded function but for rare last-bit cases; values outside
// [2^-96, 2^96] (zero, infinities and NaN among them) take the library's.
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

// LDS of one wave
template <int KIND>
struct GroupLds {
  static constexpr bool kVel = KIND == K_HIST_REL || KIND == K_HIST_DV;
  float4 lst[kGCap];                 // x, y, z and |x|^2 (weight for K_SUM_W)
  uint2 who[kGCap];                  // sorted index, image code
  float4 vel[kVel ? kGCap : 1];
  uint2 q[kGQCap];                   // FP64 queue
};

template <int DIM, int KIND>
struct Group {
  static constexpr bool kDV = KIND == K_HIST_DV;
  static constexpr bool kRel = KIND == K_HIST_REL;
  static constexpr bool kVel = kDV || kRel;
  static constexpr bool kHist = KIND == K_HIST_DIST || kVel;
  static constexpr bool kW = KIND == K_SUM_W;
  static constexpr bool kSum = KIND == K_SUM_D || KIND == K_SUM_INV_D || kW || KIND == K_LJ_E;
  static constexpr bool kMfma = !kSum;   // d^2 only classifies

  const JobDesc* J;
  GroupLds<KIND>* L;
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
  float near2, s2f;
  int nbins;
  // histogram: the bin of u = sqrt(v) (bin widths) is certain when
  // |fract(u) - 1/2| < c3 - c1 / sqrt(v), or u > over, or v < first (bin 0,
  // zero and coincident values among it)
  float c1, c3, over, first;
  double inv_h64;
  const double* E64;
  const double4* R;
  const uint32_t* IDXJ;
  const double* VJ64;
  int want_sums;
  // per lane
  f32x4 cn;                // |x_i|^2 of rows 4q .. 4q + 3
  float a_op;              // matrix operand A: component q of [-2x, -2y, -2z, 1] of row c
  float xr[4][3];          // coordinates of rows 4q .. 4q + 3
  float vr[4][3];          // velocities
  float acc[4];            // FP32 sums of the rows since the last fold
  double wr[4];            // weights of the rows
  double accE;
  unsigned long long cnt_wave, cnt_lane;
  uint32_t qband, qnear;
  uint32_t qtail, head, tail;

  __device__ __forceinline__ void hist_add(int k) {
    atomicAdd((uint32_t*)((char*)hist + ((uint32_t)k << (lgC + 2))), 1u);
  }
  __device__ __forceinline__ void hsum_add(int k, double v) {
    atomicAdd((double*)((char*)hsum + ((uint32_t)k << (lgC + 3))), v);
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

  // canonical FP64 evaluation of one queued pair
  __device__ __forceinline__ void process(const uint2 e) {
    const uint32_t j = e.x, i = gs + (e.y & 15u);
    const bool count_it = ((e.y >> 16) & 1u) != 0u;
    const double4 rI = ldu(&J->r64_x)[i];
    const double4 rJ = R[j];
    const double* tk = &J->tK[((e.y >> 8) & 31u) * 4];
    double D[3];
    D[0] = (rJ.x - rI.x) + tk[0];
    D[1] = (rJ.y - rI.y) + tk[1];
    double d2 = D[0] * D[0] + D[1] * D[1];
    if (DIM == 3) {
      D[2] = (rJ.z - rI.z) + tk[2];
      d2 = d2 + D[2] * D[2];
    }
    if (!(d2 <= rc2)) return;
    if (count_it) cnt_lane += 1;
    if constexpr (KIND == K_SUM_D) accE += sqrt(d2);
    if constexpr (KIND == K_SUM_INV_D) accE += 1.0 / sqrt(d2);
    if constexpr (kW) accE += (rI.w * rJ.w) / sqrt(d2);
    if constexpr (KIND == K_LJ_E) {
      const double x = s2 * rcp64(d2);
      const double x3 = x * x * x;
      accE += x3 * x3 - x3;
    }
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
  }

  __device__ __forceinline__ void drain(bool all) {
    uint32_t h = 0;
    const uint32_t tl = (uint32_t)uniform((int)qtail);
    while (tl - h >= (uint32_t)kWave || (all && tl != h)) {
      const uint32_t nb = min(tl - h, (uint32_t)kWave);
      if ((uint32_t)lane < nb) {
        const uint2 e = L->q[h + (uint32_t)lane];
        const uint32_t b = (e.y >> 16) & 1u;
        qband += b;
        qnear += 1u - b;
        process(e);
      }
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
    qtail += (uint32_t)__popcll(m);
  }

  // ------------------------------------------------------------ one block
  // Ring slots [pos, pos + nv) (nv <= 16, pos a multiple of 16) against the
  // group; SELF: the group against itself, pairs column > row.
  template <bool SELF>
  __device__ __forceinline__ void block(uint32_t pos, int nv) {
    const uint32_t s = (pos & (uint32_t)(kGCap - 1)) + (uint32_t)c;
    const bool have = c < nv;
    f32x4 d;
    float4 xj = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if constexpr (kMfma) {
      // operand B of lane (q, c): component q of [x, y, z, |x|^2] of candidate c
      const float b = ((const float*)&L->lst[s])[q];
      const float bb = have ? b : (q == 3 ? kFar : 0.0f);
      d = __builtin_amdgcn_mfma_f32_16x16x4f32(a_op, bb, cn, 0, 0, 0);
    } else {
      xj = L->lst[s];
      if (!have) xj.x = 1e18f;
    }
    float4 vj = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if constexpr (kVel) vj = L->vel[s];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float d2;
      if constexpr (kMfma) {
        d2 = d[r];
      } else {
        const float dx = xj.x - xr[r][0], dy = xj.y - xr[r][1];
        const float dz = DIM == 3 ? xj.z - xr[r][2] : 0.0f;
        d2 = DIM == 3 ? __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, dx * dx))
                      : __builtin_fmaf(dy, dy, dx * dx);
      }
      unsigned long long ok = ~0ull;
      if constexpr (SELF) ok = __builtin_amdgcn_ballot_w64(c > 4 * q + r);
      const unsigned long long mlo = __builtin_amdgcn_ballot_w64(d2 <= lo) & ok;
      const unsigned long long mhi = __builtin_amdgcn_ballot_w64(d2 <= hi) & ok;
      cnt_wave += (unsigned long long)__popcll(mlo);
      unsigned long long spec = mhi & ~mlo;
      const unsigned long long band = spec;
      if constexpr (KIND == K_SUM_D || KIND == K_SUM_INV_D || kW) {
        const bool in = __builtin_amdgcn_inverse_ballot_w64(mlo);
        // (coincident particles: d = 0, not 0 times infinity)
        const float rs = __builtin_amdgcn_rsqf(KIND == K_SUM_D ? fmaxf(d2, 1e-37f) : d2);
        const float t = KIND == K_SUM_D ? d2 * rs : (kW ? xj.w * rs : rs);
        acc[r] += in ? t : 0.0f;
      }
      if constexpr (KIND == K_LJ_E) {
        const unsigned long long near = __builtin_amdgcn_ballot_w64(d2 < near2) & ok;
        spec |= near;
        const bool fast = __builtin_amdgcn_inverse_ballot_w64(mlo & ~near);
        const float x = fast ? s2f * __builtin_amdgcn_rcpf(d2) : 0.0f;
        const float x3 = x * x * x;
        acc[r] += __builtin_fmaf(x3, x3, -x3);
      }
      if constexpr (kHist) {
        float v = d2;
        float qq = 0.0f;
        if constexpr (kVel) {
          const float ex = vj.x - vr[r][0], ey = vj.y - vr[r][1];
          const float ez = DIM == 3 ? vj.z - vr[r][2] : 0.0f;
          qq = DIM == 3 ? __builtin_fmaf(ez, ez, __builtin_fmaf(ey, ey, ex * ex))
                        : __builtin_fmaf(ey, ey, ex * ex);
          if constexpr (kRel) v = qq * s2f;  // (1 / bin width)^2
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
      if (spec) enqueue(spec, band, r, have ? L->who[s] : make_uint2(0u, 0u));
    }
    if (qtail >= (uint32_t)kWave) drain(false);
  }

  __device__ __forceinline__ void fold() {
    if constexpr (kSum) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        accE += kW ? wr[r] * (double)acc[r] : (double)acc[r];
        acc[r] = 0.0f;
      }
    }
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

  // lanes of m append candidate (x, j, kc) to the ring
  __device__ __forceinline__ void push(bool keep, float4 x, double w, uint32_t j, int kc) {
    const unsigned long long m = __builtin_amdgcn_ballot_w64(keep);
    if (keep) {
      const uint32_t s = (tail + (uint32_t)lane_rank(m)) & (uint32_t)(kGCap - 1);
      if constexpr (kW) x.w = (float)w;
      L->lst[s] = x;
      L->who[s] = make_uint2(j, (uint32_t)kc);
      if constexpr (kVel) L->vel[s] = (cross ? ldu(&J->vel32_y) : ldu(&J->vel32_x))[j];
    }
    tail += (uint32_t)__popcll(m);
    __builtin_amdgcn_wave_barrier();
  }

  // candidates [jb, je) of one run of cells with image code kc
  __device__ __forceinline__ void scan(uint32_t jb, uint32_t je, int kc) {
    double o[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int a = 0; a < DIM; ++a) o[a] = (ldu(&J->tK[kc * 4 + a]) - O[a]) * scale;
    for (uint32_t cb = jb; cb < je; cb += kWave) {
      const uint32_t j = cb + (uint32_t)lane;
      const bool valid = j < je;
      const double4 r = R[valid ? j : je - 1u];
      const float4 x = rel(r, o);
      const float ex = fmaxf(fmaxf(bl[0] - x.x, x.x - bh[0]), 0.0f);
      const float ey = fmaxf(fmaxf(bl[1] - x.y, x.y - bh[1]), 0.0f);
      float dd = __builtin_fmaf(ey, ey, ex * ex);
      if (DIM == 3) {
        const float ez = fmaxf(fmaxf(bl[2] - x.z, x.z - bh[2]), 0.0f);
        dd = __builtin_fmaf(ez, ez, dd);
      }
      push(valid && dd <= hi, x, r.w, j, kc);
      bool did = false;
      while (tail - head >= (uint32_t)kGrp) {
        block<false>(head, kGrp);
        head += (uint32_t)kGrp;
        did = true;
      }
      if (did) fold();
    }
  }

  // ------------------------------------------------------------ the group
  // Rows r (in visiting order) with r % ngrp == grp.
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
    const double4 ri = ldu(&J->r64_x)[gs + (uint32_t)min(c, gc - 1)];
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
      if constexpr (kHist) {
        nbins = ldu(&J->nbins);
        E64 = ldu(&J->E64);
        inv_h64 = (double)nbins / ldu(&J->hist_hi);
        want_sums = ldu(&J->want_sums);
        // v is within bv of the true value, so u is within bv / sqrt(v)
        // (|sqrt(v) - sqrt(v')| = |v - v'| / (sqrt(v) + sqrt(v'))) and a few
        // units of its own; beyond the last bin the error of a speed grows
        // with the speed: E bounds it in bin widths
        float bv = band;
        if constexpr (kRel) {
          const double ih2 = inv_h64 * inv_h64;
          s2f = (float)ih2;
          bv = (float)(ldu(ldu(&J->bandq)) * ih2 * 1.0001);
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
      const float x0 = act ? xi.x : -1e18f;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        xr[r][0] = from_lane(x0, 4 * q + r);
        xr[r][1] = from_lane(xi.y, 4 * q + r);
        xr[r][2] = DIM == 3 ? from_lane(xi.z, 4 * q + r) : 0.0f;
        acc[r] = 0.0f;
      }
      if constexpr (kW) {
#pragma unroll
        for (int r = 0; r < 4; ++r) wr[r] = __shfl(ri.w, 4 * q + r, kWave);
      }
    }
    if constexpr (KIND == K_LJ_E) {
      s2 = ldu(&J->s2);
      s2f = ldu(&J->s2f);
      near2 = ldu(&J->near2f);
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
    qtail = 0;
    head = 0;
    tail = 0;

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
    const int cy = (int)(T.row % (uint32_t)ny);
    const int cz = DIM == 3 ? (int)(T.row / (uint32_t)ny) : 0;
    // neighbour rows in visiting order: half shell (home row first, then
    // (dz, dy) > 0), cross sets all; each row's stencil is at most two runs
    // of cells (the range is no longer than the row)
    const int side = 2 * l + 1;
    const int nrow = cross ? (DIM == 3 ? side * side : side) : half_rows(DIM, l);
    const int mine = nrow > grp ? (nrow - grp + ngrp - 1) / ngrp : 0;  // rows grp, grp + ngrp, ...
    if (!cross && grp == 0) {  // the group against itself
      const bool keep = lane < gc;
      push(keep, xi, ri.w, gs + (uint32_t)lane, 13);
      block<true>(0, gc);
      fold();
      head = tail = 0;
    }
    for (int base = 0; base < mine; base += kWave / 2) {
      // lane 2 k + p: run p of row grp + (base + k) ngrp
      uint32_t jb = 0, je = 0;
      int kc = 13;
      {
        const int k = base + (lane >> 1), p = lane & 1;
        if (k < mine) {
          const int r = grp + k * ngrp;
          int dy, dz;
          if (cross) {
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
          const bool home = !cross && r == 0;
          const int xlo = home ? gx0 : gx0 - lx, xhi = gx1 + lx;
          // p = 0: the cells of the row itself; p = 1: what wraps around
          int a0, a1, px;
          if (p == 0) { a0 = max(xlo, 0); a1 = min(xhi, nx - 1); px = 0; }
          else if (xlo < 0) { a0 = xlo; a1 = min(xhi, -1); px = -1; }
          else { a0 = max(xlo, nx); a1 = xhi; px = 1; }
          if (a0 <= a1) {
            jb = OFF[rowbase + a0 - px * nx];
            je = OFF[rowbase + a1 - px * nx + 1];
            if (home && p == 0) jb = gs + (uint32_t)gc;  // after the group itself
            kc = kcode(px, py, pz);
          }
        }
      }
      unsigned long long runs = __builtin_amdgcn_ballot_w64(jb < je);
      while (runs) {
        const int s = (int)__builtin_ctzll(runs);
        runs &= runs - 1ull;
        scan((uint32_t)__builtin_amdgcn_readlane((int)jb, s), (uint32_t)__builtin_amdgcn_readlane((int)je, s),
             __builtin_amdgcn_readlane(kc, s));
      }
    }
    if (tail != head) {
      block<false>(head, (int)(tail - head));
      fold();
    }
    drain(true);
  }
};

}  // namespace

template <int DIM, int KIND>
__global__ void __launch_bounds__(kGWaves * kWave) group_kernel(const JobDesc* __restrict__ jobs,
                                                                const Tile* __restrict__ tiles,
                                                                const uint32_t* __restrict__ ntiles_dev,
                                                                int split_rows) {
  constexpr bool kHist = KIND == K_HIST_DIST || KIND == K_HIST_REL || KIND == K_HIST_DV;
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ GroupLds<KIND> lds[kGWaves];
  __shared__ double red_e[kGWaves];
  __shared__ unsigned long long red_c[kGWaves];
  __shared__ uint32_t red_g[kGWaves][2];
  const int lane = (int)__lane_id();
  const int wid = uniform((int)(threadIdx.x / kWave));
  const int cap = (int)gridDim.x;
  const int ntiles = min((int)ldu(ntiles_dev), cap);
  const int G = sweep_split(ntiles, cap, split_rows);
  const int nitems = ntiles * G;
  int b = blockIdx.x;
  if (b >= nitems) return;
  if (nitems >= 8) {  // each XCD (block mod 8) a contiguous range of items
    const int per = nitems / 8, rem = nitems % 8;
    const int xcd = b % 8, k = b / 8;
    b = (xcd < rem ? xcd * (per + 1) : rem * (per + 1) + (xcd - rem) * per) + k;
  }
  const int tile_id = b / G, grp = b - tile_id * G;
  const Tile T = ldu(&tiles[tile_id]);

  Group<DIM, KIND> S;
  S.J = &jobs[T.job];
  S.L = &lds[wid];
  S.lane = lane;
  S.accE = 0.0;
  S.cnt_wave = 0;
  S.cnt_lane = 0;
  S.qband = 0;
  S.qnear = 0;
  int nb = 0, lgC = 0;
  uint32_t* hist = nullptr;
  double* hsum = nullptr;
  if constexpr (kHist) {
    nb = ldu(&S.J->nbins);
    lgC = hist_lgC(KIND, nb);
    const int nh = (nb + 1) << lgC;
    hsum = (double*)smem;
    hist = (uint32_t*)(smem + (hist_has_sums(KIND) ? (size_t)nh * 8 : 0));
    for (int k = threadIdx.x; k < nh; k += kGWaves * kWave) {
      hist[k] = 0u;
      if constexpr (hist_has_sums(KIND)) hsum[k] = 0.0;
    }
    const int copy = (int)threadIdx.x & ((1 << lgC) - 1);
    S.hist = hist + copy;
    S.hsum = hsum + copy;
    S.lgC = lgC;
    __syncthreads();
  }
  // group of this wave; tiles of one or two groups spread their rows
  const int ng = ((int)T.count + kGrp - 1) / kGrp;
  const int nsub = ng == 1 ? 4 : (ng == 2 ? 2 : 1);
  const int g = nsub == 1 ? wid : wid % ng, sub = nsub == 1 ? 0 : wid / ng;
  if (g < ng) S.run(T, g, grp + G * sub, G * nsub);
  const unsigned long long cnt = S.cnt_wave + wave_sum_u64(S.cnt_lane);
  const double e = wave_sum_d(S.accE);
  const uint32_t gb = wave_sum_u32(S.qband), gn = wave_sum_u32(S.qnear);
  if (lane == 0) {
    red_c[wid] = cnt;
    red_e[wid] = e;
    red_g[wid][0] = gb;
    red_g[wid][1] = gn;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    const int local = (tile_id - ldu(&S.J->tile_begin)) * G + grp;
    ldu(&S.J->pcount)[local] = ((red_c[0] + red_c[1]) + red_c[2]) + red_c[3];
    double* Pp = ldu(&S.J->partials) + (size_t)local * kPartialD;
    Pp[P_SUM] = ((red_e[0] + red_e[1]) + red_e[2]) + red_e[3];
    // the re-evaluation counts go through the finalize, too: adds of every
    // wave to one address took as long as the sweep
    Pp[P_BAND] = (double)(red_g[0][0] + red_g[1][0] + red_g[2][0] + red_g[3][0]);
    Pp[P_NEAR] = (double)(red_g[0][1] + red_g[1][1] + red_g[2][1] + red_g[3][1]);
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

template <int DIM>
static hipError_t group_dispatch(int kind, unsigned grid, size_t lds, const JobDesc* jobs, const Tile* tiles,
                                 const uint32_t* nt, int split, hipStream_t s) {
  constexpr int kT = kGWaves * kWave;
  switch (kind) {
    case K_COUNT: group_kernel<DIM, K_COUNT><<<grid, kT, lds, s>>>(jobs, tiles, nt, split); break;
    case K_SUM_D: group_kernel<DIM, K_SUM_D><<<grid, kT, lds, s>>>(jobs, tiles, nt, split); break;
    case K_SUM_INV_D: group_kernel<DIM, K_SUM_INV_D><<<grid, kT, lds, s>>>(jobs, tiles, nt, split); break;
    case K_SUM_W: group_kernel<DIM, K_SUM_W><<<grid, kT, lds, s>>>(jobs, tiles, nt, split); break;
    case K_LJ_E: group_kernel<DIM, K_LJ_E><<<grid, kT, lds, s>>>(jobs, tiles, nt, split); break;
    case K_HIST_DIST: group_kernel<DIM, K_HIST_DIST><<<grid, kT, lds, s>>>(jobs, tiles, nt, split); break;
    case K_HIST_REL: group_kernel<DIM, K_HIST_REL><<<grid, kT, lds, s>>>(jobs, tiles, nt, split); break;
    case K_HIST_DV: group_kernel<DIM, K_HIST_DV><<<grid, kT, lds, s>>>(jobs, tiles, nt, split); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_group(int dim, int kind, const JobDesc* jobs, const Tile* tiles, const uint32_t* ntiles_dev,
                        int max_tiles, int nbins, hipStream_t s, int split_rows) {
  if (max_tiles <= 0) return hipSuccess;
  const bool hist = kind == K_HIST_DIST || kind == K_HIST_REL || kind == K_HIST_DV;
  const size_t lds = hist ? hist_group_bytes(kind, nbins) : 0;
  return dim == 3 ? group_dispatch<3>(kind, (unsigned)max_tiles, lds, jobs, tiles, ntiles_dev, split_rows, s)
                  : group_dispatch<2>(kind, (unsigned)max_tiles, lds, jobs, tiles, ntiles_dev, split_rows, s);
}

hipError_t launch_hist_reduce(const JobDesc* jobs, int njobs, int nbins, hipStream_t s) {
  hist_reduce_kernel<<<dim3((nbins + 4) / 4, njobs), 256, 0, s>>>(jobs);
  return hipGetLastError();
}

}  // namespace clm
