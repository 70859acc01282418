// md_kernels.hip -- velocity Verlet and a Verlet pair list on gfx950 (the
// molecular-dynamics use of the paper's section 4.2: Lennard-Jones forces,
// velocity Verlet, velocity rescaling, pair lists kept over several steps).
//
//   md_kick_drift   one thread per particle: v = lambda v + h f, x += dt v
//   md_kick         one thread per particle: v += h f, block sums of |v|^2
//   vl_drift        one thread per particle: largest |x - x_ref|^2 (atomic max
//                   on the bits of a non-negative double)
//   vl_decide       one thread: rebuild flag of this step, counters
//   (the list itself: sweep_group.hip, a list for every four rows)
//   vl_refresh      one thread per sorted slot: frame position H (Hinv x - w)
//   vl_lj           one wave per four sorted slots (rows): FP64 LJ over their
//                   list, optional fused second half-kick, block partials
//   md_finalize     one block: fixed-order sum of the block partials
//
// All are HBM- or latency-bound except vl_lj, whose bound is the FP64 VALU work
// per listed pair.
#include "clmap_internal.h"
#include "device_util.h"

namespace clm {

namespace {

// Block of kMdBlock threads: sums of kMdPart doubles and one count into
// part[b * kMdPart + k] and pcount[b] (fixed order: waves, then wave 0..3).
__device__ __forceinline__ void block_partials(const double* acc, unsigned long long cnt,
                                               double* __restrict__ part,
                                               unsigned long long* __restrict__ pcount, int b) {
  __shared__ double red[kMdBlock / kWave][kMdPart];
  __shared__ unsigned long long redc[kMdBlock / kWave];
  const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
#pragma unroll
  for (int k = 0; k < kMdPart; ++k) {
    const double s = wave_sum_d(acc[k]);
    if (lane == 0) red[w][k] = s;
  }
  const unsigned long long c = wave_sum_u64(cnt);
  if (lane == 0) redc[w] = c;
  __syncthreads();
  if (threadIdx.x < kMdPart) {
    double s = 0.0;
    for (int q = 0; q < kMdBlock / kWave; ++q) s += red[q][threadIdx.x];
    part[(size_t)b * kMdPart + threadIdx.x] = s;
  }
  if (threadIdx.x == 0 && pcount) {
    unsigned long long s = 0;
    for (int q = 0; q < kMdBlock / kWave; ++q) s += redc[q];
    pcount[b] = s;
  }
}

// Blocks are dispatched to the 8 XCDs round-robin; give each XCD a
// contiguous range of rows (spatial neighbours share that XCD's L2).
__device__ __forceinline__ int xcd_block(int b, int nblk) {
  if (nblk < 8) return b;
  const int per = nblk / 8, rem = nblk % 8;
  const int xcd = b % 8, k = b / 8;
  return (xcd < rem ? xcd * (per + 1) : rem * (per + 1) + (xcd - rem) * per) + k;
}

}  // namespace

// ---------------------------------------------------------------- integrator
__global__ void __launch_bounds__(kMdBlock) md_kick_drift_kernel(double* __restrict__ x,
                                                                 double* __restrict__ v,
                                                                 const double* __restrict__ f,
                                                                 int64_t ncomp, double h, double dt,
                                                                 double target_ke,
                                                                 const double* __restrict__ ke) {
  const int64_t k = (int64_t)blockIdx.x * kMdBlock + threadIdx.x;
  if (k >= ncomp) return;
  double vk = v[k];
  if (target_ke > 0.0) vk = sqrt(target_ke / *ke) * vk;
  vk = vk + h * f[k];
  v[k] = vk;
  x[k] = x[k] + dt * vk;
}

__global__ void __launch_bounds__(kMdBlock) md_kick_kernel(double* __restrict__ v,
                                                           const double* __restrict__ f, int n,
                                                           int dim, double h,
                                                           double* __restrict__ part) {
  const int i = blockIdx.x * kMdBlock + threadIdx.x;
  double acc[kMdPart];
#pragma unroll
  for (int k = 0; k < kMdPart; ++k) acc[k] = 0.0;
  if (i < n) {
    double q = 0.0;
    for (int a = 0; a < dim; ++a) {
      double va = v[(size_t)i * dim + a];
      if (f) {  // f == NULL: kinetic energy of v only
        va = va + h * f[(size_t)i * dim + a];
        v[(size_t)i * dim + a] = va;
      }
      q = a == 0 ? va * va : q + va * va;
    }
    acc[MP_KE] = q;
  }
  block_partials(acc, 0ull, part, nullptr, blockIdx.x);
}

// v = sqrt(target_ke / KE) v, KE the integrator's kept kinetic energy.
__global__ void __launch_bounds__(kMdBlock) md_rescale_kernel(double* __restrict__ v, int64_t ncomp,
                                                              double target_ke,
                                                              const double* __restrict__ ke) {
  const int64_t k = (int64_t)blockIdx.x * kMdBlock + threadIdx.x;
  if (k >= ncomp) return;
  v[k] = sqrt(target_ke / *ke) * v[k];
}

// One block: fixed-order sums of nb partials (each thread sums rows t,
// t + 256, ... of all components, then waves and the block combine in a fixed
// order).  energy = 2 eps sum(u) (every pair was seen from both ends), virial
// = 12 eps sum(f D D), count = pairs / 2, ke = mass / 2 sum |v|^2.
__global__ void __launch_bounds__(256) md_finalize_kernel(MdFinal F) {
  __shared__ double red[4][kMdPart];
  __shared__ unsigned long long redc[4];
  double acc[kMdPart];
#pragma unroll
  for (int k = 0; k < kMdPart; ++k) acc[k] = 0.0;
  unsigned long long c = 0;
  for (int b = threadIdx.x; b < F.nb; b += 256) {
#pragma unroll
    for (int k = 0; k < kMdPart; ++k) acc[k] += F.part[(size_t)b * kMdPart + k];
    if (F.pcount) c += F.pcount[b];
  }
  const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
#pragma unroll
  for (int k = 0; k < kMdPart; ++k) {
    const double v = wave_sum_d(acc[k]);
    if (lane == 0) red[w][k] = v;
  }
  c = wave_sum_u64(c);
  if (lane == 0) redc[w] = c;
  __syncthreads();
  if (threadIdx.x != 0) return;
  double keep[kMdPart];
  for (int k = 0; k < kMdPart; ++k) keep[k] = ((red[0][k] + red[1][k]) + red[2][k]) + red[3][k];
  const unsigned long long cnt = redc[0] + redc[1] + redc[2] + redc[3];
  if (F.energy) *F.energy = 2.0 * F.eps * keep[MP_E];
  if (F.virial) {
    const int d = F.dim;
    const int slot[3][3] = {{MP_W + 0, MP_W + 1, MP_W + 2},
                            {MP_W + 1, MP_W + 3, MP_W + 4},
                            {MP_W + 2, MP_W + 4, MP_W + 5}};
    for (int a = 0; a < d; ++a)
      for (int b = 0; b < d; ++b) F.virial[a * d + b] = 12.0 * F.eps * keep[slot[a][b]];
  }
  if (F.count) *F.count = cnt / 2;
  if (F.ke_keep) {
    const double ke = 0.5 * F.mass * keep[MP_KE];
    *F.ke_keep = ke;
    if (F.ke) *F.ke = ke;
  }
}

// ---------------------------------------------------------------- Verlet list: maintenance
// Largest squared displacement since the last rebuild: per-block maxima
// (grid-stride over the particles, at most kDriftBlocks blocks), no atomics.
__global__ void __launch_bounds__(kMdBlock) vl_drift_kernel(const double* __restrict__ x,
                                                            const double* __restrict__ xref, int n,
                                                            int dim, double* __restrict__ bmax) {
  double m = 0.0;
  for (int i = blockIdx.x * kMdBlock + threadIdx.x; i < n; i += gridDim.x * kMdBlock) {
    double q = 0.0;
    for (int a = 0; a < dim; ++a) {
      const double d = x[(size_t)i * dim + a] - xref[(size_t)i * dim + a];
      q = a == 0 ? d * d : q + d * d;
    }
    // a NaN displacement forces a rebuild
    m = fmax(m, q == q ? q : 1.0e300);
  }
  for (int d = kWave / 2; d > 0; d >>= 1) m = fmax(m, __shfl_xor(m, d, kWave));
  __shared__ double wm[kMdBlock / kWave];
  if ((threadIdx.x & (kWave - 1)) == 0) wm[threadIdx.x / kWave] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    double b = wm[0];
    for (int k = 1; k < kMdBlock / kWave; ++k) b = fmax(b, wm[k]);
    bmax[blockIdx.x] = b;
  }
}

// One block: the largest of the block maxima against (skin / 2)^2 decides
// this step's rebuild; counters.
__global__ void __launch_bounds__(256) vl_decide_kernel(const double* __restrict__ bmax, int nb,
                                                        double lim2, VlFlags* __restrict__ fl) {
  double m = 0.0;
  for (int b = threadIdx.x; b < nb; b += 256) m = fmax(m, bmax[b]);
  for (int d = kWave / 2; d > 0; d >>= 1) m = fmax(m, __shfl_xor(m, d, kWave));
  __shared__ double wm[4];
  if ((threadIdx.x & (kWave - 1)) == 0) wm[threadIdx.x / kWave] = m;
  __syncthreads();
  if (threadIdx.x != 0) return;
  const double mx = fmax(fmax(wm[0], wm[1]), fmax(wm[2], wm[3]));
  const bool g = fl->force != 0u || mx > lim2;
  fl->gate = g ? 1u : 0u;
  fl->force = 0u;
  fl->updates += 1ull;
  if (g) {
    fl->rebuilds += 1ull;
    fl->entries = 0ull;
    fl->max_row = 0u;
  }
}

// Frame position of every sorted slot: r'' = H (Hinv x - w), the canonical
// wrap's operations without the floor; x_ref = x on a rebuild step.
__global__ void __launch_bounds__(kMdBlock) vl_refresh_kernel(VlRefresh A) {
  const int s = blockIdx.x * kMdBlock + threadIdx.x;
  if (s >= A.n) return;
  const uint32_t i = A.idx[s];
  const int4 w4 = A.wrap[s];
  const int w[3] = {w4.x, w4.y, w4.z};
  double r[3] = {0.0, 0.0, 0.0};
  for (int a = 0; a < A.dim; ++a) r[a] = A.x[(size_t)i * A.dim + a];
  double f[3] = {0.0, 0.0, 0.0};
  for (int a = 0; a < A.dim; ++a) {
    double acc = A.Hinv[a * 3 + 0] * r[0];
    acc = acc + A.Hinv[a * 3 + 1] * r[1];
    if (A.dim == 3) acc = acc + A.Hinv[a * 3 + 2] * r[2];
    f[a] = acc - (double)w[a];
  }
  double q[3] = {0.0, 0.0, 0.0};
  for (int a = 0; a < A.dim; ++a) {
    double acc = A.H[a * 3 + 0] * f[0];
    acc = acc + A.H[a * 3 + 1] * f[1];
    if (A.dim == 3) acc = acc + A.H[a * 3 + 2] * f[2];
    q[a] = acc;
  }
  A.pf[s] = make_double4(q[0], q[1], q[2], A.pf[s].w);  // (w: the list's)
  if (*A.gate != 0u)
    for (int a = 0; a < A.dim; ++a) A.xref[(size_t)i * A.dim + a] = r[a];
}

// After a rebuild: row lengths (capped at the capacity), overflow flag, the
// longest row and the number of stored entries.
__global__ void __launch_bounds__(kMdBlock) vl_rowstats_kernel(uint32_t* __restrict__ cnt, int n,
                                                               int cap, VlFlags* __restrict__ fl,
                                                               const uint32_t* __restrict__ gate) {
  if (*gate == 0u) return;
  const int s = blockIdx.x * kMdBlock + threadIdx.x;
  uint32_t c = 0;
  if (s < n) {
    c = cnt[s];
    if (c > (uint32_t)cap) {
      fl->overflow = 1u;
      cnt[s] = (uint32_t)cap;
    }
  }
  uint32_t cm = c;
  unsigned long long st = c < (uint32_t)cap ? c : (uint32_t)cap;
  for (int d = kWave / 2; d > 0; d >>= 1) cm = max(cm, (uint32_t)__shfl_xor((int)cm, d, kWave));
  st = wave_sum_u64(st);
  __shared__ uint32_t wm[kMdBlock / kWave];
  __shared__ unsigned long long ws[kMdBlock / kWave];
  if ((threadIdx.x & (kWave - 1)) == 0) {
    wm[threadIdx.x / kWave] = cm;
    ws[threadIdx.x / kWave] = st;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t m = 0;
    unsigned long long t = 0;
    for (int k = 0; k < kMdBlock / kWave; ++k) {
      m = max(m, wm[k]);
      t += ws[k];
    }
    atomicMax(&fl->max_row, m);
    atomicAdd(&fl->entries, t);
  }
}

// ---------------------------------------------------------------- Verlet list: forces
// A candidate j at xj against the rows; t: its image shift (IMG).
template <int DIM, bool VIR, bool IMG>
__device__ __forceinline__ void vl_batch(const double* xj, const double* t, uint32_t j, const uint32_t* slot,
                                         const double (*xr)[3], double rc2, double s2, double (*F)[3], double* W,
                                         double& E, uint32_t& npair) {
#pragma unroll
  for (int r = 0; r < kVlRows; ++r) {
    double D[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int a = 0; a < DIM; ++a) {
      D[a] = xj[a] - xr[r][a];
      if constexpr (IMG) D[a] = D[a] + t[a];
    }
    double d2 = D[0] * D[0] + D[1] * D[1];
    if (DIM == 3) d2 = d2 + D[2] * D[2];
    const bool in = d2 <= rc2 && j != slot[r];
    const double ri = in ? rcp64(d2) : 0.0;
    const double q = s2 * ri;
    const double q3 = q * q * q;
    const double u = __builtin_fma(q3, q3, -q3);
    const double f = __builtin_fma(q3, q3, u) * ri;
    E += u;
    npair += in ? 1u : 0u;
#pragma unroll
    for (int a = 0; a < DIM; ++a) F[r][a] = __builtin_fma(f, D[a], F[r][a]);
    if constexpr (VIR) {
      const double fx = f * D[0], fy = f * D[1];
      W[0] = __builtin_fma(fx, D[0], W[0]);
      W[1] = __builtin_fma(fx, D[1], W[1]);
      W[3] = __builtin_fma(fy, D[1], W[3]);
      if (DIM == 3) {
        W[2] = __builtin_fma(fx, D[2], W[2]);
        W[4] = __builtin_fma(fy, D[2], W[4]);
        W[5] = __builtin_fma(f * D[2], D[2], W[5]);
      }
    }
  }
}

// A wave per kVlRows rows (consecutive sorted slots of a tile): the lanes hold
// candidates of the rows' list (sweep_group.hip: the partners that some row had
// within the list cutoff), the rows' positions are scalars.  Canonical FP64
// displacement in the frame, membership d2 <= rc2, Lennard-Jones u and f.
//
// What bounds it: the FP64 vector ALU.  With a list for every particle each
// pair read 4 bytes of list and gathered 32 of position, 2.5 GB a step at 10^5
// atoms of some 700 partners, and the L2 bound it (209 us, the vector ALU half
// idle); with one for 16 particles most of a list is out of a row's range (230
// us, 9.9 10^7 vector instructions instead of 6.3 10^7).  Four rows, the closest
// of 16: 191 us, 8.1 10^7, 44 % of the listed pairs in range; two copies of the
// loop, without and with image shifts (one that selects: 199 us).
template <int DIM, bool KICK, bool VIR>
__global__ void __launch_bounds__(kMdBlock) vl_lj_kernel(VlForce A) {
  constexpr int kHere = 13;
  __shared__ double tk[27 * 3];
  for (int k = threadIdx.x; k < 27 * 3; k += kMdBlock) tk[k] = A.tK[(k / 3) * 4 + k % 3];
  __syncthreads();
  const int lane = (int)threadIdx.x % kWave, wid = uniform((int)threadIdx.x / kWave);
  // items: 16 rows of a tile, kVlRows a wave
  const int64_t items = 4 * (int64_t)min((int)ldu(A.ntiles), A.max_tiles);
  const int b = xcd_block(blockIdx.x, A.nb);
  const int64_t lo = items * b / A.nb, hi = items * (b + 1) / A.nb;
  const double rc2 = A.rc2, s2 = A.s2;
  double E = 0.0, ke = 0.0;
  double W[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
  uint32_t npair = 0;
  for (int64_t it = lo; it < hi; ++it) {
    const Tile T = ldu(&A.tiles[it / 4]);
    const int first = 16 * (int)(it % 4) + kVlRows * wid;
    const int gc = min((int)T.count - first, kVlRows);
    if (gc <= 0) continue;
    const uint32_t gs = T.start + (uint32_t)first;
    const uint64_t word = (uint64_t)ldu(&A.pf[gs].w);
    const int len = (int)min((long long)(word >> 16), (long long)gc * A.cap);
    uint32_t slot[kVlRows];
    double xr[kVlRows][3], F[kVlRows][3];
#pragma unroll
    for (int r = 0; r < kVlRows; ++r) {
      slot[r] = gs - (uint32_t)(kVlRows * wid) + ((uint32_t)(word >> (4 * min(r, gc - 1))) & 15u);
      const double4 v = ldu(&A.pf[slot[r]]);
      xr[r][0] = r < gc ? v.x : 1e100;  // (no candidate reaches an absent row)
      xr[r][1] = v.y;
      xr[r][2] = v.z;
#pragma unroll
      for (int a = 0; a < 3; ++a) F[r][a] = 0.0;
    }
    const uint32_t* __restrict__ list = A.list + (size_t)gs * (size_t)A.cap;
    // entries two batches ahead, positions one
    int k = lane;
    uint32_t e = 0u, e1 = 0u;
    double4 p = make_double4(0.0, 0.0, 0.0, 0.0);
    if (k < len) {
      e = list[k];
      p = A.pf[e >> 5];
    }
    if (k + kWave < len) e1 = list[k + kWave];
    for (; k - lane < len; k += kWave) {
      const uint32_t ec = e;
      double x = k < len ? p.x : 2e100, y = p.y, z = p.z;
      e = e1;
      if (k + kWave < len) p = A.pf[e >> 5];
      if (k + 2 * kWave < len) e1 = list[k + 2 * kWave];
      const int kc = k < len ? (int)(ec & 31u) : kHere;
      const bool img = __builtin_amdgcn_ballot_w64(kc != kHere) != 0ull;
      const double xj[3] = {x, y, z};
      if (img) {
        const double t[3] = {tk[kc * 3], tk[kc * 3 + 1], tk[kc * 3 + 2]};
        vl_batch<DIM, VIR, true>(xj, t, ec >> 5, slot, xr, rc2, s2, F, W, E, npair);
      } else {
        vl_batch<DIM, VIR, false>(xj, nullptr, ec >> 5, slot, xr, rc2, s2, F, W, E, npair);
      }
    }
    // lane r: row r
    double G[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int r = 0; r < kVlRows; ++r)
#pragma unroll
      for (int a = 0; a < DIM; ++a) {
        double v = sum16(F[r][a]);
        v += __shfl_xor(v, 16, kWave);
        v += __shfl_xor(v, 32, kWave);
        G[a] = lane == r ? v : G[a];
      }
    if (lane < gc) {
      const uint32_t i = A.idx[gs - (uint32_t)(kVlRows * wid) + ((uint32_t)(word >> (4 * lane)) & 15u)];
      const double m24 = -24.0 * A.eps;
      double qq = 0.0;
#pragma unroll
      for (int a = 0; a < DIM; ++a) {
        const double Fa = m24 * G[a];
        A.forces[(size_t)i * DIM + a] = Fa;
        if constexpr (KICK) {
          const double va = A.v[(size_t)i * DIM + a] + A.h * Fa;
          A.v[(size_t)i * DIM + a] = va;
          qq = a == 0 ? va * va : qq + va * va;
        }
      }
      ke += qq;
    }
  }
  double acc[kMdPart];
  acc[MP_E] = E;
#pragma unroll
  for (int w = 0; w < 6; ++w) acc[MP_W + w] = W[w];
  acc[MP_KE] = ke;
  block_partials(acc, npair, A.part, A.pcount, b);
}

// ---------------------------------------------------------------- launchers
static inline unsigned blocks_for(int64_t n, int block) {
  int64_t g = (n + block - 1) / block;
  return (unsigned)(g < 1 ? 1 : g);
}

hipError_t launch_md_kick_drift(double* x, double* v, const double* f, int64_t ncomp, double h,
                                double dt, double target_ke, const double* ke, hipStream_t s) {
  if (ncomp == 0) return hipSuccess;
  md_kick_drift_kernel<<<blocks_for(ncomp, kMdBlock), kMdBlock, 0, s>>>(x, v, f, ncomp, h, dt,
                                                                        target_ke, ke);
  return hipGetLastError();
}

hipError_t launch_md_kick(double* v, const double* f, int n, int dim, double h, double* part,
                          hipStream_t s) {
  md_kick_kernel<<<blocks_for(n, kMdBlock), kMdBlock, 0, s>>>(v, f, n, dim, h, part);
  return hipGetLastError();
}

hipError_t launch_md_rescale(double* v, int64_t ncomp, double target_ke, const double* ke,
                             hipStream_t s) {
  if (ncomp == 0) return hipSuccess;
  md_rescale_kernel<<<blocks_for(ncomp, kMdBlock), kMdBlock, 0, s>>>(v, ncomp, target_ke, ke);
  return hipGetLastError();
}

hipError_t launch_md_finalize(const MdFinal& F, hipStream_t s) {
  md_finalize_kernel<<<1, 256, 0, s>>>(F);
  return hipGetLastError();
}

int vl_drift_blocks(int64_t n) {
  const int64_t b = (n + kMdBlock - 1) / kMdBlock;
  return (int)(b < 1 ? 1 : (b > kDriftBlocks ? kDriftBlocks : b));
}

hipError_t launch_vl_drift(const double* x, const double* xref, int n, int dim, double lim2,
                           double* bmax, VlFlags* fl, hipStream_t s) {
  const int nb = vl_drift_blocks(n);
  vl_drift_kernel<<<nb, kMdBlock, 0, s>>>(x, xref, n, dim, bmax);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  vl_decide_kernel<<<1, 256, 0, s>>>(bmax, nb, lim2, fl);
  return hipGetLastError();
}

hipError_t launch_vl_rowstats(uint32_t* cnt, int n, int cap, VlFlags* fl, const uint32_t* gate,
                              hipStream_t s) {
  vl_rowstats_kernel<<<blocks_for(n, kMdBlock), kMdBlock, 0, s>>>(cnt, n, cap, fl, gate);
  return hipGetLastError();
}

hipError_t launch_vl_refresh(const VlRefresh& A, hipStream_t s) {
  if (A.n == 0) return hipSuccess;
  vl_refresh_kernel<<<blocks_for(A.n, kMdBlock), kMdBlock, 0, s>>>(A);
  return hipGetLastError();
}

hipError_t launch_vl_lj(int dim, bool kick, bool vir, const VlForce& A, hipStream_t s) {
#define CLM_VL_LJ(D, K, V) vl_lj_kernel<D, K, V><<<A.nb, kMdBlock, 0, s>>>(A)
  if (dim == 3) {
    if (kick) { if (vir) CLM_VL_LJ(3, true, true); else CLM_VL_LJ(3, true, false); }
    else { if (vir) CLM_VL_LJ(3, false, true); else CLM_VL_LJ(3, false, false); }
  } else {
    if (kick) { if (vir) CLM_VL_LJ(2, true, true); else CLM_VL_LJ(2, true, false); }
    else { if (vir) CLM_VL_LJ(2, false, true); else CLM_VL_LJ(2, false, false); }
  }
#undef CLM_VL_LJ
  return hipGetLastError();
}

}  // namespace clm
