// nl_rows.hip -- sorted neighbour lists by rows: the list of every particle i
// is a row (partners of larger index in a single set), counted and written by
// the group sweep (sweep_group.hip); here the rows' offsets and the ascending
// order within each row.
//
// Rows keep the first index in place, so only the partners of one particle
// have to be ordered: in LDS, with one read and one write of the list.  The
// radix sort of the whole list (nl_sort.hip) moves every entry once per 8 bits
// of (i, j), five passes at 2 10^5 particles: 30.5 10^6 pairs with distances
// 3250 us, the offsets and the rows' order 280 us.
//
// A list beyond its capacity is the first entries of the whole list: of the row
// that the capacity cuts the partners are kept as a bit map over their indices,
// with the distances by index, and its smallest ones are written.
#include "clmap_internal.h"
#include "device_util.h"

namespace clm {

namespace {

constexpr int kWave = 64;
constexpr int kScanThreads = 256;
constexpr int kScanPer = 16;
constexpr int kScanRows = kScanThreads * kScanPer;  // rows of a block
// Longest rows of the classes 0 (a wave of a small block), 1 (a wave of a large
// one: its registers and LDS would cost the short rows half the waves), 2 (a
// block's LDS); 3: longer.
constexpr int kRow0 = 512, kRow1 = 1024, kRow2 = 8192;
constexpr int kLongThreads = 1024;
constexpr int kBitWords = 8192;  // bit map of a window of 2^18 indices

__device__ __forceinline__ int row_class(uint32_t cnt) {
  return (cnt > (uint32_t)kRow0 ? 1 : 0) + (cnt > (uint32_t)kRow1 ? 1 : 0) + (cnt > (uint32_t)kRow2 ? 1 : 0);
}

// Whether the capacity cuts the row.
__device__ __forceinline__ bool row_cut(const RowArgs& A, unsigned long long off, uint32_t cnt) {
  const unsigned long long cap = (unsigned long long)A.capacity;
  return off < cap && cap - off < cnt;
}

// The lists of rows of classes 1 to 3: the first two share an array.
__device__ __forceinline__ uint32_t& long_row(const RowArgs& A, int z, uint32_t p) {
  return z == 1 ? A.list[0][(uint32_t)A.n - 1u - p] : A.list[z / 2][p];
}

__device__ __forceinline__ uint32_t row_len(const RowArgs& A, unsigned long long off, uint32_t cnt) {
  const unsigned long long cap = (unsigned long long)A.capacity;
  return off >= cap ? 0u : (uint32_t)(cap - off < cnt ? cap - off : cnt);
}

// Entry t of the row at off (partner j) to place r.
__device__ __forceinline__ void put(const RowArgs& A, int i, unsigned long long off, uint32_t t, uint32_t r,
                                    uint32_t j) {
  ((int2*)A.pairs)[off + r] = make_int2(i, (int)j);
  if (A.row_d) A.dist[off + r] = A.row_d[off + t];
}

// Counts of every block's rows; the lists empty.
__global__ void __launch_bounds__(kScanThreads) row_sums_kernel(RowArgs A) {
  __shared__ unsigned long long w[kScanThreads / kWave];
  const int t = (int)threadIdx.x;
  unsigned long long s = 0;
  for (int k = 0; k < kScanPer; ++k) {
    const long long i = (long long)blockIdx.x * kScanRows + k * kScanThreads + t;
    if (i < A.n) s += A.cnt[i];
  }
  s = wave_sum_u64(s);
  if (t % kWave == 0) w[t / kWave] = s;
  __syncthreads();
  if (t == 0) {
    A.sums[blockIdx.x] = ((w[0] + w[1]) + w[2]) + w[3];
    if (blockIdx.x == 0)
      for (int z = 0; z < 4; ++z) A.longs[z] = z < 3 ? 0u : 0xffffffffu;
  }
}

// Offsets of the rows; rows too long for a wave to the lists.
__global__ void __launch_bounds__(kScanThreads) row_offsets_kernel(RowArgs A) {
  __shared__ unsigned long long w[kScanThreads / kWave], v[kScanThreads / kWave];
  __shared__ uint32_t num[3];
  const int t = (int)threadIdx.x, lane = t % kWave, wid = t / kWave;
  unsigned long long before = 0;
  for (int b = t; b < (int)blockIdx.x; b += kScanThreads) before += A.sums[b];
  before = wave_sum_u64(before);
  const long long i0 = (long long)blockIdx.x * kScanRows + (long long)t * kScanPer;
  uint32_t c[kScanPer];
  unsigned long long s = 0;
#pragma unroll
  for (int k = 0; k < kScanPer; ++k) {
    c[k] = i0 + k < A.n ? A.cnt[i0 + k] : 0u;
    s += c[k];
  }
  unsigned long long x = s;  // inclusive over the wave
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) {
    const unsigned long long y = __shfl_up(x, d, kWave);
    if (lane >= d) x += y;
  }
  if (lane == kWave - 1) w[wid] = x;
  if (lane == 0) v[wid] = before;
  if (t < 3) num[t] = 0u;
  __syncthreads();
  unsigned long long o = (((v[0] + v[1]) + v[2]) + v[3]) + (x - s);
  for (int k = 0; k < wid; ++k) o += w[k];
  // places in the lists: one add of the block to each (an add per row, all to
  // one address, took 117 us of 10^4 rows)
  uint32_t m[3] = {0u, 0u, 0u}, p[3];
#pragma unroll
  for (int k = 0; k < kScanPer; ++k) {
    if (i0 + k < A.n) A.off[i0 + k] = o;
    const uint32_t v = c[k];
    if (row_cut(A, o, v)) {  // in none of the lists
      A.longs[3] = (uint32_t)(i0 + k);
      c[k] = 0u;
    }
    o += v;
#pragma unroll
    for (int z = 0; z < 3; ++z) m[z] += row_class(c[k]) == z + 1 ? 1u : 0u;
  }
#pragma unroll
  for (int z = 0; z < 3; ++z) p[z] = m[z] ? atomicAdd(&num[z], m[z]) : 0u;
  __syncthreads();
  if (t < 3) num[t] = num[t] ? atomicAdd(&A.longs[t], num[t]) : 0u;
  __syncthreads();
#pragma unroll
  for (int z = 0; z < 3; ++z) p[z] += num[z];
#pragma unroll
  for (int k = 0; k < kScanPer; ++k) {
#pragma unroll
    for (int z = 0; z < 3; ++z)
      if (row_class(c[k]) == z + 1) long_row(A, z, p[z]++) = (uint32_t)(i0 + k);
  }
}

// A whole row of 1 to 64 PER entries in order by one wave: buckets of equal index
// ranges in LDS (about one entry each), an entry's place is its bucket's start
// and the smaller ones in the bucket.  C: 64 PER + 1, K: 64 PER words.
template <int kPer>
__device__ __forceinline__ void sort_row(const RowArgs& A, int i, int lane, uint32_t* C, uint32_t* K) {
  const unsigned long long off = A.off[i];
  const uint32_t cnt = A.cnt[i];
  const int len = uniform((int)row_len(A, off, cnt));
  if (len != uniform((int)cnt)) return;  // beyond the capacity, or cut by it
  const int m = (len + kWave - 1) / kWave;
  uint32_t key[kPer];
  uint32_t lo = 0xffffffffu, hi = 0u;
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    key[u] = 0u;
    if (u < m) {
      const int t = u * kWave + lane;
      C[t] = 0u;
      if (t < len) {
        key[u] = A.row_j[off + (uint32_t)t];
        lo = min(lo, key[u]);
        hi = max(hi, key[u]);
      }
    }
  }
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) {
    lo = min(lo, (uint32_t)__shfl_xor((int)lo, d, kWave));
    hi = max(hi, (uint32_t)__shfl_xor((int)hi, d, kWave));
  }
  const int nb = m * kWave;
  const float scale = (float)nb / ((float)(hi - lo) + 1.0f);
  uint32_t b[kPer], p[kPer];
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    b[u] = p[u] = 0u;
    if (u < m && u * kWave + lane < len) {
      b[u] = min((uint32_t)((float)(key[u] - lo) * scale), (uint32_t)(nb - 1));  // not decreasing in key
      p[u] = atomicAdd(&C[b[u]], 1u);
    }
  }
  __builtin_amdgcn_wave_barrier();
  // bucket starts: lane L holds buckets m L .. m L + m - 1
  uint32_t s = 0u;
  for (int u = 0; u < m; ++u) s += C[lane * m + u];
  uint32_t x = s;
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) {
    const uint32_t y = (uint32_t)__shfl_up((int)x, d, kWave);
    if (lane >= d) x += y;
  }
  uint32_t o = x - s;
  for (int u = 0; u < m; ++u) {
    const uint32_t c = C[lane * m + u];
    C[lane * m + u] = o;
    o += c;
  }
  if (lane == kWave - 1) C[nb] = o;
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int u = 0; u < kPer; ++u)
    if (u < m && u * kWave + lane < len) K[C[b[u]] + p[u]] = key[u];
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    if (u < m && u * kWave + lane < len) {
      const uint32_t st = C[b[u]], en = C[b[u] + 1];
      p[u] = st;
      for (uint32_t k = st; k < en; ++k) p[u] += K[k] < key[u] ? 1u : 0u;
    }
  }
  __builtin_amdgcn_wave_barrier();
  // in order in LDS first: the list is written in whole lines
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    const int t = u * kWave + lane;
    if (u < m && t < len) {
      K[p[u]] = key[u];
      C[p[u]] = (uint32_t)t;
    }
  }
  __builtin_amdgcn_wave_barrier();
  for (int r = lane; r < len; r += kWave) put(A, i, off, C[r], (uint32_t)r, K[r]);
  __builtin_amdgcn_wave_barrier();
}

// kRowsPer rows a wave, one after the other: a block for every four rows costs
// more than the rows where they hold an entry or two.
constexpr int kRowsPer = 4;

__global__ void __launch_bounds__(256) row_short_kernel(RowArgs A) {
  __shared__ uint32_t C[4][kRow0 + 1], K[4][kRow0];
  const int lane = (int)__lane_id(), wid = uniform((int)threadIdx.x / kWave);
  const long long i0 = ((long long)blockIdx.x * 4 + wid) * kRowsPer;
  for (int k = 0; k < kRowsPer && i0 + k < A.n; ++k) {
    const int i = (int)i0 + k;
    const uint32_t cnt = A.cnt[i];
    if (cnt > 1u) {
      if (row_class(cnt) == 0) sort_row<kRow0 / kWave>(A, i, lane, C[wid], K[wid]);
    } else if (cnt == 1u && lane == 0) {
      const unsigned long long off = A.off[i];
      if (row_len(A, off, 1u)) put(A, i, off, 0u, 0u, A.row_j[off]);
    }
  }
}

union LongLds {
  uint32_t wave[kLongThreads / kWave][2 * kRow1 + 1];
  uint64_t key[kRow2];
  struct {
    uint32_t bits[kBitWords], pre[kBitWords], ws[kLongThreads / kWave], wb[kLongThreads / kWave];
  } map;
};

// The cut row: its smallest partners, by one block from the bit map.
__device__ __forceinline__ void write_cut_row(const RowArgs& A, LongLds& L) {
  const uint32_t i = A.longs[3];
  if (i == 0xffffffffu) return;
  const int t = (int)threadIdx.x, lane = t % kWave, wid = t / kWave;
  const unsigned long long off = A.off[i];
  const uint32_t len = row_len(A, off, A.cnt[i]);
  const int per = (A.nbits + kLongThreads - 1) / kLongThreads;
  const int k0 = min(t * per, A.nbits), k1 = min(k0 + per, A.nbits);
  uint32_t s = 0u;
  for (int k = k0; k < k1; ++k) s += (uint32_t)__popc(A.bits[k]);
  uint32_t x = s;
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) {
    const uint32_t y = (uint32_t)__shfl_up((int)x, d, kWave);
    if (lane >= d) x += y;
  }
  if (lane == kWave - 1) L.map.ws[wid] = x;
  __syncthreads();
  uint32_t r = x - s;
  for (int k = 0; k < wid; ++k) r += L.map.ws[k];
  for (int k = k0; k < k1 && r < len; ++k)
    for (uint32_t w = A.bits[k]; w != 0u && r < len; w &= w - 1u, ++r) {
      const uint32_t j = 32u * (uint32_t)k + (uint32_t)__builtin_ctz(w);
      ((int2*)A.pairs)[off + r] = make_int2((int)i, (int)j);
      if (A.dj) A.dist[off + r] = A.dj[j];
    }
}

// The rows of the longer classes, over a grid that stays (often there are none);
// the last block: the cut row.
__global__ void __launch_bounds__(kLongThreads) row_long_kernel(RowArgs A, int windows) {
  __shared__ LongLds L;
  const unsigned nblk = gridDim.x - 1;
  if (blockIdx.x == nblk) {
    write_cut_row(A, L);
    return;
  }
  const int t0 = (int)threadIdx.x, lane = t0 % kWave, wid = uniform(t0 / kWave);
  {
    uint32_t* C = L.wave[wid];
    const uint32_t nrow = A.longs[0];
    for (uint32_t q = blockIdx.x * (kLongThreads / kWave) + (uint32_t)wid; q < nrow;
         q += nblk * (kLongThreads / kWave))
      sort_row<kRow1 / kWave>(A, (int)long_row(A, 0, q), lane, C, C + kRow1 + 1);
  }
  // a block each: a bitonic sort of (partner, entry)
  for (uint32_t q = blockIdx.x; q < A.longs[1]; q += nblk) {
    const int i = (int)long_row(A, 1, q);
    const unsigned long long off = A.off[i];
    const int len = (int)row_len(A, off, A.cnt[i]);
    int P = 2048;
    while (P < len) P *= 2;
    __syncthreads();
    for (int t = t0; t < P; t += kLongThreads)
      L.key[t] = t < len ? ((uint64_t)A.row_j[off + (uint32_t)t] << 13) | (uint64_t)t : ~0ull;
    __syncthreads();
    for (int k = 2; k <= P; k *= 2) {
      for (int d = k / 2; d > 0; d /= 2) {
        for (int t = t0; t < P / 2; t += kLongThreads) {
          const int a = 2 * t - (t & (d - 1)), b = a + d;
          const uint64_t u = L.key[a], v = L.key[b];
          if ((u > v) == ((a & k) == 0)) {
            L.key[a] = v;
            L.key[b] = u;
          }
        }
        __syncthreads();
      }
    }
    for (int t = t0; t < len; t += kLongThreads)
      put(A, i, off, (uint32_t)(L.key[t] & (kRow2 - 1)), (uint32_t)t, (uint32_t)(L.key[t] >> 13));
  }
  // a block per row and window of 2^18 indices: the places of the window's
  // partners from its bit map and the number of smaller ones
  const unsigned long long items = (unsigned long long)A.longs[2] * (unsigned)windows;
  for (unsigned long long q = blockIdx.x; q < items; q += nblk) {
    uint32_t* bits = L.map.bits;
    constexpr int kPer = kBitWords / kLongThreads;
    const int i = (int)long_row(A, 2, (uint32_t)(q / (unsigned)windows));
    const uint32_t win = (uint32_t)(q % (unsigned)windows);
    const unsigned long long off = A.off[i];
    const uint32_t len = row_len(A, off, A.cnt[i]);
    __syncthreads();
    for (int k = t0; k < kBitWords; k += kLongThreads) bits[k] = 0u;
    __syncthreads();
    uint32_t below = 0u;
    for (uint32_t t = (uint32_t)t0; t < len; t += kLongThreads) {
      const uint32_t j = A.row_j[off + t], w = j / (32u * kBitWords);
      below += w < win ? 1u : 0u;
      if (w == win) atomicOr(&bits[(j / 32u) % kBitWords], 1u << (j % 32u));
    }
    __syncthreads();
    uint32_t s = 0u;
#pragma unroll
    for (int k = 0; k < kPer; ++k) s += (uint32_t)__popc(bits[t0 * kPer + k]);
    uint32_t x = s;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
      const uint32_t y = (uint32_t)__shfl_up((int)x, d, kWave);
      if (lane >= d) x += y;
    }
    below = wave_sum_u32(below);
    if (lane == kWave - 1) L.map.ws[wid] = x;
    if (lane == 0) L.map.wb[wid] = below;
    __syncthreads();
    uint32_t o = x - s;
#pragma unroll
    for (int k = 0; k < kLongThreads / kWave; ++k) o += L.map.wb[k] + (k < wid ? L.map.ws[k] : 0u);
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      L.map.pre[t0 * kPer + k] = o;
      o += (uint32_t)__popc(bits[t0 * kPer + k]);
    }
    __syncthreads();
    for (uint32_t t = (uint32_t)t0; t < len; t += kLongThreads) {
      const uint32_t j = A.row_j[off + t];
      if (j / (32u * kBitWords) == win) {
        const uint32_t w = (j / 32u) % kBitWords;
        put(A, i, off, t, L.map.pre[w] + (uint32_t)__popc(bits[w] & ((1u << (j % 32u)) - 1u)), j);
      }
    }
  }
}

}  // namespace

int row_scan_blocks(int n) { return (int)(((long long)n + kScanRows - 1) / kScanRows); }

hipError_t launch_row_offsets(const RowArgs& A, hipStream_t s) {
  row_sums_kernel<<<row_scan_blocks(A.n), kScanThreads, 0, s>>>(A);
  row_offsets_kernel<<<row_scan_blocks(A.n), kScanThreads, 0, s>>>(A);
  return hipGetLastError();
}

// nj: the partners' index range
hipError_t launch_row_sort(const RowArgs& A, long long nj, hipStream_t s) {
  row_short_kernel<<<(unsigned)(((long long)A.n + 4 * kRowsPer - 1) / (4 * kRowsPer)), 256, 0, s>>>(A);
  const int windows = (int)((nj + 32 * kBitWords - 1) / (32 * kBitWords));
  row_long_kernel<<<256, kLongThreads, 0, s>>>(A, windows);  // (one a CU)
  return hipGetLastError();
}

}  // namespace clm
