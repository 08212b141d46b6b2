// CountSketch on gfx950: hash, stable binning of rows by bucket, and the
// bucket-owned row reduction that forms S*A.
//
// Paper mapping (arXiv 2203.02798): the hash is Definition 3; the binned row
// list is the Block-Column CountSketch of section 2.3 (b_r = r: per bucket a
// list of signed row indices, n indices in total); the reduction is Algorithm
// bcs_multiply with one bucket's rows summed by one wavefront, so no two
// workers ever write the same output row (no atomics, deterministic order).
//
// Binning is a stable LSD radix sort of (bucket, row|sign) pairs with equal
// digits of up to 10 bits: per 2048-key tile a digit histogram, one exclusive
// scan over (digit, tile), then a stable scatter whose in-tile ranks come from
// wavefront ballots.  The first pass hashes its keys itself, twice, instead of
// reading them.  Stability keeps each bucket's rows in increasing row order,
// which fixes the summation order.  Few keys are bound by launches, many by
// the passes' reads and scattered writes, so both are kept few: up to 1024
// buckets take one pass and four launches, up to 2^20 two passes (8-bit
// digits, stored keys and three launches a scan before: twelve launches of
// 51 us in all for 1e4 rows in 1024 buckets, now four of 25).
#include <utility>

#include "internal.hpp"

namespace psk {
namespace {

constexpr int kDigitBits = 10;  // at most; kSortThreads threads own 4 digits each
constexpr int kSortThreads = 256;
constexpr int kSortItems = 8;
constexpr int kSortWaves = kSortThreads / 64;
constexpr int kSortTile = kSortThreads * kSortItems;  // 2048 keys per block
constexpr int kOwnDigits = (1 << kDigitBits) / kSortThreads;
constexpr int kScanThreads = 256;
constexpr int kScanItems = 16;
constexpr int kScanTile = kScanThreads * kScanItems;  // 4096 per block

// ---------------------------------------------------------------------------
// hash
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_hash_export(int64_t row0, int64_t count,
                                                     uint32_t r, uint64_t seed,
                                                     int32_t *__restrict__ h,
                                                     int8_t *__restrict__ sign) {
  const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= count) return;
  uint32_t b, neg;
  cs_hash_row((uint64_t)(row0 + j), r, seed, b, neg);
  if (h) h[j] = (int32_t)b;
  if (sign) sign[j] = neg ? (int8_t)-1 : (int8_t)1;
}

// Where a sort pass takes pair j from.
struct StoredPairs {
  const uint32_t *keys, *vals;
  __device__ __forceinline__ void get(int64_t j, uint32_t &k, uint32_t &v) const {
    k = keys[j];
    v = vals[j];
  }
};

// row j of a dense A
struct HashedRows {
  uint32_t r;
  uint64_t seed;
  __device__ __forceinline__ void get(int64_t j, uint32_t &k, uint32_t &v) const {
    uint32_t neg;
    cs_hash_row((uint64_t)j, r, seed, k, neg);
    v = (uint32_t)j | (neg << 31);
  }
};

// OSNAP with s non-zeros per row of A (block construction): pair j = i s + k
// is non-zero k of row i, so each row's s entries are adjacent and, after the
// stable sort, every bucket lists its rows in increasing order
struct HashedOsnap {
  uint32_t s, rb;
  uint64_t seed;
  __device__ __forceinline__ void get(int64_t j, uint32_t &k, uint32_t &v) const {
    const int64_t i = j / s;
    uint32_t neg;
    osnap_hash_nz((uint64_t)i, (uint32_t)(j - i * s), rb, seed, k, neg);
    v = (uint32_t)i | (neg << 31);
  }
};

// the listed rows of a CSR A, s non-zeros each (s = 1: the CountSketch hash,
// non-zero 0 with rb = r)
struct HashedList {
  const uint32_t *rows;
  uint32_t s, rb;
  uint64_t seed;
  __device__ __forceinline__ void get(int64_t j, uint32_t &k, uint32_t &v) const {
    const int64_t q = j / s;
    const uint32_t i = rows[q];
    uint32_t neg;
    osnap_hash_nz((uint64_t)i, (uint32_t)(j - q * s), rb, seed, k, neg);
    v = i | (neg << 31);
  }
};

__global__ __launch_bounds__(256) void k_hash_export_osnap(int64_t row0, int64_t pairs,
                                                           uint32_t s, uint32_t rb,
                                                           uint64_t seed,
                                                           int32_t *__restrict__ h,
                                                           int8_t *__restrict__ sign) {
  const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= pairs) return;
  const int64_t i = j / s;
  const uint32_t k = (uint32_t)(j - i * s);
  uint32_t b, neg;
  osnap_hash_nz((uint64_t)(row0 + i), k, rb, seed, b, neg);
  if (h) h[j] = (int32_t)b;
  if (sign) sign[j] = neg ? (int8_t)-1 : (int8_t)1;
}

template <int THREADS>
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t t, uint32_t &total) {
  __shared__ uint32_t wsum[THREADS / 64];
  const int lane = threadIdx.x & 63;
  const int w = threadIdx.x >> 6;
  uint32_t inc = t;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t y = __shfl_up(inc, off, 64);
    if (lane >= off) inc += y;
  }
  if (lane == 63) wsum[w] = inc;
  __syncthreads();
  uint32_t pre = 0;
  total = 0;
#pragma unroll
  for (int q = 0; q < THREADS / 64; ++q) {
    if (q < w) pre += wsum[q];
    total += wsum[q];
  }
  __syncthreads();
  return pre + inc - t;
}

// sum of sums[0 .. b - 1] over the workgroup, loads side by side
__device__ __forceinline__ uint32_t sum_before(const uint32_t *__restrict__ sums, int64_t b) {
  uint32_t t = 0, total;
#pragma unroll 4
  for (int64_t i = threadIdx.x; i < b; i += kScanThreads) t += sums[i];
  block_excl_scan<kScanThreads>(t, total);
  return total;
}

// Tiles whose sums every tile may add up itself (16 loads a thread).
constexpr int64_t kPairTiles = 4096;

// CSR A: only rows that hold an entry are binned (an empty row adds nothing
// to any sum, so the bins and the sums of the others are unchanged).  Tile t
// is rounds x 4096 rows, a wavefront takes 1024 in a row at a time; the first
// launch counts a tile's rows, the second lists them from the sum of the
// tiles before it: the row pointers are read twice and the list written once
// (flags, a scan of them and a compaction took five launches; n = 1e7: 81 us
// then, 31 now).
constexpr int kListRows = 4096;

template <bool LIST>
__global__ __launch_bounds__(256) void k_row_list(const int64_t *__restrict__ indptr, int64_t n,
                                                  int rounds, uint32_t s,
                                                  uint32_t *__restrict__ sums,
                                                  uint32_t *__restrict__ rows,
                                                  uint32_t *__restrict__ cnt) {
  __shared__ uint32_t wc[2][4];
  constexpr int IT = kListRows / 256;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  uint32_t at = LIST ? sum_before(sums, blockIdx.x) : 0u;  // rows listed before this round
  for (int q = 0; q < rounds; ++q) {
    const int64_t base = ((int64_t)blockIdx.x * rounds + q) * kListRows + w * (IT * 64);
    int64_t p0[IT], p1[IT];
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const int64_t i = base + it * 64 + lane;
      p0[it] = indptr[i < n ? i : n];
      p1[it] = indptr[i < n ? i + 1 : n];
    }
    uint64_t m[IT];
    uint32_t c = 0;
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      m[it] = __ballot(p1[it] > p0[it]);
      c += (uint32_t)__popcll(m[it]);
    }
    if (lane == 0) wc[q & 1][w] = c;
    __syncthreads();
    uint32_t pos = at;
    for (int v = 0; v < w; ++v) pos += wc[q & 1][v];
    at += wc[q & 1][0] + wc[q & 1][1] + wc[q & 1][2] + wc[q & 1][3];
    if constexpr (LIST) {
      const uint64_t lt = lane == 0 ? 0ull : ((~0ull) >> (64 - lane));
#pragma unroll
      for (int it = 0; it < IT; ++it) {
        if ((m[it] >> lane) & 1)
          rows[pos + (uint32_t)__popcll(m[it] & lt)] = (uint32_t)(base + it * 64 + lane);
        pos += (uint32_t)__popcll(m[it]);
      }
    }
  }
  if (!LIST && threadIdx.x == 0) sums[blockIdx.x] = at;
  // cnt[0] = rows listed, cnt[1] = s times that (the pairs to bin)
  if (LIST && threadIdx.x == 0 && blockIdx.x == gridDim.x - 1) {
    cnt[0] = at;
    cnt[1] = at * s;
  }
}

// ---------------------------------------------------------------------------
// radix sort pass: per-tile digit histogram (digit-major layout)
// ---------------------------------------------------------------------------
// The keys in use: n, or the count at dn (at most n) when given.  Tiles past
// them neither write nor are scanned: the layout is that of the tiles in use.
__device__ __forceinline__ int64_t keys_in_use(int64_t n, const uint32_t *dn) {
  return dn ? (int64_t)dn[0] : n;
}

template <class SRC>
__global__ __launch_bounds__(kSortThreads) void k_radix_hist(SRC src, int64_t n,
                                                             const uint32_t *__restrict__ dn,
                                                             int shift, int nbits,
                                                             uint32_t *__restrict__ hist) {
  __shared__ uint32_t h[1 << kDigitBits];
  n = keys_in_use(n, dn);
  const int64_t base = (int64_t)blockIdx.x * kSortTile;
  if (base >= n) return;
  const int64_t ntiles = ceil_div(n, (int64_t)kSortTile);
  const int D = 1 << nbits;
  const uint32_t mask = (uint32_t)D - 1u;
  for (int e = threadIdx.x; e < D; e += kSortThreads) h[e] = 0;
  __syncthreads();
#pragma unroll
  for (int it = 0; it < kSortItems; ++it) {
    const int64_t idx = base + it * kSortThreads + threadIdx.x;
    if (idx < n) {
      uint32_t k, v;
      src.get(idx, k, v);
      atomicAdd(&h[(k >> shift) & mask], 1u);
    }
  }
  __syncthreads();
  for (int e = threadIdx.x; e < D; e += kSortThreads) hist[e * ntiles + blockIdx.x] = h[e];
}

// Stable scatter of one tile.  A wavefront takes 512 keys of the tile in a
// row, 64 at a time: ranks come from ballots and from its own running counts
// of the digits in LDS (no barrier in the loop).  The counts of the
// wavefronts and the tile's digit starts then place each key in LDS at its
// digit's tile-local run, and the tile is written out run by run, consecutive
// threads to consecutive addresses of a digit's run in kout / vout (instead of
// every key straight to its own run).  The tile's count of a digit is the
// difference of two neighbouring scanned offsets.
template <class SRC>
__global__ __launch_bounds__(kSortThreads) void k_radix_scatter(
    SRC src, int64_t n, const uint32_t *__restrict__ dn, int shift, int nbits,
    const uint32_t *__restrict__ offs, uint32_t *__restrict__ kout, uint32_t *__restrict__ vout) {
  extern __shared__ uint32_t counts[];  // per wavefront, then start and target of each digit's run
  __shared__ uint32_t sk[kSortTile], sv[kSortTile];
  n = keys_in_use(n, dn);
  const int64_t base = (int64_t)blockIdx.x * kSortTile;
  if (base >= n) return;  // nothing of this tile in use
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
  const int D = 1 << nbits;
  const uint32_t mask = (uint32_t)D - 1u;
  const int64_t ntiles = ceil_div(n, (int64_t)kSortTile);
  volatile uint32_t *mine = counts + w * D;
  uint32_t *lstart = counts + kSortWaves * D, *goff = lstart + D;
  for (int e = tid; e < kSortWaves * D; e += kSortThreads) counts[e] = 0;
  uint32_t k[kSortItems], v[kSortItems];
#pragma unroll
  for (int it = 0; it < kSortItems; ++it) {
    const int64_t idx = base + (w * kSortItems + it) * 64 + lane;
    k[it] = v[it] = 0u;
    if (idx < n) src.get(idx, k[it], v[it]);
  }
  // this thread's digits (own in a row): where the tile's runs go and start
  const int own = D > kSortThreads ? D / kSortThreads : 1;
  uint32_t g0[kOwnDigits], len[kOwnDigits], sum = 0;
#pragma unroll
  for (int i = 0; i < kOwnDigits; ++i) {
    const int dg = tid * own + i;
    g0[i] = len[i] = 0u;
    if (i < own && dg < D) {
      const int64_t o = (int64_t)dg * ntiles + blockIdx.x;
      g0[i] = offs[o];
      len[i] = (o + 1 < (int64_t)D * ntiles ? offs[o + 1] : (uint32_t)n) - g0[i];
    }
    sum += len[i];
  }
  uint32_t total;
  uint32_t run = block_excl_scan<kSortThreads>(sum, total);  // counts are zero behind its barriers
#pragma unroll
  for (int i = 0; i < kOwnDigits; ++i) {
    const int dg = tid * own + i;
    if (i < own && dg < D) {
      lstart[dg] = run;
      goff[dg] = g0[i];
    }
    run += len[i];
  }
  const uint64_t lt = lane == 0 ? 0ull : ((~0ull) >> (64 - lane));
  uint32_t rank[kSortItems];
#pragma unroll
  for (int it = 0; it < kSortItems; ++it) {
    const bool valid = base + (w * kSortItems + it) * 64 + lane < n;
    const uint32_t dg = (k[it] >> shift) & mask;
    uint64_t peers = __ballot(valid);
    for (int b = 0; b < nbits; ++b) {
      const bool bit = (dg >> b) & 1u;
      const uint64_t bb = __ballot(bit);
      peers &= bit ? bb : ~bb;
    }
    const uint32_t among = (uint32_t)__popcll(peers & lt);
    const uint32_t before = valid ? mine[dg] : 0u;
    rank[it] = before + among;
    // the first of equal digits counts them all, after every lane has read
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (valid && among == 0) mine[dg] = before + (uint32_t)__popcll(peers);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
  __syncthreads();
  // where each wavefront's keys of a digit start in the tile
  for (int e = tid; e < D; e += kSortThreads) {
    uint32_t at = lstart[e];
#pragma unroll
    for (int q = 0; q < kSortWaves; ++q) {
      const uint32_t c = counts[q * D + e];
      counts[q * D + e] = at;
      at += c;
    }
  }
  __syncthreads();
#pragma unroll
  for (int it = 0; it < kSortItems; ++it) {
    if (base + (w * kSortItems + it) * 64 + lane < n) {
      const uint32_t pos = mine[(k[it] >> shift) & mask] + rank[it];
      sk[pos] = k[it];
      sv[pos] = v[it];
    }
  }
  __syncthreads();
  const int cnt = (int)(n - base < kSortTile ? n - base : kSortTile);
  for (int e = tid; e < cnt; e += kSortThreads) {
    const uint32_t key = sk[e];
    const uint32_t dg = (key >> shift) & mask;
    const uint32_t pos = goff[dg] + ((uint32_t)e - lstart[dg]);
    kout[pos] = key;
    vout[pos] = sv[e];
  }
}

// ---------------------------------------------------------------------------
// exclusive scan of uint32 in place
// ---------------------------------------------------------------------------
// Up to kScanOne values one workgroup does it all.  Up to kPairTiles tiles in
// two launches: the tiles' sums, then every tile scans its values from the
// sum of the tiles before it, which it adds up itself; the values are read
// twice and written once.  More tiles: their sums are scanned in between.
// (Three launches that wrote every value twice before: 42 us on average for
// the scans of a 1e7-row CSR sketch, now 26.)
// dn: the values in use are those of per-tile counts of dn[0] keys (D digits).
constexpr int kScanOneThreads = 1024;
constexpr int64_t kScanOne = (int64_t)kScanOneThreads * kScanItems;

__device__ __forceinline__ int64_t scan_length(int64_t L, const uint32_t *dn, int D) {
  return dn ? (int64_t)D * ceil_div((int64_t)dn[0], (int64_t)kSortTile) : L;
}

template <int THREADS>
__device__ __forceinline__ void scan_tile(uint32_t *__restrict__ data, int64_t L, int64_t tile,
                                          uint32_t first) {
  const int64_t base = (tile * THREADS + threadIdx.x) * kScanItems;
  uint32_t v[kScanItems], t = 0, total;
#pragma unroll
  for (int i = 0; i < kScanItems; ++i) {
    v[i] = base + i < L ? data[base + i] : 0u;
    t += v[i];
  }
  uint32_t run = first + block_excl_scan<THREADS>(t, total);
#pragma unroll
  for (int i = 0; i < kScanItems; ++i) {
    if (base + i < L) data[base + i] = run;
    run += v[i];
  }
}

__global__ __launch_bounds__(kScanOneThreads) void k_scan_one(uint32_t *__restrict__ data,
                                                              int64_t L,
                                                              const uint32_t *__restrict__ dn,
                                                              int D) {
  scan_tile<kScanOneThreads>(data, scan_length(L, dn, D), 0, 0u);
}

__global__ __launch_bounds__(kScanThreads) void k_scan_tiles(const uint32_t *__restrict__ data,
                                                             int64_t L,
                                                             const uint32_t *__restrict__ dn,
                                                             int D,
                                                             uint32_t *__restrict__ sums) {
  L = scan_length(L, dn, D);
  const int64_t base = (int64_t)blockIdx.x * kScanTile;
  if (base >= L) return;
  uint32_t t = 0, total;
#pragma unroll
  for (int i = 0; i < kScanItems; ++i) {
    const int64_t e = base + i * kScanThreads + threadIdx.x;
    t += e < L ? data[e] : 0u;
  }
  block_excl_scan<kScanThreads>(t, total);
  if (threadIdx.x == 0) sums[blockIdx.x] = total;
}

__global__ __launch_bounds__(kScanThreads) void k_scan_sums(uint32_t *__restrict__ sums,
                                                            int64_t nb) {
  uint32_t carry = 0;
  for (int64_t c0 = 0; c0 < nb; c0 += kScanTile) {
    const int64_t base = c0 + (int64_t)threadIdx.x * kScanItems;
    uint32_t v[kScanItems];
    uint32_t t = 0;
#pragma unroll
    for (int i = 0; i < kScanItems; ++i) {
      v[i] = (base + i < nb) ? sums[base + i] : 0u;
      t += v[i];
    }
    uint32_t total;
    uint32_t run = carry + block_excl_scan<kScanThreads>(t, total);
#pragma unroll
    for (int i = 0; i < kScanItems; ++i) {
      if (base + i < nb) sums[base + i] = run;
      run += v[i];
    }
    carry += total;
  }
}

// SUMMED: sums holds the scanned sums
template <bool SUMMED>
__global__ __launch_bounds__(kScanThreads) void k_scan_apply(uint32_t *__restrict__ data,
                                                             int64_t L,
                                                             const uint32_t *__restrict__ dn,
                                                             int D,
                                                             const uint32_t *__restrict__ sums) {
  L = scan_length(L, dn, D);
  const int64_t b = blockIdx.x;
  if (b * kScanTile >= L) return;
  scan_tile<kScanThreads>(data, L, b, SUMMED ? sums[b] : sum_before(sums, b));
}

int scan_plan_impl(int64_t L, Arena &ws, uint32_t **sums) {
  *sums = ws.take<uint32_t>((size_t)ceil_div(L, kScanTile) + 1);
  return 0;
}

void scan_run_impl(uint32_t *data, int64_t L, uint32_t *sums, hipStream_t st,
                   const uint32_t *dn = nullptr, int D = 0) {
  if (L <= kScanOne) {
    k_scan_one<<<1, kScanOneThreads, 0, st>>>(data, L, dn, D);
    return;
  }
  const int64_t nb = ceil_div(L, kScanTile);
  k_scan_tiles<<<(unsigned)nb, kScanThreads, 0, st>>>(data, L, dn, D, sums);
  if (nb <= kPairTiles) {
    k_scan_apply<false><<<(unsigned)nb, kScanThreads, 0, st>>>(data, L, dn, D, sums);
  } else {
    // (sums of tiles not in use are not written, nor read where it counts)
    k_scan_sums<<<1, kScanThreads, 0, st>>>(sums, nb);
    k_scan_apply<true><<<(unsigned)nb, kScanThreads, 0, st>>>(data, L, dn, D, sums);
  }
}

// bucket b's range starts at the first sorted position whose key is >= b
__global__ __launch_bounds__(256) void k_bucket_ptr(const uint32_t *__restrict__ skeys,
                                                    int64_t n, const uint32_t *__restrict__ dn,
                                                    uint32_t r, uint32_t *__restrict__ bptr) {
  const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  n = keys_in_use(n, dn);
  if (j > n) return;
  const int64_t prev = j > 0 ? (int64_t)skeys[j - 1] : -1;
  const int64_t cur = j < n ? (int64_t)skeys[j] : (int64_t)r;
  for (int64_t b = prev + 1; b <= cur; ++b) bptr[b] = (uint32_t)j;
}

// The same pointers with the key count on the device: one thread per
// bucket b in [0, r], bptr[b] = the first position whose key is >= b
// (a binary search, so the work stays bounded when the keys in use are few
// and the buckets many).
__global__ __launch_bounds__(256) void k_bucket_ptr_search(const uint32_t *__restrict__ skeys,
                                                           const uint32_t *__restrict__ dn,
                                                           uint32_t r,
                                                           uint32_t *__restrict__ bptr) {
  const int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (b > (int64_t)r) return;
  uint32_t lo = 0, hi = dn[0];
  while (lo < hi) {
    const uint32_t mid = lo + ((hi - lo) >> 1);
    if ((int64_t)skeys[mid] < b) lo = mid + 1;
    else hi = mid;
  }
  bptr[b] = lo;
}


// ---------------------------------------------------------------------------
// S*A, dense A: one wavefront per (bucket, split); each lane owns VW adjacent
// columns in each of CH column groups, accumulating in registers.
// ---------------------------------------------------------------------------
template <typename T, int VW>
struct Vec;
template <>
struct Vec<double, 1> { typedef double type; };
template <>
struct Vec<double, 2> { typedef double2 type; };
template <>
struct Vec<float, 1> { typedef float type; };
template <>
struct Vec<float, 2> { typedef float2 type; };
template <>
struct Vec<float, 4> { typedef float4 type; };
template <>
struct Vec<double, 4> { typedef double4 type; };

template <typename T, int VW>
__device__ __forceinline__ void vload(const T *p, T (&x)[VW]) {
  typedef typename Vec<T, VW>::type V;
  const V v = *reinterpret_cast<const V *>(p);
  const T *e = reinterpret_cast<const T *>(&v);
#pragma unroll
  for (int q = 0; q < VW; ++q) x[q] = e[q];
}

template <typename T, int VW>
__device__ __forceinline__ void vstore(T *p, const T (&x)[VW]) {
  typedef typename Vec<T, VW>::type V;
  V v;
  T *e = reinterpret_cast<T *>(&v);
#pragma unroll
  for (int q = 0; q < VW; ++q) e[q] = x[q];
  *reinterpret_cast<V *>(p) = v;
}

// VW adjacent outputs: one vector store where the vector type exists (the
// row of out is aligned whenever the loads of A are), else element stores
template <typename TO, int VW>
__device__ __forceinline__ void store_out(TO *p, const TO (&x)[VW]) {
  if constexpr (sizeof(TO) * VW <= 16) {
    vstore<TO, VW>(p, x);
  } else {
#pragma unroll
    for (int q = 0; q < VW; q += 2) {
      const TO y[2] = {x[q], x[q + 1]};
      vstore<TO, 2>(p + q, y);
    }
  }
}

// The U rows of a batch are loaded together and branch-free (a row past the
// bucket, or columns past d, load an element of row 0 at column 0 and are
// masked), so all of them are in flight at once, and the bin entries of the
// next batch are loaded while this one is summed.  Rows are added in bin
// order, in FP64.
template <typename T, typename TO, int VW, int CH, int U>
__global__ __launch_bounds__(256) void k_scatter_dense(
    const T *__restrict__ A, int64_t ld, int64_t d, int64_t r,
    const uint32_t *__restrict__ perm, const uint32_t *__restrict__ bptr,
    int splits, double scale, TO *__restrict__ out) {
  const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  if (wave >= r * splits) return;
  const int64_t b = wave / splits;
  const int s = (int)(wave - b * splits);
  const uint32_t lo = bptr[b];
  const uint32_t len = bptr[b + 1] - lo;
  const uint32_t j0 = lo + (uint32_t)(((uint64_t)len * s) / splits);
  const uint32_t j1 = lo + (uint32_t)(((uint64_t)len * (s + 1)) / splits);
  TO *orow = out + ((int64_t)s * r + b) * d;
  const int lane = threadIdx.x & 63;
  constexpr int64_t kSpan = 64 * VW * CH;
  for (int64_t c0 = 0; c0 < d; c0 += kSpan) {
    double acc[CH][VW];
#pragma unroll
    for (int c = 0; c < CH; ++c)
#pragma unroll
      for (int q = 0; q < VW; ++q) acc[c][q] = 0.0;
    // column offsets of this lane's groups, clamped to 0 past d
    int64_t coff[CH];
    bool cok[CH];
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      const int64_t col = c0 + (int64_t)(c * 64 + lane) * VW;
      cok[c] = col < d;
      coff[c] = cok[c] ? col : 0;
    }
    uint32_t pv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) pv[u] = perm[(j0 + u < j1) ? j0 + u : lo];
    for (uint32_t j = j0; j < j1; j += U) {
      T x[U][CH][VW];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const bool rok = j + u < j1;
        const int64_t row = rok ? (int64_t)(pv[u] & 0x7fffffffu) : 0;
#pragma unroll
        for (int c = 0; c < CH; ++c) vload<T, VW>(A + row * ld + coff[c], x[u][c]);
      }
      double sg[U];
#pragma unroll
      for (int u = 0; u < U; ++u) sg[u] = (j + u < j1) ? ((pv[u] >> 31) ? -1.0 : 1.0) : 0.0;
      // the next batch's bin entries
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const uint32_t jn = j + U + u;
        pv[u] = perm[jn < j1 ? jn : lo];
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int c = 0; c < CH; ++c)
#pragma unroll
          for (int q = 0; q < VW; ++q) {
            const double xv = cok[c] ? (double)x[u][c][q] : 0.0;
            acc[c][q] = fma(sg[u], xv, acc[c][q]);
          }
    }
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      if (cok[c]) {
        TO ov[VW];
#pragma unroll
        for (int q = 0; q < VW; ++q) ov[q] = (TO)(acc[c][q] * scale);
        store_out<TO, VW>(orow + coff[c], ov);
      }
    }
  }
}

// ---------------------------------------------------------------------------
// S*A, CSR A: one wavefront per (bucket, split) with a private LDS row of d
// FP64 accumulators; rows of the bucket are applied one after another
// (bucket_rows_add).
// ---------------------------------------------------------------------------
template <typename T, typename TO>
__global__ __launch_bounds__(256) void k_scatter_csr(
    const T *__restrict__ vals, const int64_t *__restrict__ indptr,
    const int32_t *__restrict__ indices, int64_t d, int64_t dpad, int64_t r,
    const uint32_t *__restrict__ perm, const uint32_t *__restrict__ bptr,
    int splits, double scale, TO *__restrict__ out) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  double *acc = reinterpret_cast<double *>(smem_raw) + (threadIdx.x >> 6) * dpad;
  const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  if (wave >= r * splits) return;
  const int lane = threadIdx.x & 63;
  const int64_t b = wave / splits;
  const int s = (int)(wave - b * splits);
  const uint32_t lo = bptr[b];
  const uint32_t len = bptr[b + 1] - lo;
  const uint32_t j0 = lo + (uint32_t)(((uint64_t)len * s) / splits);
  const uint32_t j1 = lo + (uint32_t)(((uint64_t)len * (s + 1)) / splits);
  for (int64_t c = lane; c < d; c += 64) acc[c] = 0.0;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  bucket_rows_add(vals, indptr, indices, perm, j0, j1, acc);
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  TO *orow = out + ((int64_t)s * r + b) * d;
  for (int64_t c = lane; c < d; c += 64) orow[c] = (TO)(acc[c] * scale);
}

// SA[b, c] = sum over splits of partial[s, b, c] (FP64), splits in
// increasing order, rounded once to the output type
template <typename TO>
__global__ __launch_bounds__(256) void k_combine_splits(const double *__restrict__ part,
                                                        int64_t rd, int splits,
                                                        double scale,
                                                        TO *__restrict__ SA) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= rd) return;
  double acc = part[e];
  for (int s = 1; s < splits; ++s) acc += part[(int64_t)s * rd + e];
  SA[e] = (TO)(acc * scale);
}

int choose_splits(int64_t n, int64_t r) {
  // Enough wavefronts to cover the chip when buckets are few and long;
  // at least ~32 rows per split on average.
  const int64_t target_waves = 8192;
  if (r >= target_waves) return 1;
  int64_t s = ceil_div(target_waves, r);
  const int64_t by_rows = n / (r * 32);
  if (s > by_rows) s = by_rows;
  if (s > 64) s = 64;
  return s < 1 ? 1 : (int)s;
}

template <typename T, typename TO, int VW>
void launch_dense(const psk_mat &A, int64_t r, const uint32_t *perm,
                  const uint32_t *bptr, int splits, double scale, TO *out, hipStream_t st) {
  const int64_t waves = r * splits;
  const unsigned blocks = (unsigned)ceil_div(waves, 4);
  const int64_t span1 = 64 * VW;  // columns per lane group
  // one column group: six rows a batch (84 VGPRs with FP32 rows, against
  // 104 at eight) run as fast alone and leave more room beside a kernel of
  // another stream
  if (A.d <= span1)
    k_scatter_dense<T, TO, VW, 1, 6><<<blocks, 256, 0, st>>>(
        (const T *)A.values, A.ld, A.d, r, perm, bptr, splits, scale, out);
  else if (A.d <= 2 * span1)
    k_scatter_dense<T, TO, VW, 2, 4><<<blocks, 256, 0, st>>>(
        (const T *)A.values, A.ld, A.d, r, perm, bptr, splits, scale, out);
  else
    k_scatter_dense<T, TO, VW, 4, 4><<<blocks, 256, 0, st>>>(
        (const T *)A.values, A.ld, A.d, r, perm, bptr, splits, scale, out);
}

// VW adjacent columns per lane where the rows of A and of the output allow
// aligned vector accesses
template <typename T, typename TO>
void launch_dense_vw(const psk_mat &A, int64_t r, const uint32_t *perm,
                     const uint32_t *bptr, int splits, double scale, TO *out,
                     hipStream_t st) {
  const uintptr_t addr = (uintptr_t)A.values, oaddr = (uintptr_t)out;
  constexpr int es = (int)sizeof(T), os = (int)sizeof(TO);
  const bool v4 = es == 4 && (A.d % 4 == 0) && (A.ld % 4 == 0) && (addr % 16 == 0) &&
                  oaddr % (os == 4 ? 16 : 16) == 0;
  const bool v2 = (A.d % 2 == 0) && (A.ld % 2 == 0) && (addr % (2 * es) == 0) &&
                  oaddr % (2 * os) == 0;
  if constexpr (sizeof(T) == 4) {
    if (v4) return launch_dense<T, TO, 4>(A, r, perm, bptr, splits, scale, out, st);
  }
  if (v2) return launch_dense<T, TO, 2>(A, r, perm, bptr, splits, scale, out, st);
  launch_dense<T, TO, 1>(A, r, perm, bptr, splits, scale, out, st);
}

// LDS of the CSR scatter: FP64 accumulators of wpb wavefronts
constexpr size_t kCsrLdsMax = 163840;

}  // namespace

// ---------------------------------------------------------------------------
// host entry points
// ---------------------------------------------------------------------------
int cs_splits(int64_t n, int64_t r) { return choose_splits(n, r); }
int scan_plan(int64_t L, Arena &ws, uint32_t **sums) { return scan_plan_impl(L, ws, sums); }
void scan_run(uint32_t *data, int64_t L, uint32_t *sums, hipStream_t st) {
  scan_run_impl(data, L, sums, st);
}

int cs_hash_export(int64_t row0, int64_t count, uint32_t r, uint64_t seed,
                   int32_t *h, int8_t *sign, hipStream_t st) {
  if (count == 0) return 0;
  k_hash_export<<<(unsigned)ceil_div(count, 256), 256, 0, st>>>(row0, count, r,
                                                                 seed, h, sign);
  PSK_HIP_TRY(hipGetLastError());
  return 0;
}

namespace {

// One bucket: the pairs as they come.
template <class SRC>
__global__ __launch_bounds__(256) void k_write_pairs(SRC src, int64_t n,
                                                     const uint32_t *__restrict__ dn,
                                                     uint32_t *__restrict__ k,
                                                     uint32_t *__restrict__ v,
                                                     uint32_t *__restrict__ ptr) {
  n = keys_in_use(n, dn);
  const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (j == 0 && ptr) {
    ptr[0] = 0u;
    ptr[1] = (uint32_t)n;
  }
  if (j < n && k) src.get(j, k[j], v[j]);
}

// The sort of n pairs from src (dn: their count on the device, n at most)
// by keys below r.  The first pass reads src and writes (k0, v0); later ones
// go back and forth between (k0, v0) and (k1, v1), which are only needed then.
// A lean workspace keeps to 8-bit digits (a quarter of the counts), unless a
// single pass of the pairs is the smaller one: with `arrays`, where the caller
// takes (k1, v1) only for a second pass, 8 bytes a pair against the counts.
int sort_passes(uint32_t r, bool lean, int64_t n, bool arrays) {
  int bits = 0;
  while (bits < 32 && ((uint64_t)1 << bits) < (uint64_t)r) ++bits;
  const int most = lean ? 8 : kDigitBits;
  const int passes = bits > most ? (bits + most - 1) / most : 1;
  if (!lean || !arrays || passes == 1 || bits > kDigitBits) return passes;
  const int64_t more = ((int64_t)1 << bits) - ((int64_t)1 << (bits + 1) / 2);  // digits
  return more * ceil_div(n, (int64_t)kSortTile) * 4 <= 8 * n ? 1 : passes;
}

template <class SRC>
int sort_run(SRC src, int64_t n, uint32_t r, uint32_t *k0, uint32_t *v0, uint32_t *k1,
             uint32_t *v1, int passes, Arena &ws, hipStream_t st, uint32_t **skeys,
             uint32_t **svals, uint32_t *ptr, const uint32_t *dn) {
  int bits = 0;
  while (bits < 32 && ((uint64_t)1 << bits) < (uint64_t)r) ++bits;
  if (r == 1) {
    if (ws.dry()) return 0;
    if (!ws.ok()) return fail(PSK_ENOMEM, "workspace too small for a radix sort");
    k_write_pairs<<<(unsigned)(n > 0 ? ceil_div(n, (int64_t)256) : 1), 256, 0, st>>>(
        src, n, dn, k0, v0, ptr);
    PSK_HIP_TRY(hipGetLastError());
    *skeys = k0;
    *svals = v0;
    return 0;
  }
  const int nbits = (bits + passes - 1) / passes;  // equal digits: fewer counts to scan
  const int D = 1 << nbits;
  const int64_t ntiles = ceil_div(n, kSortTile);
  const int64_t L = (int64_t)D * ntiles;
  uint32_t *hist = ws.take<uint32_t>(L);
  uint32_t *sums = nullptr;
  scan_plan_impl(L, ws, &sums);
  if (ws.dry()) return 0;
  if (!ws.ok()) return fail(PSK_ENOMEM, "workspace too small for a radix sort");
  const size_t lds = (size_t)(kSortWaves + 2) * D * sizeof(uint32_t);
  auto pass = [&](auto from, int p, uint32_t *kout, uint32_t *vout) {
    const int shift = nbits * p;
    const unsigned g = (unsigned)ntiles;
    k_radix_hist<<<g, kSortThreads, 0, st>>>(from, n, dn, shift, nbits, hist);
    scan_run_impl(hist, L, sums, st, dn, D);
    k_radix_scatter<<<g, kSortThreads, lds, st>>>(from, n, dn, shift, nbits, hist, kout, vout);
  };
  if (n > 0) {
    pass(src, 0, k0, v0);
    for (int p = 1; p < passes; ++p) {
      pass(StoredPairs{k0, v0}, p, k1, v1);
      std::swap(k0, k1);
      std::swap(v0, v1);
    }
  }
  if (ptr && dn)
    k_bucket_ptr_search<<<(unsigned)ceil_div((int64_t)r + 1, 256), 256, 0, st>>>(k0, dn, r, ptr);
  else if (ptr)
    k_bucket_ptr<<<(unsigned)ceil_div(n + 1, 256), 256, 0, st>>>(k0, n, nullptr, r, ptr);
  PSK_HIP_TRY(hipGetLastError());
  *skeys = k0;
  *svals = v0;
  return 0;
}

}  // namespace

int sort_pairs(uint32_t *keys, uint32_t *vals, int64_t n, uint32_t r, Arena &ws,
               hipStream_t st, uint32_t **skeys, uint32_t **svals, uint32_t *ptr,
               const uint32_t *dn) {
  // one bucket: the pairs stay where they are
  uint32_t *k0 = r > 1 ? ws.take<uint32_t>(n) : nullptr;
  uint32_t *v0 = r > 1 ? ws.take<uint32_t>(n) : nullptr;
  const int rc = sort_run(StoredPairs{keys, vals}, n, r, k0, v0, keys, vals,
                          sort_passes(r, ws.lean, n, false), ws, st, skeys, svals, ptr, dn);
  if (r == 1 && !rc) {
    *skeys = keys;
    *svals = vals;
  }
  return rc;
}

int osnap_hash_export(int64_t row0, int64_t count, uint32_t s, uint32_t r, uint64_t seed,
                      int32_t *h, int8_t *sign, hipStream_t st) {
  const int64_t pairs = count * (int64_t)s;
  if (pairs == 0) return 0;
  k_hash_export_osnap<<<(unsigned)ceil_div(pairs, 256), 256, 0, st>>>(row0, pairs, s, r / s,
                                                                       seed, h, sign);
  PSK_HIP_TRY(hipGetLastError());
  return 0;
}

// Bins of the (row, non-zero) pairs: s per row (s = 1 for CountSketch,
// rb = r / s rows of S per block).  For CSR A only the rows holding an
// entry are listed first (their count stays on the device and bounds the
// sort), so a matrix with many empty rows sorts only the others.
static int bin_pairs(const psk_mat &A, uint32_t s, uint32_t r, uint64_t seed, Arena &ws,
                     hipStream_t st, uint32_t **perm, uint32_t **bptr) {
  const int64_t n = A.n;
  const int64_t pairs = n * (int64_t)s;
  const bool compact = A.format == PSK_CSR;
  const int passes = sort_passes(r, ws.lean, pairs, true);
  const bool two = passes > 1;
  uint32_t *k0 = ws.take<uint32_t>(pairs);
  uint32_t *v0 = ws.take<uint32_t>(pairs);
  uint32_t *k1 = two ? ws.take<uint32_t>(pairs) : nullptr;
  uint32_t *v1 = two ? ws.take<uint32_t>(pairs) : nullptr;
  uint32_t *bp = ws.take<uint32_t>((size_t)r + 1);
  // tiles of the row list: whole rounds of rows, few enough to be summed by all
  const int64_t rounds = ceil_div(ceil_div(n, (int64_t)kListRows), kPairTiles);
  const int64_t ltiles = ceil_div(n, rounds * kListRows);
  uint32_t *rows = nullptr, *cnt = nullptr, *lsum = nullptr;
  if (compact) {
    rows = ws.take<uint32_t>((size_t)n);
    cnt = ws.take<uint32_t>(2);
    lsum = ws.take<uint32_t>((size_t)ltiles);
  }
  if (!ws.dry() && !ws.ok()) return fail(PSK_ENOMEM, "workspace too small for the binning");
  KTimer timer("cs_bin", st, !ws.dry());
  if (!ws.dry() && compact) {
    const unsigned g = (unsigned)ltiles;
    k_row_list<false><<<g, 256, 0, st>>>(A.indptr, n, (int)rounds, s, lsum, rows, cnt);
    k_row_list<true><<<g, 256, 0, st>>>(A.indptr, n, (int)rounds, s, lsum, rows, cnt);
  }
  uint32_t *sk = nullptr;
  int rc;
  // for CSR A the pairs of the listed rows (cnt[1]) bound the sort
  if (compact)
    rc = sort_run(HashedList{rows, s, r / s, seed}, pairs, r, k0, v0, k1, v1, passes, ws, st,
                  &sk, perm, bp, cnt + 1);
  else if (s == 1)
    rc = sort_run(HashedRows{r, seed}, pairs, r, k0, v0, k1, v1, passes, ws, st, &sk, perm, bp,
                  nullptr);
  else
    rc = sort_run(HashedOsnap{s, r / s, seed}, pairs, r, k0, v0, k1, v1, passes, ws, st, &sk, perm,
                  bp, nullptr);
  if (rc) return rc;
  *bptr = bp;
  return 0;
}

int cs_bin(const psk_mat &A, uint32_t r, uint64_t seed, Arena &ws, hipStream_t st,
           uint32_t **perm, uint32_t **bptr) {
  return bin_pairs(A, 1u, r, seed, ws, st, perm, bptr);
}

int osnap_bin(const psk_mat &A, uint32_t s, uint32_t r, uint64_t seed, Arena &ws,
              hipStream_t st, uint32_t **perm, uint32_t **bptr) {
  return bin_pairs(A, s, r, seed, ws, st, perm, bptr);
}

int cs_apply(const psk_mat &A, uint32_t r, const uint32_t *perm,
             const uint32_t *bptr, void *SA, Arena &ws, hipStream_t st, bool out_f64,
             double scale, int64_t entries) {
  const int splits = choose_splits(entries > 0 ? entries : A.n, r);
  const bool o64 = out_f64 || A.dtype == PSK_F64;
  void *part = nullptr;
  if (splits > 1) part = ws.take<double>((size_t)splits * r * A.d);
  const int64_t dpad = (A.d + 3) & ~(int64_t)3;
  if (A.format == PSK_CSR && (size_t)dpad * 8 > kCsrLdsMax)
    return fail(PSK_EUNSUPPORTED, "CSR S*A supports d <= 20480");
  if (ws.dry()) return 0;
  if (!ws.ok()) return fail(PSK_ENOMEM, "workspace too small for S*A");
  KTimer timer("cs_scatter", st);
  if (A.format == PSK_DENSE) {
    // K-split partials are written unscaled; the combine applies the scale
    if (splits > 1) {
      if (A.dtype == PSK_F64)
        launch_dense_vw<double, double>(A, r, perm, bptr, splits, 1.0, (double *)part, st);
      else
        launch_dense_vw<float, double>(A, r, perm, bptr, splits, 1.0, (double *)part, st);
    } else if (A.dtype == PSK_F64) {
      launch_dense_vw<double, double>(A, r, perm, bptr, 1, scale, (double *)SA, st);
    } else if (o64) {
      launch_dense_vw<float, double>(A, r, perm, bptr, 1, scale, (double *)SA, st);
    } else {
      launch_dense_vw<float, float>(A, r, perm, bptr, 1, scale, (float *)SA, st);
    }
  } else {
    int wpb = 4;
    while (wpb > 1 && (size_t)wpb * dpad * 8 > 65536) --wpb;
    const size_t lds = (size_t)wpb * dpad * 8;
    const int64_t waves = (int64_t)r * splits;
    const unsigned blocks = (unsigned)ceil_div(waves, wpb);
#define PSK_SCSR(T, TO, OUT, SC)                                                           \
  do {                                                                                     \
    if (lds > 65536)                                                                       \
      PSK_HIP_TRY(hipFuncSetAttribute((const void *)k_scatter_csr<T, TO>,                  \
                                      hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds)); \
    k_scatter_csr<T, TO><<<blocks, 64 * wpb, lds, st>>>((const T *)A.values, A.indptr,     \
                                                        A.indices, A.d, dpad, r, perm, bptr, \
                                                        splits, (SC), (TO *)(OUT));        \
  } while (0)
    if (splits > 1) {
      if (A.dtype == PSK_F64) PSK_SCSR(double, double, part, 1.0);
      else PSK_SCSR(float, double, part, 1.0);
    } else if (A.dtype == PSK_F64) {
      PSK_SCSR(double, double, SA, scale);
    } else if (o64) {
      PSK_SCSR(float, double, SA, scale);
    } else {
      PSK_SCSR(float, float, SA, scale);
    }
#undef PSK_SCSR
  }
  if (splits > 1) {
    const int64_t rd = (int64_t)r * A.d;
    if (o64)
      k_combine_splits<double><<<(unsigned)ceil_div(rd, 256), 256, 0, st>>>(
          (const double *)part, rd, splits, scale, (double *)SA);
    else
      k_combine_splits<float><<<(unsigned)ceil_div(rd, 256), 256, 0, st>>>(
          (const double *)part, rd, splits, scale, (float *)SA);
  }
  PSK_HIP_TRY(hipGetLastError());
  return 0;
}

}  // namespace psk
