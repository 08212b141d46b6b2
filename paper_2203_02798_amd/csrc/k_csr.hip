// Gram matrix and squared row norms of a CSR matrix on gfx950, FP64.
//
// Paper mapping (arXiv 2203.02798):
// * Gram: Algorithm gram_serial's outer-product loop (B[J_k, J_j] +=
//   V_k V_j over pairs of a row's entries), parallelised by output rows as
//   Algorithm gram_parallel_memory_effcient does (each worker owns output
//   rows, so no partial Grams and no reduction), but where that algorithm
//   scans every row of A and filters its entries, here the entries are first
//   sorted by column (a stable radix sort: the column index of A), so the
//   wavefront owning output row j visits exactly the rows with an entry in
//   column j: nnz_2(A) work in total.  Only k >= j is accumulated and the
//   other triangle is mirrored, so C is exactly symmetric.
// * Row norms: Algorithm squared_row_norms: Bt = B B^T once, then per row
//   sum_{k,j} V_k V_j Bt[J_j, J_k].  Rows of up to 4 entries (6 to 9 where a
//   wavefront has many) take one lane each, up to 16 a quarter of a wavefront, longer ones
//   a wavefront (lanes over k) from a list.
//   That costs a row nnz^2 scattered reads of Bt; a row with more than
//   max(32, k/8) entries costs less as the product itself, ||V B[J, :]||^2
//   (nnz contiguous rows of B, k values each): such rows are listed too and
//   taken by a workgroup each (k_rownorm_csr_listed).
#include "internal.hpp"

namespace psk {
namespace {

// rowidx[p] = row of stored entry p
__global__ __launch_bounds__(256) void k_row_of_entry(const int64_t *__restrict__ indptr,
                                                      int64_t n, uint32_t *__restrict__ rowidx) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  for (int64_t p = indptr[i]; p < indptr[i + 1]; ++p) rowidx[p] = (uint32_t)i;
}

// (column, position) pairs of the stored entries, to be sorted by column
__global__ __launch_bounds__(256) void k_col_keys(const int32_t *__restrict__ indices,
                                                  int64_t nnz, uint32_t *__restrict__ keys,
                                                  uint32_t *__restrict__ vals) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= nnz) return;
  keys[p] = (uint32_t)indices[p];
  vals[p] = (uint32_t)p;
}

// One wavefront per output row j: for every entry A[i, j] of column j (rows
// in increasing order), add A[i, j] * A[i, k] over the entries of row i with
// k >= j into a private LDS row; then write C[j, k] and its mirror C[k, j].
template <typename T, typename TO>
__global__ __launch_bounds__(256) void k_gram_csc(
    const T *__restrict__ vals, const int64_t *__restrict__ indptr,
    const int32_t *__restrict__ indices, const uint32_t *__restrict__ rowidx,
    const uint32_t *__restrict__ cperm, const uint32_t *__restrict__ cptr, int64_t d,
    int64_t dpad, double alpha, double beta, TO *__restrict__ C) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  double *acc = reinterpret_cast<double *>(smem_raw) + (threadIdx.x >> 6) * dpad;
  const int64_t j = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  if (j >= d) return;
  const int lane = threadIdx.x & 63;
  for (int64_t c = j + lane; c < d; c += 64) acc[c] = 0.0;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  const uint32_t e1 = cptr[j + 1];
  for (uint32_t e0 = cptr[j]; e0 < e1; e0 += 64) {
    const uint32_t e = e0 + lane;
    if (e < e1) {
      const uint32_t p = cperm[e];
      const double v = (double)vals[p];
      const uint32_t i = rowidx[p];
      for (int64_t h = indptr[i]; h < indptr[i + 1]; ++h) {
        const int32_t c = indices[h];
        if (c >= j) atomicAdd(&acc[c], v * (double)vals[h]);
      }
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  for (int64_t k = j + lane; k < d; k += 64) {
    const double g = alpha * acc[k];
    const int64_t up = j * d + k, lo = k * d + j;
    C[up] = (TO)(beta != 0.0 ? g + beta * (double)C[up] : g);
    if (k > j) C[lo] = (TO)(beta != 0.0 ? g + beta * (double)C[lo] : g);
  }
}

// The rows of up to kRowGroup entries; the others are only listed: up to tl
// entries from the front of the list, longer ones from its back (count[0] and
// count[1] of them; n places hold both).  The order of the lists does not
// matter, each row's value is computed alone.
// What bounds it is a chain: one lane's loads of Bt for a row of 30 entries
// are 900 dependent steps, and a few such rows held the launch (1e7 rows, 41,000
// of them holding entries, Zipf lengths: 549 us; row pointers and x alone
// take 33).  With the longer rows' lanes over k, their loads side by side, it
// takes 89 and the listed rows of up to 125 entries 87.
// Four rows of 5 to 16 entries side by side take 1.4 us, a wavefront full of
// them 22; rows of up to 9 entries one lane each take half a us an entry of
// the longest, whatever their number, so from 2.5 rows an entry on they do
// (1e6 rows of 5 entries, d = 20: 196 us in fours, 61 by lanes).  Beyond 262,144
// rows it is the scattered loads of Bt that count and not the chain: then up
// to 8 entries for d up to 256 and up to 6 for more (1e6 rows of 8, lanes /
// fours: d = 140 156 / 200 us, d = 500 255 / 211).
constexpr int kRowLane = 4, kRowGroup = 16, kRowMany = 9;

int row_many(int64_t n, int64_t d) { return n <= 262144 ? kRowMany : d <= 256 ? 8 : 6; }

template <typename T>
__global__ __launch_bounds__(256) void k_rownorm_csr(
    const T *__restrict__ vals, const int64_t *__restrict__ indptr,
    const int32_t *__restrict__ indices, int64_t n, int64_t d,
    const double *__restrict__ Bt, double alpha, double beta, double *__restrict__ x,
    int64_t tl, int most, uint32_t *__restrict__ list, uint32_t *__restrict__ count) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int lane = threadIdx.x & 63;
  const bool have = i < n;
  int64_t p0 = 0, p1 = 0;
  if (have) {
    p0 = indptr[i];
    p1 = indptr[i + 1];
  }
  const int64_t len = p1 - p0;
  auto finish = [&](int64_t row, double v) {
    x[row] = beta != 0.0 ? alpha * v + beta * x[row] : alpha * v;
  };
  if (have && len <= kRowLane) {
    double v[kRowLane];
    int64_t c[kRowLane];
#pragma unroll
    for (int k = 0; k < kRowLane; ++k) {
      v[k] = k < len ? (double)vals[p0 + k] : 0.0;
      c[k] = k < len ? indices[p0 + k] : 0;
    }
    double acc = 0.0;
#pragma unroll
    for (int k = 0; k < kRowLane; ++k) {
      if (k >= len) break;
      double t = 0.0;
#pragma unroll
      for (int j = 0; j < kRowLane; ++j)
        if (j < len) t += v[j] * Bt[c[j] * d + c[k]];
      acc += v[k] * t;
    }
    finish(i, acc);
  }
  // rows for the lists: one counter update a wavefront and list
  const uint64_t lt = lane == 0 ? 0ull : ((~0ull) >> (64 - lane));
#pragma unroll
  for (int which = 0; which < 2; ++which) {
    const bool mine = which ? len > tl && len > kRowGroup : len > kRowGroup && len <= tl;
    const uint64_t m = __ballot(mine);
    if (!m) continue;
    uint32_t at = 0;
    if (lane == 0) at = atomicAdd(&count[which], (uint32_t)__popcll(m));
    at = __shfl(at, 0, 64) + (uint32_t)__popcll(m & lt);
    if (mine) list[which ? (uint32_t)n - 1u - at : at] = (uint32_t)i;
  }
  // many rows of kRowLane + 1 .. most entries: a lane each
  const bool some = len > kRowLane && len <= most;
  int longest = most;
  while (longest > kRowLane && !__ballot(len == longest)) --longest;
  const bool many = longest > kRowLane && 2 * __popcll(__ballot(some)) >= 5 * longest;
  if (many && some) {
    double v[kRowMany], acc = 0.0;
    int64_t c[kRowMany];
#pragma unroll
    for (int j = 0; j < kRowMany; ++j) {
      v[j] = j < len ? (double)vals[p0 + j] : 0.0;
      c[j] = j < len ? indices[p0 + j] : 0;
    }
    for (int k = 0; k < len; ++k) {
      const int64_t ck = indices[p0 + k];
      double t = 0.0;
#pragma unroll
      for (int j = 0; j < kRowMany; ++j)
        if (j < len) t += v[j] * Bt[c[j] * d + ck];
      acc += (double)vals[p0 + k] * t;
    }
    finish(i, acc);
  }
  // the others of kRowLane + 1 .. kRowGroup entries, four at a time
  uint64_t pending = __ballot(len > (many ? most : kRowLane) && len <= kRowGroup);
  const int g = lane >> 4, l = lane & 15;
  while (pending) {
    int src = -1;  // this group's row: the g-th pending one
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (!pending) break;
      const int b = __ffsll((unsigned long long)pending) - 1;
      pending &= pending - 1;
      if (q == g) src = b;
    }
    // (all lanes shuffle: the row's own lane may be in a group without one)
    const int64_t q0 = __shfl(p0, src < 0 ? 0 : src, 64);
    const int64_t row = __shfl(i, src < 0 ? 0 : src, 64);
    const int len0 = (int)__shfl(len, src < 0 ? 0 : src, 64);
    const int L = src < 0 ? 0 : len0;
    const bool in = l < L;
    const double vk = in ? (double)vals[q0 + l] : 0.0;
    const int ck = in ? indices[q0 + l] : 0;
    double t = 0.0;
#pragma unroll
    for (int j = 0; j < kRowGroup; ++j) {
      const double vj = __shfl(vk, (lane & 48) + j, 64);
      const int cj = __shfl(ck, (lane & 48) + j, 64);
      const double b = Bt[(int64_t)cj * d + ck];  // (0, 0) past the row's end
      if (in && j < L) t += vj * b;
    }
    double part = vk * t;
#pragma unroll
    for (int off = 8; off > 0; off >>= 1) part += __shfl_xor(part, off, 64);
    if (l == 0 && src >= 0) finish(row, part);
  }
}

// The counts of the two lists of rows cleared and (first not NULL) first[c] =
// the first column of row c of B (d x k) holding a nonzero, k if none: a
// wavefront per row.
__global__ __launch_bounds__(256) void k_row_first(const double *__restrict__ B, int64_t d,
                                                   int64_t k, uint32_t *__restrict__ count,
                                                   uint32_t *__restrict__ first) {
  if (blockIdx.x == 0 && threadIdx.x < 2) count[threadIdx.x] = 0u;
  if (!first) return;
  const int64_t c = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (c >= d) return;
  for (int64_t j0 = 0; j0 < k; j0 += 64) {
    const bool nz = j0 + lane < k && B[c * k + j0 + lane] != 0.0;  // NaN is a nonzero
    const uint64_t m = __ballot(nz);
    if (m) {
      if (lane == 0) first[c] = (uint32_t)(j0 + __ffsll((unsigned long long)m) - 1);
      return;
    }
  }
  if (lane == 0) first[c] = (uint32_t)k;
}

// The listed rows.  Those at the front of the list: a wavefront each, lane
// over k, the entries j eight at a time with their loads together.  Those at
// its back as the product itself: a workgroup each (grid-stride over the
// list), thread t holds y_j = sum_p V_p B[J_p, j] for its columns j = t + TH q,
// q < Q (and TH Q further on, when k is wider), the entries taken in row order, kRnU at
// a time with their rows of B loaded together; then the squares summed in a
// fixed order (thread, wavefront, workgroup).
// The product is bound by the rows of B coming from the caches, in a chain of
// batches as long as the longest row.  Its entries are staged in LDS TH at a
// time, so that a batch waits for B alone, and a triangular B's leading zeros
// (up to first[c]) are not read, their lanes taking the row's last element
// instead; an entry that is not finite takes the whole row, zeros too, and a
// place past the row's end takes none of B (its row 0 may not be finite).  1900
// rows of 350 entries, k = 1000: 592 us with 8 entries and 4 columns a thread,
// 486 with staging and without the zeros, 446 with 16 entries and 2 columns
// of 512 threads (1024 threads: 456; a launch per 256 columns, which an XCD's
// L2 holds: 1200).  20,000 rows of 60 entries, k = 100: 782, now 196.
constexpr int kRnU = 16;  // entries whose B rows are in flight together
template <typename T, int TH, int Q>
__global__ __launch_bounds__(TH) void k_rownorm_csr_listed(
    const T *__restrict__ vals, const int64_t *__restrict__ indptr,
    const int32_t *__restrict__ indices, const uint32_t *__restrict__ list, int64_t n,
    const uint32_t *__restrict__ count, const uint32_t *__restrict__ first, int64_t d,
    const double *__restrict__ Bt, const double *__restrict__ B, int64_t k, double alpha,
    double beta, double *__restrict__ x) {
  __shared__ double red[TH / 64];
  __shared__ double ev[TH];
  __shared__ uint32_t ec[TH], ef[TH];
  const int tid = threadIdx.x, lane = tid & 63;
  auto finish = [&](int64_t row, double v) {
    x[row] = beta != 0.0 ? alpha * v + beta * x[row] : alpha * v;
  };
  const uint32_t nmid = count[0], nlong = count[1];
  for (uint32_t e = blockIdx.x * (TH / 64) + (tid >> 6); e < nmid; e += gridDim.x * (TH / 64)) {
    const uint32_t row = (uint32_t)__builtin_amdgcn_readfirstlane((int)list[e]);
    const int64_t q0 = indptr[row], q1 = indptr[row + 1];
    double part = 0.0;
    for (int64_t k0 = q0; k0 < q1; k0 += 64) {
      const int64_t p = k0 + lane;
      const double vk = p < q1 ? (double)vals[p] : 0.0;
      const int64_t ck = p < q1 ? indices[p] : 0;
      double t = 0.0;
      for (int64_t j = q0; j < q1; j += 8) {
        double v[8], b[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int64_t ju = j + u < q1 ? j + u : q0;
          v[u] = (double)vals[ju];
          b[u] = Bt[(int64_t)indices[ju] * d + ck];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
          if (j + u < q1) t += v[u] * b[u];
      }
      part += p < q1 ? vk * t : 0.0;
    }
    part = wave_sum(part);
    if (lane == 0) finish(row, part);
  }
  for (uint32_t l = blockIdx.x; l < nlong; l += gridDim.x) {
    const int64_t i = (int64_t)list[(uint32_t)n - 1u - l];
    const int64_t p0 = indptr[i], p1 = indptr[i + 1];
    double s = 0.0;
    for (int64_t j0 = tid; j0 - tid < k; j0 += TH * Q) {
      double y[Q];
#pragma unroll
      for (int q = 0; q < Q; ++q) y[q] = 0.0;
      for (int64_t s0 = p0; s0 < p1; s0 += TH) {
        const int64_t p = s0 + tid;
        const double ve = p < p1 ? (double)vals[p] : 0.0;
        const uint32_t c = p < p1 ? (uint32_t)indices[p] : 0u;
        const uint32_t f = first ? first[c] : 0u;
        __syncthreads();  // the entries before have been used
        ev[tid] = ve;
        ec[tid] = c;
        ef[tid] = p >= p1 ? UINT32_MAX : fabs(ve) <= 1.7976931348623157e308 ? f : 0u;
        __syncthreads();
        const int m = (int)(p1 - s0 < TH ? p1 - s0 : TH);
        for (int e0 = 0; e0 < m; e0 += kRnU) {  // past m: 0 times 0
          double b[kRnU][Q];
#pragma unroll
          for (int u = 0; u < kRnU; ++u) {
            const double *br = B + (int64_t)ec[e0 + u] * k;
            const uint32_t fu = ef[e0 + u];
#pragma unroll
            for (int q = 0; q < Q; ++q) {
              const int64_t j = j0 + TH * q;
              const bool in = j < k && (uint32_t)j >= fu;
              const double e = br[in ? j : k - 1];
              b[u][q] = in ? e : 0.0;
            }
          }
#pragma unroll
          for (int u = 0; u < kRnU; ++u)
#pragma unroll
            for (int q = 0; q < Q; ++q) y[q] = fma(ev[e0 + u], b[u][q], y[q]);
        }
      }
#pragma unroll
      for (int q = 0; q < Q; ++q)
        if (j0 + TH * q < k) s = fma(y[q], y[q], s);
    }
    s = wave_sum(s);
    if (lane == 0) red[tid >> 6] = s;
    __syncthreads();
    if (tid == 0) {
      double t = red[0];
#pragma unroll
      for (int w = 1; w < TH / 64; ++w) t += red[w];
      finish(i, t);
    }
    __syncthreads();  // red is reused by the next row
  }
}

}  // namespace

int gram_csr(double alpha, const psk_mat &A, double beta, void *C, Arena &ws,
             hipStream_t st, bool out_f64) {
  const int64_t d = A.d, n = A.n, nnz = A.nnz;
  if (d > 8192) return fail(PSK_EUNSUPPORTED, "CSR gram supports d <= 8192");
  if (nnz >= ((int64_t)1 << 32)) return fail(PSK_EUNSUPPORTED, "CSR gram needs nnz < 2^32");
  const int64_t cnt = nnz > 0 ? nnz : 1;
  uint32_t *keys = ws.take<uint32_t>(cnt);
  uint32_t *vals = ws.take<uint32_t>(cnt);
  uint32_t *rowidx = ws.take<uint32_t>(cnt);
  uint32_t *cptr = ws.take<uint32_t>((size_t)d + 1);
  if (!ws.dry()) {
    k_col_keys<<<(unsigned)ceil_div(cnt, 256), 256, 0, st>>>(A.indices, nnz, keys, vals);
    k_row_of_entry<<<(unsigned)ceil_div(n, 256), 256, 0, st>>>(A.indptr, n, rowidx);
  }
  uint32_t *skeys = nullptr, *cperm = nullptr;
  int rc = sort_pairs(keys, vals, nnz, (uint32_t)d, ws, st, &skeys, &cperm, cptr);
  if (rc) return rc;
  if (ws.dry()) return 0;
  if (!ws.ok()) return fail(PSK_ENOMEM, "workspace too small for CSR gram");
  const int64_t dpad = (d + 1) & ~(int64_t)1;
  int wpb = 4;
  while (wpb > 1 && (size_t)wpb * dpad * sizeof(double) > 65536) --wpb;
  const size_t lds = (size_t)wpb * dpad * sizeof(double);
  const unsigned blocks = (unsigned)ceil_div(d, wpb);
  KTimer timer("gram", st);
  if (A.dtype == PSK_F64)
    k_gram_csc<double, double><<<blocks, 64 * wpb, lds, st>>>(
        (const double *)A.values, A.indptr, A.indices, rowidx, cperm, cptr, d, dpad, alpha,
        beta, (double *)C);
  else if (out_f64)
    k_gram_csc<float, double><<<blocks, 64 * wpb, lds, st>>>(
        (const float *)A.values, A.indptr, A.indices, rowidx, cperm, cptr, d, dpad, alpha,
        beta, (double *)C);
  else
    k_gram_csc<float, float><<<blocks, 64 * wpb, lds, st>>>(
        (const float *)A.values, A.indptr, A.indices, rowidx, cperm, cptr, d, dpad, alpha,
        beta, (float *)C);
  PSK_HIP_TRY(hipGetLastError());
  return 0;
}

int rownorms_csr(double alpha, const psk_mat &A, const double *B, int64_t k,
                 double beta, double *x, Arena &ws, hipStream_t st) {
  const int64_t d = A.d;
  if (d > 8192) return fail(PSK_EUNSUPPORTED, "CSR row norms support d <= 8192");
  double *Bt = ws.take<double>((size_t)d * d);
  // rows for the product form: more than max(32, k/8) entries (k <= 2048)
  const int64_t tl = k <= 2048 ? (k / 8 > 32 ? k / 8 : 32) : INT64_MAX;
  uint32_t *list = ws.take<uint32_t>((size_t)A.n);
  uint32_t *count = ws.take<uint32_t>(2);
  uint32_t *first = !ws.lean && tl != INT64_MAX ? ws.take<uint32_t>((size_t)d) : nullptr;
  // B * B^T (d x d) with the FP64 GEMM
  int rc = dgemm(false, true, d, d, k, 1.0, B, k, B, k, 0.0, Bt, d, ws, st);
  if (rc) return rc;
  if (ws.dry()) return 0;
  if (!ws.ok()) return fail(PSK_ENOMEM, "workspace too small for CSR row norms");
  const unsigned blocks = (unsigned)ceil_div(A.n, 256);
  KTimer timer("rownorm", st);
  k_row_first<<<first ? (unsigned)ceil_div(d, (int64_t)4) : 1u, 256, 0, st>>>(B, d, k, count,
                                                                             first);
  // a fixed grid walks the listed rows (their counts stay on the device)
  auto run = [&](auto t) {
    typedef decltype(t) T;
    const T *vals = (const T *)A.values;
    k_rownorm_csr<T><<<blocks, 256, 0, st>>>(vals, A.indptr, A.indices, A.n, d, Bt, alpha, beta,
                                             x, tl, row_many(A.n, d), list, count);
#define PSK_RNL(TH, Q)                                                                       \
  k_rownorm_csr_listed<T, TH, Q><<<2048, TH, 0, st>>>(vals, A.indptr, A.indices, list, A.n, \
                                                      count, first, d, Bt, B, k, alpha, beta, x)
    if (k <= 256) PSK_RNL(256, 1);
    else if (k <= 512) PSK_RNL(512, 1);
    else PSK_RNL(512, 2);
#undef PSK_RNL
  };
  if (A.dtype == PSK_F64) run(double{});
  else run(float{});
  PSK_HIP_TRY(hipGetLastError());
  return 0;
}

}  // namespace psk
