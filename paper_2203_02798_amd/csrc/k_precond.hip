// The sketch's preconditioner sharpened by A's own Gram matrix, for LSQR
// (FP64, gfx950).
//
// Paper mapping (arXiv 2203.02798): Algorithm least_squares_precondition
// solves min ||A N y - b|| with N = R^{-1} of the sketch.  A N then has
// singular values in about [1 / (1 + e), 1 / (1 - e)], e = sqrt(d / m), and
// LSQR reads A ln(1 / tol) / ln(1 / e) times: 31 for m = 8 d at 1e-14.  One
// more pass over A gives G = A^T A on the matrix cores, and with
//   W = N^T G N = S^T S  (Cholesky),  P = N S^{-1},
// A P has orthonormal columns up to the rounding of G, so LSQR on A P stops
// after two or three passes.  Forming W from G squares cond(A) where forming
// A N would not, but costs half of A N's own products and no n x d scratch.
//
// The rounding is taken as |dG_kl| ~ c u g_k g_l with g_k = ||A e_k|| and c = 16,
// which makes the error of P^T G P about E = c u sum_j t_j^2, t_j =
// sum_k |P_kj| g_k, in Frobenius norm, whatever the scaling of A's columns.
// That is an estimate and no bound: a sum's worst rounding grows with its
// length (rows of a slab, entries of a column of a CSR A) and its typical one
// with the root of it.  What it decides is only how many passes LSQR takes; its
// stopping rule and the refinement do not rest on it.  k_guard sums t_j^2.
// It is asked twice: before G is formed, with N in P's place and g from R (or,
// for a caller's N, a lower bound of it from N's diagonal and, where that leaves
// doubt, some of A's rows), where E above kPrecondMax leaves the sketch's N as
// it is (cond(A) beyond about 7e6 / sqrt(d)); and afterwards with P and G's
// diagonal, on the device: k_precond_pick puts N back into P when E is too large
// or a pivot failed, so such a P never reaches LSQR.
#include <math.h>

#include <cmath>

#include "internal.hpp"

namespace psk {
namespace {

constexpr double kGuardC = 16.0 * 1.1102230246251565e-16;  // c u
constexpr int kGuardCols = 64;   // columns of a k_guard workgroup
constexpr int kMaxGuard = 1024 / kGuardCols;
static_assert(kMaxGuard == kPrecondGuards, "a part for every workgroup of k_guard");

// A workgroup takes 64 columns j, a lane each; its 16 wavefronts take every
// 16th row k <= j, eight rows' loads in flight (one at a time, by four
// wavefronts, d = 500 took 77 us).  term(k, j) summed over k, the wavefronts'
// sums then in order, valid in wavefront 0.
constexpr int kGuardWaves = 16;
constexpr int kGuardBatch = 8;

template <class Load, class Use>
__device__ __forceinline__ double column_sum(int64_t d, Load load, Use use) {
  __shared__ double red[kGuardWaves][kGuardCols];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t j = (int64_t)blockIdx.x * kGuardCols + lane;
  const int64_t jend = (int64_t)(blockIdx.x + 1) * kGuardCols < d
                           ? (int64_t)(blockIdx.x + 1) * kGuardCols : d;  // rows of the block
  double s = 0.0;
  for (int64_t k0 = wave; k0 < jend; k0 += kGuardWaves * kGuardBatch) {
    double m[kGuardBatch], g[kGuardBatch];
#pragma unroll
    for (int q = 0; q < kGuardBatch; ++q) {
      const int64_t k = k0 + kGuardWaves * q;
      load(k < jend ? k : jend - 1, j < d ? j : d - 1, m[q], g[q]);  // clamped; masked below
    }
#pragma unroll
    for (int q = 0; q < kGuardBatch; ++q)
      if (k0 + kGuardWaves * q <= j && j < d) s = use(s, m[q], g[q]);
  }
  red[wave][lane] = s;
  __syncthreads();
  double t = red[0][lane];
#pragma unroll
  for (int q = 1; q < kGuardWaves; ++q) t += red[q][lane];
  return t;
}

// g[k] = ||R e_k||, R upper triangular
__global__ __launch_bounds__(64 * kGuardWaves) void k_col_norm_upper(
    const double *__restrict__ R, int64_t d, double *__restrict__ g) {
  const double s = column_sum(
      d, [&](int64_t k, int64_t j, double &m, double &) { m = R[k * d + j]; },
      [](double s2, double m, double) { return fma(m, m, s2); });
  const int64_t j = (int64_t)blockIdx.x * kGuardCols + threadIdx.x;
  if (threadIdx.x < kGuardCols && j < d) g[j] = sqrt(s);
}

// g[k], three quarters of about ||A e_k|| of a dense A from 256 of its rows, and
// not below 1 / |N_kk| = |R_kk|: four groups of 64 rows, one row in every
// stretch of n / 256, each group's sum of squares scaled to n rows, the least of the
// four (a few heavy rows must not look like all of them).  Three quarters: P's
// bound is about 0.75 of N's, and on the line a Gram matrix formed for nothing
// costs a tenth of the solve, one not formed three quarters.
constexpr int kNormRows = 256;

template <typename T>
__global__ __launch_bounds__(64 * kGuardWaves) void k_col_norm_sample(
    const T *__restrict__ A, int64_t ld, int64_t n, int64_t d, const double *__restrict__ N,
    double *__restrict__ g) {
  __shared__ double red[kGuardWaves][kGuardCols];
  constexpr int kEach = kNormRows / kGuardWaves;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t j = (int64_t)blockIdx.x * kGuardCols + lane;
  T x[kEach];
#pragma unroll
  for (int q = 0; q < kEach; ++q)  // rows of one wavefront are spread over all of A
    x[q] = A[(n * (q * kGuardWaves + wave) / kNormRows) * ld + (j < d ? j : d - 1)];
  double s = 0.0;
#pragma unroll
  for (int q = 0; q < kEach; ++q) s = fma((double)x[q], (double)x[q], s);
  red[wave][lane] = s;
  __syncthreads();
  if (wave || j >= d) return;
  double least = INFINITY;
#pragma unroll
  for (int q = 0; q < 4; ++q)
    least = fmin(least, (red[q][lane] + red[q + 4][lane]) + (red[q + 8][lane] + red[q + 12][lane]));
  g[j] = fmax(0.75 * sqrt(least * (double)n * (4.0 / kNormRows)), 1.0 / fabs(N[j * d + j]));
}

// part[b] = sum over the workgroup's columns j of (sum_{k <= j} |M_kj| g_k)^2,
// g_k = g[k] (mode 0), 1 / |g[k d + k]| (mode 1) or sqrt(g[k d + k]) (mode 2)
__global__ __launch_bounds__(64 * kGuardWaves) void k_guard(const double *__restrict__ M,
                                                            int64_t d,
                                                            const double *__restrict__ g,
                                                            int mode,
                                                            double *__restrict__ part) {
  const double t = column_sum(
      d,
      [&](int64_t k, int64_t j, double &m, double &gk) {
        m = M[k * d + j];
        gk = mode == 0 ? g[k] : g[k * d + k];
      },
      [&](double s, double m, double gk) {
        return fma(fabs(m), mode == 0 ? gk : mode == 1 ? 1.0 / fabs(gk) : sqrt(gk), s);
      });
  if (threadIdx.x < kGuardCols) {
    const int64_t j = (int64_t)blockIdx.x * kGuardCols + threadIdx.x;
    const double s = wave_sum(j < d ? t * t : 0.0);
    if (threadIdx.x == 0) part[blockIdx.x] = s;
  }
}

// U = the upper triangle of X, zero below (a caller's R^{-1} is read in its
// upper triangle only)
__global__ __launch_bounds__(256) void k_upper(const double *__restrict__ X, int64_t d,
                                               double *__restrict__ U) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= d * d) return;
  U[e] = e % d >= e / d ? X[e] : 0.0;
}

// P = N where the guard's sum (nb partials in order) or a pivot says so
__global__ __launch_bounds__(256) void k_precond_pick(const double *__restrict__ N, int64_t d,
                                                      const double *__restrict__ part, int nb,
                                                      const int *__restrict__ flag,
                                                      double *__restrict__ P) {
  double s = 0.0;
  for (int b = 0; b < nb; ++b) s += part[b];
  if (*flag == 0 && kGuardC * s <= kPrecondMax) return;  // NaN: not taken
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e < d * d) P[e] = N[e];
}

// What the times of a CSR LSQR pass and Gram matrix depend on, from workgroup b
// in part[b + kPrecondRowParts q]: sums of squared (q 0) and cubed (q 1) row
// lengths, what the pass's longer rows take (q 2, us), and the largest share of one
// column in up to kSample of the entries (q 3), less two standard deviations
// of a count (even columns are not to look like fewer).  Every workgroup's
// sample is spread over all the rows, an entry at a scattered place of every
// stretch of `step` (a fixed place could meet the same column of every row).
constexpr int kSample = 1024;  // one a thread: 64 x 1024 in all (4096 took 8 us more at 1e6 rows)
// us of a pass: a row past 16 entries takes a wavefront of its own (4.8 us, 4096
// wavefronts side by side), an entry past the fourth of a shorter one is not
// held in registers (20 us a million); both fitted to whole passes of 5e3 to
// 2e6 rows
constexpr double kLongRowUs = 4.8 / 4096.0, kDeepEntryUs = 20e-6;

__global__ __launch_bounds__(1024) void k_row_stats(const int64_t *__restrict__ indptr,
                                                    const int32_t *__restrict__ indices,
                                                    int64_t n, int64_t nnz, int d,
                                                    double *__restrict__ part) {
  __shared__ int hist[1024];
  __shared__ double red[4][16];
  const int tid = threadIdx.x;
  hist[tid] = 0;
  constexpr int64_t kAll = (int64_t)kSample * kPrecondRowParts;
  const int64_t step = nnz > kAll ? nnz / kAll : 1;
  int64_t taken = (nnz - blockIdx.x + kPrecondRowParts - 1) / kPrecondRowParts;
  taken = taken < 0 ? 0 : taken > kSample ? kSample : taken;
  int col = -1;  // used after the rows
  if (tid < taken) {
    const int64_t j = (int64_t)tid * kPrecondRowParts + blockIdx.x;  // j * step + step <= nnz
    const uint32_t off = (((uint32_t)j * 2654435761u) >> 4) % (uint32_t)step;  // nnz < 2^31
    col = indices[j * step + off];
  }
  double s2 = 0.0, s3 = 0.0, us = 0.0;
#pragma unroll 4
  for (int64_t i = (int64_t)blockIdx.x * 1024 + tid; i < n; i += 1024 * kPrecondRowParts) {
    const double c = (double)(indptr[i + 1] - indptr[i]);
    s2 = fma(c, c, s2);
    s3 = fma(c * c, c, s3);
    us += c > 16.0 ? kLongRowUs : c > 4.0 ? kDeepEntryUs * (c - 4.0) : 0.0;
  }
  __syncthreads();
  if (col >= 0) atomicAdd(&hist[col], 1);
  s2 = wave_sum(s2);
  s3 = wave_sum(s3);
  us = wave_sum(us);
  __syncthreads();
  double most = tid < d ? (double)hist[tid] : 0.0;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) most = fmax(most, __shfl_xor(most, off, 64));
  if ((tid & 63) == 0) {
    red[0][tid >> 6] = s2;
    red[1][tid >> 6] = s3;
    red[2][tid >> 6] = us;
    red[3][tid >> 6] = most;
  }
  __syncthreads();
  if (tid) return;
  for (int w = 1; w < 16; ++w) {
    s2 += red[0][w];
    s3 += red[1][w];
    us += red[2][w];
    most = fmax(most, red[3][w]);
  }
  part[blockIdx.x] = s2;
  part[kPrecondRowParts + blockIdx.x] = s3;
  part[2 * kPrecondRowParts + blockIdx.x] = us;
  part[3 * kPrecondRowParts + blockIdx.x] =
      taken > 0 ? fmax(most - 2.0 * sqrt(most), 0.0) / (double)taken : 0.0;
}

unsigned guard_blocks(int64_t d) { return (unsigned)ceil_div(d, (int64_t)kGuardCols); }

}  // namespace

void precond_estimate(const psk_mat &A, const double *R, const double *N, double *g,
                      double *est, hipStream_t st) {
  const int64_t d = A.d;
  if (R) {
    k_col_norm_upper<<<guard_blocks(d), 64 * kGuardWaves, 0, st>>>(R, d, g);
    k_guard<<<guard_blocks(d), 64 * kGuardWaves, 0, st>>>(N, d, g, 0, est);
  } else {
    k_guard<<<guard_blocks(d), 64 * kGuardWaves, 0, st>>>(N, d, N, 1, est);
  }
  if (A.format == PSK_CSR)
    k_row_stats<<<kPrecondRowParts, 1024, 0, st>>>(A.indptr, A.indices, A.n, A.nnz, (int)d,
                                                  est + kMaxGuard);
}

bool precond_doubtful(const psk_mat &A, double err) {
  return A.format == PSK_DENSE && A.n >= 4 * kNormRows && err > 1e-3 && err <= kPrecondMax;
}

void precond_estimate_rows(const psk_mat &A, const double *N, double *g, double *est,
                           hipStream_t st) {
  const int64_t d = A.d;
  const unsigned nb = guard_blocks(d);
  if (A.dtype == PSK_F64)
    k_col_norm_sample<<<nb, 64 * kGuardWaves, 0, st>>>((const double *)A.values, A.ld, A.n, d, N, g);
  else
    k_col_norm_sample<<<nb, 64 * kGuardWaves, 0, st>>>((const float *)A.values, A.ld, A.n, d, N, g);
  k_guard<<<nb, 64 * kGuardWaves, 0, st>>>(N, d, g, 0, est);
}

double precond_error(const double *est, int64_t d) {
  double s = 0.0;
  for (unsigned b = 0; b < guard_blocks(d); ++b) s += est[b];
  return kGuardC * s;
}

RowStats precond_row_stats(const double *est, int64_t d) {
  RowStats r{0.0, 0.0, 0.0, 0.0};
  for (int b = 0; b < kPrecondRowParts; ++b) {
    r.squares += est[kMaxGuard + b];
    r.cubes += est[kMaxGuard + kPrecondRowParts + b];
    r.pass_us += est[kMaxGuard + 2 * kPrecondRowParts + b];
    r.share += est[kMaxGuard + 3 * kPrecondRowParts + b] / kPrecondRowParts;
  }
  r.share = fmax(r.share, 1.0 / (double)d);
  return r;
}

RowStats precond_row_bounds(const psk_mat &A) {
  const double nnz = (double)A.nnz, len = std::fmax(nnz / (double)A.n, 1.0);
  return RowStats{len, len * len, nnz / 17.0 * kLongRowUs + 0.75 * nnz * kDeepEntryUs,
                  1.0 / (double)A.d};
}

int precond_sharpen(const psk_mat &A, const double *N, bool caller, double *P, Arena &ws,
                    hipStream_t st) {
  const int64_t d = A.d;
  double *G = ws.take<double>((size_t)d * d);
  double *W = ws.take<double>((size_t)d * d);
  double *S = ws.take<double>((size_t)d * d);
  double *X = ws.take<double>((size_t)d * d);
  double *U = caller ? ws.take<double>((size_t)d * d) : nullptr;
  double *part = ws.take<double>(kMaxGuard);
  int *flag = ws.take<int>(4);
  const bool run = !ws.dry();
  if (run && !ws.ok()) return fail(PSK_ENOMEM, "workspace too small for the preconditioner");
  const size_t mk = ws.mark();
  const unsigned ew = (unsigned)ceil_div(d * d, (int64_t)256);
  int rc = A.format == PSK_DENSE ? gram_dense(1.0, A, 0.0, G, ws, st, true)
                                 : gram_csr(1.0, A, 0.0, G, ws, st, true);
  if (rc) return rc;
  ws.release(mk);
  const double *T = N;
  if (caller) {
    if (run) k_upper<<<ew, 256, 0, st>>>(N, d, U);
    T = U;
  }
  if ((rc = dgemm(false, false, d, d, d, 1.0, G, d, T, d, 0.0, S, d, ws, st, kTriB))) return rc;
  ws.release(mk);
  if ((rc = dgemm(true, false, d, d, d, 1.0, T, d, S, d, 0.0, W, d, ws, st, kTriAT))) return rc;
  ws.release(mk);
  if ((rc = chol_factor(W, d, S, X, flag, ws, st))) return rc;
  ws.release(mk);
  if ((rc = dgemm(false, false, d, d, d, 1.0, T, d, X, d, 0.0, P, d, ws, st, kTriA | kTriB)))
    return rc;
  ws.release(mk);
  if (!run) return 0;
  k_guard<<<guard_blocks(d), 64 * kGuardWaves, 0, st>>>(P, d, G, 2, part);
  k_precond_pick<<<ew, 256, 0, st>>>(N, d, part, (int)guard_blocks(d), flag, P);
  PSK_HIP_TRY(hipGetLastError());
  return 0;
}

}  // namespace psk
