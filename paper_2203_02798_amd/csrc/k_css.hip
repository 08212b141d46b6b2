// Column subset selection and the leverage scores of the selected columns
// (arXiv 2203.02798, section 4.1 Algorithm cgrrqr and section 4.3 Algorithm
// ls_hrn_exact).
//
// css_select: the sketch B = G S A (or S A for m == 0), then the first k
// steps of the column-pivoted Householder QR of B (Businger and Golub): at
// step j the remaining column with the largest norm of its rows j .. rows-1
// is chosen (lowest index on ties) and a Householder reflector that zeroes
// its rows below j is applied to every remaining column.  The chosen columns
// are the selection.  Only the permutation is kept (R is not returned).
//
// leverage_css: the exact leverage scores of A[:, K] for the selected K
// (Algorithm ls_direct on the column subset).  A[:, K] is never formed: its
// Gram matrix is the K x K block of A^T A, whose Cholesky factor R_K gives
// theta_i = ||e_i^T A[:, K] R_K^{-1}||^2 = ||e_i^T A B||^2 with B the d x k
// matrix that holds the rows of R_K^{-1} at the rows K and zeros elsewhere.
//
// Layout and kernels.  The sketch (rows x d, row-major) is transposed once so
// that every column is contiguous (k_transpose, 32 x 32 tiles through LDS).
// k_col_norms gives the squared column norms.  One k_qrcp_step launch per
// pivot: every workgroup finds the pivot p from the norms of the previous
// step (a redundant argmax over d values), and each wavefront owns one
// column: it forms w = v^T c with the reflector v read from column p, updates
// its column and recomputes the squared norm of its rows j+1 .. rows-1
// exactly (no downdating).  The norms are double-buffered across launches, so
// no launch reads what it writes; column p is only read during its step.
// Sums run over lanes in a fixed order and then a fixed butterfly, so the
// selection is deterministic.
//
// A launch per pivot is bound by the launch (1000 x 500: 6.3 us a pivot, two
// of them work), and the choice itself needs inner products only.  So the
// pivots are first looked for in the Gram matrix of the sketch: the pivoted
// Cholesky factorization of G = B^T B meets the same columns, its remaining
// diagonal being the squared norms that the QR recomputes.  One workgroup
// takes a panel of up to 16 pivots with its rows of the factor in LDS
// (k_pivot_panel: 23 us for 16 at d = 500), the whole chip then takes the
// panel out of G (k_schur: 5 us), and 100 pivots of 1000 x 500 take 0.23 ms
// with G, not 0.63.  What squaring loses is watched: a pivot counts only if it leads the
// next candidate by more than kPivotGap of the largest squared norm, some
// 1e5 times what rounding can have moved either.  At the first that does not
// (equal columns, norms near rounding level, nothing left) the QR steps take
// over.  They need the sketch as the steps before would have left it, and with
// the pivots known that is made sixteen steps a pass (k_replay_panel and
// k_replay_rest: 24 + 18 us for 16 at 1000 x 500, 2.6 a pivot), in the steps' own
// arithmetic: the rest of the selection is, bit for bit, what steps from the
// start choose.  Whole calls in us, steps alone / search and steps: 1000 x 500,
// k = 500, singular values over eight decades 2867 / 2620, equal columns near the
// start 2910 / 2890; 2000 x 1000, k = 1000, eight decades 11,515 / 9080.
#include <type_traits>

#include "internal.hpp"

namespace psk {
namespace {

constexpr int kTile = 32;

// Bt[c * rows + i] = C[i * d + c]; blockIdx.x over row tiles, blockIdx.y
// over column tiles; 256 threads = 32 x 8.
__global__ __launch_bounds__(256) void k_transpose(const double *__restrict__ C, int64_t rows,
                                                   int64_t d, double *__restrict__ Bt) {
  __shared__ double tile[kTile][kTile + 1];
  const int64_t i0 = (int64_t)blockIdx.x * kTile, c0 = (int64_t)blockIdx.y * kTile;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  for (int y = ty; y < kTile; y += 8) {
    const int64_t i = i0 + y, c = c0 + tx;
    if (i < rows && c < d) tile[y][tx] = C[i * d + c];
  }
  __syncthreads();
  for (int y = ty; y < kTile; y += 8) {
    const int64_t c = c0 + y, i = i0 + tx;
    if (i < rows && c < d) Bt[c * rows + i] = tile[tx][y];
  }
}

// norms[c] = sum_i Bt[c, i]^2, a wavefront per column.
__global__ __launch_bounds__(256) void k_col_norms(const double *__restrict__ Bt, int64_t rows,
                                                   int64_t d, double *__restrict__ norms) {
  const int lane = threadIdx.x & 63;
  const int64_t c = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (c >= d) return;
  const double *col = Bt + c * rows;
  double s = 0.0;
  for (int64_t i = lane; i < rows; i += 64) s = fma(col[i], col[i], s);
  s = wave_sum(s);
  if (lane == 0) norms[c] = s;
}

// Rows per lane that k_qrcp_step keeps in registers (the rows below the
// pivot row of up to 64 * kQrReg rows); longer columns stream through memory
// twice.  Both forms add the same terms in the same order.
constexpr int kQrReg = 16;

// (v, i) pair reduction: the larger value, the lower index on equal values.
__device__ __forceinline__ void argmax_merge(double &v, int &i, double v2, int i2) {
  if (v2 > v || (v2 == v && i2 < i)) {
    v = v2;
    i = i2;
  }
}

// One pivot step j.  nin: squared norms of rows j.. of the live columns, -1
// for chosen ones; nout receives the same for step j + 1.
__global__ __launch_bounds__(256) void k_qrcp_step(double *__restrict__ Bt, int64_t rows,
                                                   int64_t d, int64_t j,
                                                   const double *__restrict__ nin,
                                                   double *__restrict__ nout,
                                                   int32_t *__restrict__ cols) {
  __shared__ double sv[4];
  __shared__ int si[4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // argmax over the live columns, lowest index on equal norms; a NaN norm
  // (non-finite input) counts as -0.5, below every other live column but
  // above the chosen ones (-1), so p is always a live column (j < d)
  double best = -1.0;
  int bi = 0x7fffffff;
  for (int c = tid; c < d; c += 256) {
    const double v0 = nin[c];
    const double v = v0 != v0 ? -0.5 : v0;
    if (v > best) {
      best = v;
      bi = c;
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1)
    argmax_merge(best, bi, __shfl_xor(best, off, 64), __shfl_xor(bi, off, 64));
  if (lane == 0) {
    sv[wave] = best;
    si[wave] = bi;
  }
  __syncthreads();
  best = sv[0];
  bi = si[0];
#pragma unroll
  for (int w = 1; w < 4; ++w) argmax_merge(best, bi, sv[w], si[w]);
  const int p = bi;
  const double n2 = best;
  // no barrier below this point
  const int64_t c = (int64_t)blockIdx.x * 4 + wave;
  if (c >= d) return;
  const double nc = nin[c];
  if (nc < 0.0) {
    if (lane == 0) nout[c] = -1.0;
    return;
  }
  if (c == p) {
    if (lane == 0) {
      nout[c] = -1.0;
      cols[j] = (int32_t)c;
    }
    return;
  }
  double *col = Bt + c * rows;
  const double *x = Bt + (int64_t)p * rows;
  // reflector H = I - 2 v v^T / (v^T v), v = x - beta e_j on rows j..
  double v0 = 0.0, vtv = 1.0;
  const bool reflect = n2 > 0.0;
  if (reflect) {
    const double alpha = x[j];
    const double nx = sqrt(n2);
    const double beta = alpha >= 0.0 ? -nx : nx;
    v0 = alpha - beta;
    vtv = 2.0 * beta * (beta - alpha);
  }
  const double cj = col[j];
  const int64_t i0 = j + 1 + lane;
  double nn;
  if (rows - (j + 1) <= 64 * kQrReg) {
    double xr[kQrReg], cr[kQrReg];
#pragma unroll
    for (int t = 0; t < kQrReg; ++t) {
      const int64_t i = i0 + 64 * t;
      xr[t] = i < rows ? x[i] : 0.0;
      cr[t] = i < rows ? col[i] : 0.0;
    }
    double s = 0.0;
    if (reflect) {
      double part = 0.0;
#pragma unroll
      for (int t = 0; t < kQrReg; ++t) part = fma(xr[t], cr[t], part);
      s = 2.0 * fma(v0, cj, wave_sum(part)) / vtv;
    }
    double part2 = 0.0;
#pragma unroll
    for (int t = 0; t < kQrReg; ++t) {
      const int64_t i = i0 + 64 * t;
      const double y = fma(-s, xr[t], cr[t]);
      if (i < rows) col[i] = y;
      part2 = fma(y, y, part2);
    }
    nn = wave_sum(part2);
    if (lane == 0) col[j] = fma(-s, v0, cj);
  } else {
    double s = 0.0;
    if (reflect) {
      double part = 0.0;
#pragma unroll 4
      for (int64_t i = i0; i < rows; i += 64) part = fma(x[i], col[i], part);
      s = 2.0 * fma(v0, cj, wave_sum(part)) / vtv;
    }
    double part2 = 0.0;
#pragma unroll 4
    for (int64_t i = i0; i < rows; i += 64) {
      const double y = fma(-s, x[i], col[i]);
      col[i] = y;
      part2 = fma(y, y, part2);
    }
    nn = wave_sum(part2);
    if (lane == 0) col[j] = fma(-s, v0, cj);
  }
  if (lane == 0) nout[c] = nn;
}

// ---------------------------------------------------------------------------
// steps whose pivots are known
// ---------------------------------------------------------------------------
// A column of Bt as a wavefront holds it from row 64 tb on: lane l has the rows
// 64 (tb + u) + l, in registers (R > 0: u < R reaches the column's end) or in
// memory (R = 0; a lane reads back only what it wrote itself).  Row j is in
// u = 0 or 1 for the steps of one pass that starts in row block tb.
// k_qrcp_step's lane i at step j sums the rows j + 1 + i, j + 1 + i + 64, ..: the
// rows below j of this lane's (j + 1 + i) mod 64, in the same order.  So a sum
// here takes zeros for the rows up to j, which leave it as it is, and its lanes
// are rotated before they are added: the same additions.
template <int R>
struct QrColumn {
  double *col;
  int64_t rows, tb;
  int lane;
  double c[R > 0 ? R : 1];

  __device__ __forceinline__ int64_t row(int64_t u) const { return 64 * (tb + u) + lane; }
  __device__ __forceinline__ void load() {
    if constexpr (R > 0) {
#pragma unroll
      for (int u = 0; u < R; ++u) c[u] = row(u) < rows ? col[row(u)] : 0.0;
    }
  }
  __device__ __forceinline__ void store() {
    if constexpr (R > 0) {
#pragma unroll
      for (int u = 0; u < R; ++u)
        if (row(u) < rows) col[row(u)] = c[u];
    }
  }
  // row j of the column (uniform)
  __device__ __forceinline__ double at(int64_t j) const {
    const int64_t u = (j >> 6) - tb;
    double e;
    if constexpr (R > 0) e = u == 0 ? c[0] : c[1];
    else e = row(u) < rows ? col[row(u)] : 0.0;
    return __shfl(e, (int)(j & 63), 64);
  }
  // sum over the lanes in the order of step j
  __device__ __forceinline__ double sum(double part, int64_t j) const {
    return wave_sum(__shfl(part, (int)((lane + j + 1) & 63), 64));
  }
  // The step j of this column, as k_qrcp_step makes it: x(u) is the reflector's
  // column at row(u), zero up to row j and past the end.  Returns the squared
  // norm of the rows below j when it is asked for.
  template <class X>
  __device__ __forceinline__ double step(X x, double v0, double vtv, int64_t j, bool norm) {
    constexpr int N = R > 0 ? R : 16;  // R = 0: as many rows loaded at once
    const int64_t end = R > 0 ? N : (rows + 63) / 64 - tb;
    const double cj = at(j);
    double s = 0.0, part = 0.0, part2 = 0.0;
    for (int64_t b = 0; b < end; b += N) {
      double xv[N], cv[N];
#pragma unroll
      for (int u = 0; u < N; ++u) {
        xv[u] = x(b + u);
        cv[u] = R > 0 ? c[R > 0 ? u : 0] : row(b + u) < rows ? col[row(b + u)] : 0.0;
      }
#pragma unroll
      for (int u = 0; u < N; ++u) part = fma(xv[u], cv[u], part);
    }
    if (vtv != 0.0) s = 2.0 * fma(v0, cj, sum(part, j)) / vtv;
    for (int64_t b = 0; b < end; b += N) {
      double xv[N], cv[N];
#pragma unroll
      for (int u = 0; u < N; ++u) {
        xv[u] = x(b + u);
        cv[u] = R > 0 ? c[R > 0 ? u : 0] : row(b + u) < rows ? col[row(b + u)] : 0.0;
      }
#pragma unroll
      for (int u = 0; u < N; ++u) {
        const double y = fma(-s, xv[u], cv[u]);
        if constexpr (R > 0) c[u] = y;
        else if (row(b + u) < rows) col[row(b + u)] = y;
        const double z = (R == 0 || u < 2) && row(b + u) <= j ? 0.0 : y;
        part2 = fma(z, z, part2);
      }
    }
    return norm ? sum(part2, j) : 0.0;
  }
};

// The steps j0 .. j0 + nb - 1, nb <= W, of the columns that they choose
// (cols[j0 ..]): one workgroup, a wavefront per column.  Column t is final after
// t steps, is handed to the others through LDS (R = 0: through memory) and is
// the reflector of the next.  refl[2 t], refl[2 t + 1]: v's first element and
// v^T v, 0 for no reflection.  Two buffers, so one barrier a step.  Bound by the
// chain of a step: two sums over the lanes, a square root and a division.
template <int R, int W>
__global__ __launch_bounds__(64 * W) void k_replay_panel(double *__restrict__ Bt, int64_t rows,
                                                         int64_t j0, int nb,
                                                         const double *__restrict__ norms,
                                                         const int32_t *__restrict__ cols,
                                                         double *__restrict__ refl) {
  extern __shared__ double xs[];  // 2 x 64 R
  __shared__ double vs[2][2];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const bool mine = wave < nb;
  const int64_t p = mine ? cols[j0 + wave] : 0;
  QrColumn<R> q{Bt + p * rows, rows, j0 >> 6, lane};
  if (mine) q.load();
  double n2 = mine ? norms[p] : 0.0;
  for (int t = 0; t < nb; ++t) {
    const int64_t j = j0 + t;
    double *xt = xs + (t & 1) * 64 * R;
    if (wave == t) {
      double v0 = 0.0, vtv = 0.0;
      if (n2 > 0.0) {
        const double alpha = q.at(j);
        const double nx = sqrt(n2);
        const double beta = alpha >= 0.0 ? -nx : nx;
        v0 = alpha - beta;
        vtv = 2.0 * beta * (beta - alpha);
      }
      if constexpr (R > 0) {
#pragma unroll
        for (int u = 0; u < R; ++u) xt[64 * u + lane] = u < 2 && q.row(u) <= j ? 0.0 : q.c[u];
      }
      if (lane == 0) {
        vs[t & 1][0] = refl[2 * t] = v0;
        vs[t & 1][1] = refl[2 * t + 1] = vtv;
      }
    }
    __syncthreads();
    if (!mine || wave <= t) continue;
    const double v0 = vs[t & 1][0], vtv = vs[t & 1][1];
    const bool next = wave == t + 1;
    double nn;
    if constexpr (R > 0) {
      nn = q.step([&](int64_t u) { return xt[64 * u + lane]; }, v0, vtv, j, next);
    } else {
      const double *x = Bt + (int64_t)cols[j] * rows;
      nn = q.step([&](int64_t u) { return q.row(u) > j && q.row(u) < rows ? x[q.row(u)] : 0.0; },
                  v0, vtv, j, next);
    }
    if (next) n2 = nn;
  }
  if (mine) q.store();
}

// The same steps of every other live column, a wavefront each; norms: theirs
// after the last of them, -1 for the columns chosen.  A workgroup stages the
// reflector of the next step in LDS beside a step (R = 0: reads it from memory).
template <int R>
__global__ __launch_bounds__(256) void k_replay_rest(double *__restrict__ Bt, int64_t rows,
                                                     int64_t d, int64_t j0, int nb,
                                                     const double *__restrict__ refl,
                                                     const int32_t *__restrict__ cols,
                                                     double *__restrict__ norms) {
  extern __shared__ double xs[];  // 2 x 64 R
  const int lane = threadIdx.x & 63;
  const int64_t c = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  const bool chosen =
      __ballot(lane < nb && cols[j0 + (lane < nb ? lane : 0)] == c) != 0;
  const bool live = c < d && !chosen && !(norms[c < d ? c : 0] < 0.0);
  if (chosen && lane == 0) norms[c] = -1.0;
  QrColumn<R> q{Bt + (live ? c : 0) * rows, rows, j0 >> 6, lane};
  if (live) q.load();
  double nn = 0.0;
  if constexpr (R > 0) {
    constexpr int M = R / 4;  // elements of a reflector a thread stages
    const int64_t first = 64 * (j0 >> 6) + threadIdx.x;
    double x[M];
    auto fetch = [&](int t) __attribute__((always_inline)) {
      const double *xp = Bt + (int64_t)cols[j0 + t] * rows;
#pragma unroll
      for (int u = 0; u < M; ++u) {
        const int64_t i = first + 256 * u;
        x[u] = i < rows && i > j0 + t ? xp[i] : 0.0;
      }
    };
    fetch(0);
    for (int t = 0; t < nb; ++t) {
      double *xt = xs + (t & 1) * 64 * R;
#pragma unroll
      for (int u = 0; u < M; ++u) xt[threadIdx.x + 256 * u] = x[u];
      __syncthreads();
      if (t + 1 < nb) fetch(t + 1);
      if (live)
        nn = q.step([&](int64_t u) { return xt[64 * u + lane]; }, refl[2 * t], refl[2 * t + 1],
                    j0 + t, t == nb - 1);
    }
  } else if (live) {
    for (int t = 0; t < nb; ++t) {
      const int64_t j = j0 + t;
      const double *x = Bt + (int64_t)cols[j] * rows;
      nn = q.step([&](int64_t u) { return q.row(u) > j && q.row(u) < rows ? x[q.row(u)] : 0.0; },
                  refl[2 * t], refl[2 * t + 1], j, t == nb - 1);
    }
  }
  if (!live) return;
  q.store();
  if (lane == 0) norms[c] = nn;
}

// ---------------------------------------------------------------------------
// pivots from the Gram matrix
// ---------------------------------------------------------------------------
constexpr int kPanel = 16;  // pivots a panel at most
constexpr double kPivotGap = 1e-10;
constexpr double kPivotTiny = 1e-290;  // squared norms down here have lost their digits

// The largest value of a wavefront in every lane: four shifts inside rows of
// 16 lanes and two row broadcasts leave it in lane 63 (register moves, where
// a shuffle goes through LDS).
__device__ __forceinline__ double wave_max(double v) {
  auto step = [&](auto ctrl, auto rows) __attribute__((always_inline)) {
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)b, hi = (uint32_t)(b >> 32);
    const uint32_t l2 = (uint32_t)__builtin_amdgcn_update_dpp((int)lo, (int)lo, decltype(ctrl)::value,
                                                              decltype(rows)::value, 0xf, false);
    const uint32_t h2 = (uint32_t)__builtin_amdgcn_update_dpp((int)hi, (int)hi, decltype(ctrl)::value,
                                                              decltype(rows)::value, 0xf, false);
    v = fmax(v, __longlong_as_double((long long)(((uint64_t)h2 << 32) | l2)));
  };
  using std::integral_constant;
  step(integral_constant<int, 0x111>{}, integral_constant<int, 0xf>{});  // row_shr 1
  step(integral_constant<int, 0x112>{}, integral_constant<int, 0xf>{});  // row_shr 2
  step(integral_constant<int, 0x114>{}, integral_constant<int, 0xf>{});  // row_shr 4
  step(integral_constant<int, 0x118>{}, integral_constant<int, 0xf>{});  // row_shr 8
  step(integral_constant<int, 0x142>{}, integral_constant<int, 0xa>{});  // row_bcast 15
  step(integral_constant<int, 0x143>{}, integral_constant<int, 0xc>{});  // row_bcast 31
  const uint64_t b = (uint64_t)__double_as_longlong(v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, 63);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), 63);
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// The best and second best of the candidates: value and column of the best,
// value of the second (equal to the best where two tie).
struct Top2 {
  double v1, v2;
  int i1;
};

__device__ __forceinline__ void top2_merge(Top2 &a, double v1, int i1, double v2) {
  if (v1 > a.v1) {
    a.v2 = fmax(a.v1, v2);
    a.v1 = v1;
    a.i1 = i1;
  } else {
    a.v2 = fmax(a.v2, v1);
  }
}

// res[c] = G[c, c], state: pivots found, 1 once the search has stopped
__global__ __launch_bounds__(256) void k_pivot_start(const double *__restrict__ G, int64_t d,
                                                     double *__restrict__ res,
                                                     int *__restrict__ state) {
  const int64_t c = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (c < d) res[c] = G[c * d + c];
  if (c == 0) state[0] = state[1] = 0;
}

// Pivots j0 .. j0 + nb - 1 of G, from which the factor rows before j0 are
// taken out.  Thread t owns columns t, t + blockDim.x, .. (OWN of them) and
// keeps its entries of the panel's factor rows in registers; LDS holds the
// rows too, for the pivot column's entries.  res: remaining squared norms, -1
// for chosen columns; L: the panel's rows of the factor (nb x d).  top[0]: the
// largest squared norm of all (written by the first panel).  One barrier a
// pivot: the reductions alternate between two buffers, and a factor row
// written before the barrier is read after it.  Bound by latencies in a row
// (the reduction, the barrier, the row of G): 0.8 us a pivot at d = 500.
template <int OWN, int NP>
__global__ __launch_bounds__(1024) void k_pivot_panel(const double *__restrict__ G, int64_t d,
                                                      int64_t j0, int nb,
                                                      double *__restrict__ res,
                                                      double *__restrict__ top,
                                                      double *__restrict__ L,
                                                      int *__restrict__ state,
                                                      int32_t *__restrict__ cols) {
  extern __shared__ double Ls[];  // NP x d
  __shared__ double r1[2][16], r2[2][16];
  __shared__ int ri[2][16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int nw = blockDim.x >> 6;
  if (state[1]) return;
  double rv[OWN], l[OWN][NP];
#pragma unroll
  for (int u = 0; u < OWN; ++u) {
    const int c = tid + u * (int)blockDim.x;
    rv[u] = c < d ? res[c] : -1.0;
  }
  double gap = j0 ? fmax(kPivotGap * top[0], kPivotTiny) : 0.0;
  int done = 0;
  bool stop = false;
#pragma unroll
  for (int t = 0; t < NP; ++t) {
    if (t >= nb || stop) continue;  // uniform
    Top2 b = {-1.0, -1.0, 0x7fffffff};
#pragma unroll
    for (int u = 0; u < OWN; ++u)  // a chosen column, or a NaN, is no candidate
      if (rv[u] >= 0.0) top2_merge(b, rv[u], tid + u * (int)blockDim.x, -1.0);
    const double m1 = wave_max(b.v1);
    const uint64_t at = __ballot(b.v1 == m1);  // never empty: no candidate is a NaN
    const int src = __ffsll((unsigned long long)at) - 1;
    const double m2 = wave_max(lane == src ? b.v2 : b.v1);
    const int i1 = __builtin_amdgcn_readlane(b.i1, src);
    if (lane == 0) {
      r1[t & 1][wave] = m1;
      r2[t & 1][wave] = m2;
      ri[t & 1][wave] = i1;
    }
    __syncthreads();
    b = {r1[t & 1][0], r2[t & 1][0], ri[t & 1][0]};
    for (int w = 1; w < nw; ++w) top2_merge(b, r1[t & 1][w], ri[t & 1][w], r2[t & 1][w]);
    if (j0 == 0 && t == 0) {
      gap = fmax(kPivotGap * b.v1, kPivotTiny);
      if (tid == 0) top[0] = b.v1;
    }
    // no clear leader (uniform; also true for NaN): leave the rest to the QR
    if (!(b.v1 > gap && b.v1 - fmax(b.v2, 0.0) > gap)) {
      stop = true;
      continue;
    }
    const int p = __builtin_amdgcn_readfirstlane(b.i1);
    const double *gp = G + (int64_t)p * d;
    double g[OWN], lp[NP];
#pragma unroll
    for (int u = 0; u < OWN; ++u) {
      const int c = tid + u * (int)blockDim.x;
      g[u] = gp[c < d ? c : 0];
    }
#pragma unroll
    for (int q = 0; q < t; ++q) lp[q] = Ls[q * d + p];
    const double inv = 1.0 / sqrt(b.v1);
#pragma unroll
    for (int u = 0; u < OWN; ++u) {
      const int c = tid + u * (int)blockDim.x;
#pragma unroll
      for (int q = 0; q < t; ++q) g[u] = fma(-lp[q], l[u][q], g[u]);
      l[u][t] = rv[u] >= 0.0 ? g[u] * inv : 0.0;
      if (c < d) Ls[t * d + c] = l[u][t];
      if (c == p) {
        rv[u] = -1.0;
        cols[j0 + t] = (int32_t)c;
      } else if (rv[u] >= 0.0) {
        rv[u] = fmax(fma(-l[u][t], l[u][t], rv[u]), 0.0);
      }
    }
    done = t + 1;
  }
  if (tid == 0) {
    state[0] = (int)j0 + done;
    state[1] = stop ? 1 : 0;
  }
  if (stop) return;
#pragma unroll
  for (int u = 0; u < OWN; ++u) {
    const int c = tid + u * (int)blockDim.x;
    if (c >= d) continue;
    res[c] = rv[u];
#pragma unroll
    for (int q = 0; q < NP; ++q)
      if (q < nb) L[(int64_t)q * d + c] = l[u][q];
  }
}

// G -= L^T L for the nb rows of a panel (all of G: rows and columns of chosen
// pivots are not read again): 16 x 64 elements a workgroup, its columns of L
// loaded together
__global__ __launch_bounds__(256) void k_schur(double *__restrict__ G, int64_t d, int nb,
                                               const double *__restrict__ L,
                                               const int *__restrict__ state) {
  __shared__ double la[kPanel][16];
  const int stopped = state[1];
  if (d > 1024 && stopped) return;  // (waited for: below, that is most of the launch)
  const int x = threadIdx.x & 63, y = threadIdx.x >> 6;
  const int64_t c = (int64_t)blockIdx.x * 64 + x, a0 = (int64_t)blockIdx.y * 16;
  const int64_t cc = c < d ? c : d - 1;
  double lc[kPanel], g[4];
#pragma unroll
  for (int q = 0; q < kPanel; ++q) lc[q] = q < nb ? L[(int64_t)q * d + cc] : 0.0;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int64_t a = a0 + 4 * y + u;
    g[u] = G[(a < d ? a : d - 1) * d + cc];
  }
  {
    const int q = threadIdx.x >> 4;
    const int64_t a = a0 + (threadIdx.x & 15);
    la[q][threadIdx.x & 15] = q < nb ? L[(int64_t)q * d + (a < d ? a : d - 1)] : 0.0;
  }
  __syncthreads();
  if (stopped || c >= d) return;
#pragma unroll
  for (int q = 0; q < kPanel; ++q)
#pragma unroll
    for (int u = 0; u < 4; ++u) g[u] = fma(-la[q][4 * y + u], lc[q], g[u]);
#pragma unroll
  for (int u = 0; u < 4; ++u)
    if (a0 + 4 * y + u < d) G[(a0 + 4 * y + u) * d + c] = g[u];
}

// W[a, b] = G[cols[a], cols[b]] (k x k block of the d x d Gram matrix).
__global__ __launch_bounds__(256) void k_gather_block(const double *__restrict__ G, int64_t d,
                                                      const int32_t *__restrict__ cols, int64_t k,
                                                      double *__restrict__ W) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= k * k) return;
  const int64_t a = idx / k, b = idx - a * k;
  W[idx] = G[(int64_t)cols[a] * d + cols[b]];
}

// B (d x k, zero on entry) gets row a of X (k x k) at row cols[a].
__global__ __launch_bounds__(256) void k_scatter_rows(const double *__restrict__ X, int64_t k,
                                                      const int32_t *__restrict__ cols,
                                                      double *__restrict__ B) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= k * k) return;
  const int64_t a = idx / k, b = idx - a * k;
  B[(int64_t)cols[a] * k + b] = X[idx];
}

__global__ __launch_bounds__(256) void k_zero(double *__restrict__ p, int64_t count) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += stride)
    p[i] = 0.0;
}

unsigned grid_for(int64_t count) {
  const int64_t b = ceil_div(count, 256);
  return (unsigned)(b < 8192 ? b : 8192);
}

}  // namespace

int css_select_impl(const psk_mat &A, int64_t m, int64_t r, int64_t k, uint64_t seed, int prec,
                    int32_t *cols, Arena &ws, hipStream_t st) {
  const int64_t d = A.d;
  if (d > 4096) return fail(PSK_EUNSUPPORTED, "column subset selection supports d <= 4096");
  const int64_t rows = m > 0 ? m : r;
  double *C = ws.take<double>((size_t)rows * d);
  double *Bt = ws.take<double>((size_t)rows * d);
  double *na = ws.take<double>((size_t)d);
  double *nb = ws.take<double>((size_t)d);
  int *flag = ws.take<int>(4);  // [0]: non-finite sketch; [2], [3]: the pivot search's state
  const bool run = !ws.dry();
  if (run && !ws.ok()) return fail(PSK_ENOMEM, "workspace too small for css_select");
  const size_t mk = ws.mark();
  int rc;
  if ((rc = sketch_f64(A, m, r, seed, prec, C, ws, st))) return rc;
  ws.release(mk);
  if (!run) return 0;
  // pivots chosen by norms with a NaN in them are meaningless: the sketch is
  // checked first and read back before the selection runs
  k_zero<<<1, 64, 0, st>>>(reinterpret_cast<double *>(flag), 2);
  flag_nonfinite(C, rows * d, flag, st);
  // The search in the Gram matrix, where that is the shorter way (in us: G at
  // 40 TFLOP/s, four launches, two a panel and 1.5 a pivot or more, against 5
  // a pivot and the sketch read and written at 4 TB/s for each) and the
  // transposed sketch's room holds G and the partial sums of it.  Measured
  // whole calls, 20,000 rows, steps / search: d = 32, k = 16 352 / 159; d =
  // 500, k = 20 636 / 325; d = 1000, k = 100 1992 / 1045.
  const double gram_us = 20.0 + (double)rows * d * d / 40e6 + 10.0 * ceil_div(k, (int64_t)kPanel) +
                         (double)k * (1.5 + (double)d * 1e-3);
  const double steps_us = (double)k * (5.0 + (double)rows * d * 16.0 / 4e6);
  const int64_t room = rows * d - d * d;
  const bool search =
      k > 1 && gram_us < steps_us && room >= dgram_room(d) && room >= kPanel * d;
  int h[4] = {0, 0, 0, 1};  // h[2]: pivots found, h[3]: some are left to the steps
  if (search) {
    KTimer timer("pivots", st);
    double *G = Bt, *L = Bt + d * d;  // L where the partial sums of G were
    if ((rc = dgram(C, rows, d, G, Bt + d * d, room, st))) return rc;
    k_pivot_start<<<(unsigned)ceil_div(d, (int64_t)256), 256, 0, st>>>(G, d, na, flag + 2);
    const dim3 sg((unsigned)ceil_div(d, (int64_t)64), (unsigned)ceil_div(d, (int64_t)16));
    // a column a thread while 1024 threads suffice; the factor rows of a panel
    // fit LDS (128 KiB)
    ReadBack early;
    auto panels = [&](auto own, auto np) -> int {
      constexpr int OWN = decltype(own)::value, NP = decltype(np)::value;
      const unsigned threads = (unsigned)(ceil_div(d, (int64_t)(64 * OWN)) * 64);
      const size_t lds = (size_t)NP * d * sizeof(double);
      PSK_HIP_TRY(hipFuncSetAttribute((const void *)k_pivot_panel<OWN, NP>,
                                      hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
      for (int64_t j = 0; j < k; j += NP) {
        const int n1 = (int)(k - j < NP ? k - j : NP);
        k_pivot_panel<OWN, NP><<<1, threads, lds, st>>>(G, d, j, n1, na, nb, L, flag + 2, cols);
        if (j + n1 < k) k_schur<<<sg, 256, 0, st>>>(G, d, n1, L, flag + 2);
        // Panels after a stop find nothing to do, at two launches each.  A long
        // search that has stopped in its first two panels is ended; the third runs
        // while the host waits to know (1000 x 500, k = 500, the first two columns
        // equal: 3230 us without, 2940 so).
        if (j == NP && k > 14 * NP) {
          if (int rb = early.start(flag + 2, 2 * sizeof(int), st)) return rb;
          if (int rb = early.mark(st)) return rb;
        } else if (j == 2 * NP && k > 14 * NP) {
          if (int rb = early.wait(h + 2)) return rb;
          if (h[3]) break;
        }
      }
      return 0;
    };
    using std::integral_constant;
    if (d <= 1024) rc = panels(integral_constant<int, 1>{}, integral_constant<int, kPanel>{});
    else if (d <= 2048) rc = panels(integral_constant<int, 2>{}, integral_constant<int, 8>{});
    else rc = panels(integral_constant<int, 4>{}, integral_constant<int, 4>{});
    if (rc) return rc;
  }
  if ((rc = read_back(h, flag, (search ? 4 : 1) * sizeof(int), st))) return rc;
  if ((rc = factor_status(h[0], ""))) return rc;
  if (search && !h[3]) return 0;
  KTimer timer("qrcp", st);
  const dim3 tg((unsigned)ceil_div(rows, (int64_t)kTile), (unsigned)ceil_div(d, (int64_t)kTile));
  k_transpose<<<tg, 256, 0, st>>>(C, rows, d, Bt);
  const unsigned cb = (unsigned)ceil_div(d, (int64_t)4);
  k_col_norms<<<cb, 256, 0, st>>>(Bt, rows, d, na);
  // the steps whose pivots are known, a pass of 16 or 8 (the registers of a column)
  auto replay = [&](auto regs, auto width, int64_t j) -> int {
    constexpr int R = decltype(regs)::value, W = decltype(width)::value;
    const int steps = (int)(h[2] - j < W ? h[2] - j : W);
    const size_t lds = (size_t)2 * 64 * R * sizeof(double);
    double *refl = C;  // the sketch is in Bt now
    PSK_HIP_TRY(hipFuncSetAttribute((const void *)k_replay_panel<R, W>,
                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    PSK_HIP_TRY(hipFuncSetAttribute((const void *)k_replay_rest<R>,
                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    k_replay_panel<R, W><<<1, 64 * W, lds, st>>>(Bt, rows, j, steps, na, cols, refl);
    k_replay_rest<R><<<cb, 256, lds, st>>>(Bt, rows, d, j, steps, refl, cols, na);
    return steps;
  };
  for (int64_t j = 0; j < h[2];) {
    using std::integral_constant;
    using W16 = integral_constant<int, 16>;
    using W8 = integral_constant<int, 8>;
    const int64_t blocks = ceil_div(rows, (int64_t)64) - (j >> 6);
    const int rc = blocks <= 16   ? replay(W16{}, W16{}, j)
                   : blocks <= 32 ? replay(integral_constant<int, 32>{}, W8{}, j)
                   : blocks <= 64 ? replay(integral_constant<int, 64>{}, W8{}, j)
                                  : replay(integral_constant<int, 0>{}, W16{}, j);
    if (rc < 0) return rc;
    j += rc;
  }
  for (int64_t j = h[2]; j < k; ++j) {
    k_qrcp_step<<<cb, 256, 0, st>>>(Bt, rows, d, j, na, nb, cols);
    double *t = na;
    na = nb;
    nb = t;
  }
  PSK_HIP_TRY(hipGetLastError());
  return 0;
}

int leverage_css_impl(const psk_mat &A, int64_t m, int64_t r, int64_t k, uint64_t seed, int prec,
                      double *theta, int32_t *cols, Arena &ws, hipStream_t st) {
  const int64_t d = A.d;
  if (d > 4096) return fail(PSK_EUNSUPPORTED, "leverage_css supports d <= 4096");
  int32_t *kc = cols ? cols : ws.take<int32_t>((size_t)k);
  double *G = ws.take<double>((size_t)d * d);
  double *W = ws.take<double>((size_t)k * k);
  double *R = ws.take<double>((size_t)k * k);
  double *X = ws.take<double>((size_t)k * k);
  double *B = ws.take<double>((size_t)d * k);
  int *flag = ws.take<int>(4);
  const bool run = !ws.dry();
  if (run && !ws.ok()) return fail(PSK_ENOMEM, "workspace too small for leverage_css");
  const size_t mk = ws.mark();
  int rc;
  if ((rc = css_select_impl(A, m, r, k, seed, prec, kc, ws, st))) return rc;
  ws.release(mk);
  rc = A.format == PSK_DENSE ? gram_dense(1.0, A, 0.0, G, ws, st, true)
                             : gram_csr(1.0, A, 0.0, G, ws, st, true);
  if (rc) return rc;
  ws.release(mk);
  if (run) k_gather_block<<<(unsigned)ceil_div(k * k, (int64_t)256), 256, 0, st>>>(G, d, kc, k, W);
  if ((rc = chol_factor(W, k, R, X, flag, ws, st))) return rc;
  ws.release(mk);
  if (run) {
    k_zero<<<grid_for(d * k), 256, 0, st>>>(B, d * k);
    k_scatter_rows<<<(unsigned)ceil_div(k * k, (int64_t)256), 256, 0, st>>>(X, k, kc, B);
  }
  rc = A.format == PSK_DENSE ? rownorms_dense(1.0, A, B, k, 0.0, theta, ws, st)
                             : rownorms_csr(1.0, A, B, k, 0.0, theta, ws, st);
  if (rc) return rc;
  if (!run) return 0;
  PSK_HIP_TRY(hipGetLastError());
  flag_nonfinite(theta, A.n, flag, st);
  int h = 0;
  if ((rc = read_back(&h, flag, sizeof(int), st))) return rc;
  return factor_status(h, "a Cholesky pivot was not positive: the selected columns are numerically rank deficient");
}

}  // namespace psk
