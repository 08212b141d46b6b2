// R and R^{-1} of an FP64 sketch C (m x d) on gfx950 by shifted
// Cholesky-QR with two extra Cholesky-QR passes (sCQR3: Fukaya, Kannan,
// Nakatsukasa, Yamamoto, Yanagisawa, "Shifted Cholesky QR for computing the
// QR factorization of ill-conditioned matrices", SIAM J. Sci. Comput. 2020).
//
// Paper mapping (arXiv 2203.02798): the sketch-based algorithms
// (ls_approximate_drineas, least_squares_precondition) factor the sketch
// G*S*A and use the inverse factor as an orthogonaliser / right
// preconditioner; the paper uses an SVD, here the triangular factor of a QR
// (the same column space, so the same leverage scores and an equally good
// preconditioner).  Cholesky-QR keeps the work in GEMMs on the matrix cores
// (W = C^T C, Q = C R^{-1}); the shift s = 11 (m d + d (d+1)) u ||C||_F^2 on
// the first pass keeps the Cholesky factorization defined for condition
// numbers up to about 1/u, and up to two unshifted passes restore
// orthogonality.  The second pass stops the factorisation when its Gram
// matrix is within 1/2 of the identity: then the first pass's Q was
// already that well conditioned, the second pass leaves it orthonormal
// to rounding level (Cholesky-QR loses orthogonality like cond(Q)^2 u), and
// a third pass would change R only by rounding.  Otherwise (ill-conditioned
// C) the third pass runs as in sCQR3.
//
// The d x d Cholesky and the inverse of its factor are blocked by 64 columns
// with one launch per block step (k_chol_step, below): the panel, the
// trailing update, the partial products of R^{-1} and the factorization of
// the next diagonal block all happen in the same launch, so a pass costs
// ceil(d/64) + 2 launches besides its two GEMMs with C.  Up to 64 columns a
// pass is one workgroup's launch (k_chol_small, k_later_small).
#include "internal.hpp"

namespace psk {
namespace {

// Before a blocked Cholesky, in one launch: R = X = 0, flag cleared (when
// given) and W[i][i] += coef * trace(W) (coef != 0), the last by workgroup 0.
__global__ __launch_bounds__(256) void k_chol_prep(double *__restrict__ W, int64_t d, double coef,
                                                   double *__restrict__ R, double *__restrict__ X,
                                                   int *__restrict__ flag) {
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < d * d;
       e += (int64_t)gridDim.x * 256) {
    R[e] = 0.0;
    X[e] = 0.0;
  }
  if (blockIdx.x != 0) return;
  if (flag && threadIdx.x < 4) flag[threadIdx.x] = 0;
  if (coef == 0.0) return;
  __shared__ double red[4];
  double s = 0.0;
  for (int64_t i = threadIdx.x; i < d; i += 256) s += W[i * d + i];
  s = wave_sum(s);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  const double tr = red[0] + red[1] + red[2] + red[3];
  for (int64_t i = threadIdx.x; i < d; i += 256) W[i * d + i] += coef * tr;
}

// ---------------------------------------------------------------------------
// Blocked Cholesky W = R^T R with X = R^{-1}, 64-column blocks, one kernel
// launch per block step.  Step j (k_chol_step) runs one 256-thread workgroup
// per 64 x 64 tile of work:
//   panel    R[j, J]  = X_jj^T W[j, J]                       (J > j)
//   trailing W[I, J] -= P_I^T P_J,  P_K = X_jj^T W[j, K]     (j < I <= J)
//   partial  P_j[I][K] = X[I, K] R[K, j]                     (I <= K <= j-2)
//   finish   X[I, c]  = -(sum_K P_c[I][K] + X[I, c-1] R[c-1, c]) X_cc
//                                                   (c = j - 1, I < c)
// and the workgroup that owns the next diagonal tile (j+1, j+1), whose update
// is the last one it receives, factors it in the same launch (Cholesky and
// triangular inverse of the 64 x 64 block), so the next step finds R_{j+1,j+1}
// and X_{j+1,j+1} ready.  The off-diagonal blocks of X = R^{-1}, whose sums
// run over up to d - 64 terms, are split into 64-term partial products so
// that no workgroup carries a long sum; a block column is summed (in K
// order) and finished one launch after its partials, and one extra launch
// finishes the last column.  Block 0 is factored by k_chol_first.  W is read
// in its upper block triangle and destroyed.
//
// What bounds a step is the one workgroup that ends in a factorization, a
// chain of 64 pivots; the other tiles of the launch hide behind it.  The 64 x 64
// products run on the matrix cores, operands in LDS; inside the factorization
// one wavefront factors a 16 x 16 block while the other three update the
// rest, and the inverse is carried along with the updates instead of being
// formed after them.
// ---------------------------------------------------------------------------
typedef double v4d __attribute__((ext_vector_type(4)));
constexpr int kLd = 68;      // LDS row stride of 64-wide tiles (doubles)
constexpr int kTh = 256;
constexpr int kVb = 16 * 17;  // one 16 x 16 block inverse in LDS (row stride 17)

struct CholSmem {
  double X[64 * kLd];        // an operand tile; the inverse of the factored tile
  double PI[64 * kLd];       // operand tiles; PJ also the tile to factor
  double PJ[64 * kLd];
  double V[4 * kVb];         // block inverses of the diagonal factor
};

// lane L of each row of 16 lanes, to all of that row (one DPP move)
template <int L>
__device__ __forceinline__ double row_bcast(double v) {
  return __builtin_amdgcn_update_dpp(0.0, v, 0x150 + L, 0xf, 0xf, true);
}

__device__ __forceinline__ void wave_sync_lds() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ v4d mfma16(double a, double b, v4d c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// 1/sqrt(x) to about an ulp: the hardware estimate (about 2^-24) and one
// third-order correction from the residual e = 1 - x y^2 taken with an FMA.
__device__ __forceinline__ double rsqrt_acc(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double e = fma(-(x * y), y, 1.0);
  return fma(y * e, fma(e, 0.375, 0.5), y);
}

// x_r -= U_kr u and z_r -= U_kr zk for N consecutive rows r of a step, U_kr
// being u's element in lane r of the row of 16: one FMA each, its DPP operand
// doing the broadcast (the compiler makes a move and a dependent FMA of it, 32
// cycles a row against 8.5).  The s_nop gives the two wait states a DPP operand
// needs after the VALU has written it.
#define PSK_ROW_UPDATE(X, Z, U, ZK, R)                                                  \
  "v_fmac_f64_dpp %" X ", -%" U ", %" U " row_newbcast:%" R " row_mask:0xf bank_mask:0xf\n\t" \
  "v_fmac_f64_dpp %" Z ", -%" U ", %" ZK " row_newbcast:%" R " row_mask:0xf bank_mask:0xf\n\t"

template <int R, int N>
__device__ __forceinline__ void update_rows(double (&x)[16], double (&z)[16], double u,
                                            double zk) {
  if constexpr (N >= 5) {
    asm("s_nop 1\n\t" PSK_ROW_UPDATE("0", "5", "10", "11", "12")
            PSK_ROW_UPDATE("1", "6", "10", "11", "13") PSK_ROW_UPDATE("2", "7", "10", "11", "14")
                PSK_ROW_UPDATE("3", "8", "10", "11", "15")
                    PSK_ROW_UPDATE("4", "9", "10", "11", "16")
        : "+v"(x[R]), "+v"(x[R + 1]), "+v"(x[R + 2]), "+v"(x[R + 3]), "+v"(x[R + 4]),
          "+v"(z[R]), "+v"(z[R + 1]), "+v"(z[R + 2]), "+v"(z[R + 3]), "+v"(z[R + 4])
        : "v"(u), "v"(zk), "n"(R), "n"(R + 1), "n"(R + 2), "n"(R + 3), "n"(R + 4));
    update_rows<R + 5, N - 5>(x, z, u, zk);
  } else if constexpr (N >= 2) {
    asm("s_nop 1\n\t" PSK_ROW_UPDATE("0", "2", "4", "5", "6")
            PSK_ROW_UPDATE("1", "3", "4", "5", "7")
        : "+v"(x[R]), "+v"(x[R + 1]), "+v"(z[R]), "+v"(z[R + 1])
        : "v"(u), "v"(zk), "n"(R), "n"(R + 1));
    update_rows<R + 2, N - 2>(x, z, u, zk);
  } else if constexpr (N == 1) {
    asm("s_nop 1\n\t" PSK_ROW_UPDATE("0", "1", "2", "3", "4")
        : "+v"(x[R]), "+v"(z[R])
        : "v"(u), "v"(zk), "n"(R));
  }
}

// Step k of factor16 and those after it.
template <int K>
__device__ __forceinline__ void factor16_step(double (&x)[16], double (&z)[16], double &dg,
                                              int &bad) {
  const double piv = row_bcast<K>(dg);
  double rs = rsqrt_acc(piv);
  bad |= !(piv > 0.0) ? 1 : 0;
  bad |= !(fabs(piv) <= 1.7976931348623157e308) ? 2 : 0;  // NaN or infinite
  rs = piv > 0.0 ? rs : 1.0;
  const double u = x[K] * rs, zk = z[K] * rs;
  x[K] = u;
  z[K] = zk;
  if constexpr (K < 15) {
    dg = fma(-u, u, dg);
    update_rows<K + 1, 15 - K>(x, z, u, zk);
    factor16_step<K + 1>(x, z, dg, bad);
  }
}

// One wavefront: Cholesky of the symmetric 16 x 16 block at (o, o) of the LDS
// tile T; every row of 16 lanes does the same work, lane l % 16 holding column
// l % 16 of the block in x and of the identity in z.  The row operations that
// turn the block into U (scale row k by 1/U_kk, subtract U_ki times row k
// from row i) turn the identity into U^{-T}, so lane l ends with row l of V =
// U^{-1} in z.  U overwrites the block's upper triangle (what is left below
// the diagonal means nothing) and V goes to Vb (row-major, stride 17).  A
// step's chain is pivot, reciprocal square root, scaled row, next pivot; each
// lane keeps its column's diagonal entry apart, whose update needs only the
// lane's own element of the row.  With the multipliers through LDS (a write
// and up to seven 16-byte reads a step) a block took 5100 cycles, now
// 3300.  Returns bit 1 when a pivot was not positive (its row is then not
// scaled), bit 2 when one was NaN or infinite.
__device__ __forceinline__ int factor16(double *__restrict__ T, int o,
                                        double *__restrict__ Vb) {
  const int lane = threadIdx.x & 63, l = lane & 15;
  double x[16], z[16], dg = T[(o + l) * kLd + o + l];
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    x[i] = T[(o + i) * kLd + o + l];
    z[i] = i == l ? 1.0 : 0.0;
  }
  int bad = 0;
  factor16_step<0>(x, z, dg, bad);
  if (lane < 16) {
#pragma unroll
    for (int i = 0; i < 16; ++i) T[(o + i) * kLd + o + l] = x[i];
  } else if (lane < 32) {
#pragma unroll
    for (int i = 0; i < 16; ++i) Vb[l * 17 + i] = z[i];
  }
  return bad;
}

// 16 x 16 tiles in LDS, one wavefront.  The accumulator's element e of lane
// (kq, li) = (lane / 16, lane % 16) is row kq + 4 e, column li.
__device__ __forceinline__ v4d tile_get(const double *__restrict__ T, int ld) {
  const int li = threadIdx.x & 15, kq = (threadIdx.x >> 4) & 3;
  v4d c;
#pragma unroll
  for (int e = 0; e < 4; ++e) c[e] = T[(kq + 4 * e) * ld + li];
  return c;
}
__device__ __forceinline__ void tile_put(double *__restrict__ T, int ld, v4d c) {
  const int li = threadIdx.x & 15, kq = (threadIdx.x >> 4) & 3;
#pragma unroll
  for (int e = 0; e < 4; ++e) T[(kq + 4 * e) * ld + li] = c[e];
}
// c + sign * P^T Q (TN) or c + sign * P Q, all 16 x 16
template <bool TN>
__device__ __forceinline__ v4d tile_mul(const double *__restrict__ P, int ldp,
                                        const double *__restrict__ Q, int ldq, double sign,
                                        v4d c) {
  const int li = threadIdx.x & 15, kq = (threadIdx.x >> 4) & 3;
  double a[4], b[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    a[s] = TN ? P[(4 * s + kq) * ldp + li] : P[li * ldp + 4 * s + kq];
    b[s] = Q[(4 * s + kq) * ldq + li];
  }
  // two chains: a product waits for two matrix instructions, not four
  v4d c2 = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    c = mfma16(sign * a[s], b[s], c);
    c2 = mfma16(sign * a[2 + s], b[2 + s], c2);
  }
  return c + c2;
}

// All 256 threads.  T: the 64 x 64 tile (row-major, stride kLd), of which the
// leading nb x nb block's upper triangle is used (the rest is taken as
// identity); XT: LDS for the inverse.  Right-looking Cholesky over four
// 16-column blocks.  Once block kb is factored (U_kb, V_kb = U_kb^{-1}):
//   panel     U[kb, J] = V_kb^T T[kb, J] (J > kb),
//             X[I, kb] = Y[I, kb] V_kb   (I < kb), X[kb, kb] = V_kb
//   trailing  T[I, J] -= U[kb, I]^T U[kb, J]  (kb < I <= J)
//             Y[I, J] -= X[I, kb] U[kb, J]    (I <= kb < J; Y starts as 0)
// so the inverse's sums ride along with the updates.  Wavefront 0 updates and
// factors the next diagonal block while the others do the rest.  Writes the nb x nb
// blocks of R (= U, zero below the diagonal) and X at (j0, j0).
// A 64 x 64 tile takes 24,000 cycles (10 us): 3300 a diagonal block, 1900 the panel and update
// between two, 2800 writing R and X.  With VALU products and the inverse formed afterwards it took
// 62,000; a step (m = 2000, d = 500) 18 us instead of 37.
__device__ __forceinline__ void factor_diag(double *__restrict__ T, double *__restrict__ XT,
                                            CholSmem &S, int nb, int64_t d, int64_t j0,
                                            double *__restrict__ R, double *__restrict__ X,
                                            int *__restrict__ flag) {
  const int tid = threadIdx.x, wave = tid >> 6;
  if (nb < 64) {
    for (int e = tid; e < 64 * 64; e += kTh) {
      const int i = e >> 6, j = e & 63;
      if (i >= nb || j >= nb) T[i * kLd + j] = (i == j) ? 1.0 : 0.0;
    }
    __syncthreads();
  }
  auto tb = [&](double *M, int I, int J) { return M + 16 * I * kLd + 16 * J; };
  int bad = 0;
  // one copy of the code for all four blocks: straight-line code run once is
  // fetched once, and the fetch, not the arithmetic, then sets its pace
#pragma unroll 1
  for (int kb = 0; kb < 4; ++kb) {
    // V_{kb-1} is at hand; update what block kb - 1 leaves to update
    if (wave == 0) {
      double *t = tb(T, kb, kb);
      if (kb > 0) {
        const double *u = tb(T, kb - 1, kb);
        tile_put(t, kLd, tile_mul<true>(u, kLd, u, kLd, -1.0, tile_get(t, kLd)));
        wave_sync_lds();
      }
      bad |= factor16(T, 16 * kb, S.V + kb * kVb);
    } else if (kb > 0) {
      // the other products of block row kb - 1, dealt to wavefronts 1 .. 3
      int n = 0;
#pragma unroll 1
      for (int J = kb; J < 4; ++J) {
#pragma unroll 1
        for (int I = 0; I <= J; ++I) {
          if ((I == kb && J == kb) || n++ % 3 != wave - 1) continue;
          const double *q = tb(T, kb - 1, J);
          if (I >= kb) {
            double *t = tb(T, I, J);
            tile_put(t, kLd,
                     tile_mul<true>(tb(T, kb - 1, I), kLd, q, kLd, -1.0, tile_get(t, kLd)));
          } else {
            double *y = tb(XT, I, J);  // its first product when I = kb - 1
            v4d c = {0.0, 0.0, 0.0, 0.0};
            if (I < kb - 1) c = tile_get(y, kLd);
            tile_put(y, kLd, tile_mul<false>(tb(XT, I, kb - 1), kLd, q, kLd, -1.0, c));
          }
        }
      }
    }
    __syncthreads();
    // panel: three products whatever kb, one each for wavefronts 0 .. 2;
    // wavefront 3 copies V_kb
    const double *V = S.V + kb * kVb;
    if (wave < 3 - kb) {
      double *t = tb(T, kb, kb + 1 + wave);
      tile_put(t, kLd, tile_mul<true>(V, 17, t, kLd, 1.0, v4d{0.0, 0.0, 0.0, 0.0}));
    } else if (wave < 3) {
      double *y = tb(XT, wave - (3 - kb), kb);
      tile_put(y, kLd, tile_mul<false>(y, kLd, V, 17, 1.0, v4d{0.0, 0.0, 0.0, 0.0}));
    } else {
      tile_put(tb(XT, kb, kb), kLd, tile_get(V, 17));
    }
    __syncthreads();
  }
  const int j = tid & 63;
  double rv[16], xv[16];
#pragma unroll
  for (int p = 0; p < 16; ++p) {
    const int i = wave + 4 * p;
    const bool up = (i >> 4) <= (j >> 4);  // the blocks below hold nothing
    const double a = T[i * kLd + j], b = XT[i * kLd + j];
    rv[p] = i <= j ? a : 0.0;
    xv[p] = up ? b : 0.0;
  }
#pragma unroll
  for (int p = 0; p < 16; ++p) {
    const int i = wave + 4 * p;
    if (i < nb && j < nb) {
      R[(j0 + i) * d + j0 + j] = rv[p];
      X[(j0 + i) * d + j0 + j] = xv[p];
    }
  }
  if (bad) atomicOr(flag, bad);
}

// a 64 x 64 tile of a row-major d-wide matrix at (r0, c0), rows < rows and
// columns < cols of it, zero outside: loaded into registers, then stored
struct Tile64 {
  double v[16];
  __device__ __forceinline__ void load(const double *__restrict__ M, int64_t d, int64_t r0,
                                       int64_t c0, int rows, int cols) {
    const int j = threadIdx.x & 63, i0 = threadIdx.x >> 6;
    const bool jin = j < cols;
#pragma unroll
    for (int p = 0; p < 16; ++p) {
      const int i = i0 + 4 * p;
      const bool in = jin && i < rows;
      const double x = M[in ? (r0 + i) * d + c0 + j : 0];
      v[p] = in ? x : 0.0;
    }
  }
  __device__ __forceinline__ void store(double *__restrict__ T) const {
    const int j = threadIdx.x & 63, i0 = threadIdx.x >> 6;
#pragma unroll
    for (int p = 0; p < 16; ++p) T[(i0 + 4 * p) * kLd + j] = v[p];
  }
};

// This wavefront's 16-column strip w of a 64 x 64 product, four 16 x 16
// blocks down it.  TN: acc[a] += sign * P^T Q with P, Q in LDS by rows of the
// summed index; else acc[a] += sign * P Q.  TRI 1: P^T is lower triangular,
// 2: Q is upper triangular (products with their zero blocks left out).
template <bool TN, int TRI>
__device__ __forceinline__ void strip_mul(v4d (&acc)[4], const double *__restrict__ P,
                                          const double *__restrict__ Q, int w, double sign) {
  const int li = threadIdx.x & 15, kq = (threadIdx.x >> 4) & 3;
#pragma unroll
  for (int K = 0; K < 4; ++K) {
    if (TRI == 2 && K > w) break;  // uniform over the wavefront
#pragma unroll
    for (int s = 4 * K; s < 4 * K + 4; ++s) {
      const double b = Q[(4 * s + kq) * kLd + 16 * w + li];
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        if (TRI == 1 && K > a) continue;
        const double p = TN ? P[(4 * s + kq) * kLd + 16 * a + li]
                            : P[(16 * a + li) * kLd + 4 * s + kq];
        acc[a] = mfma16(sign * p, b, acc[a]);
      }
    }
  }
}

__device__ __forceinline__ void strip_zero(v4d (&acc)[4]) {
#pragma unroll
  for (int a = 0; a < 4; ++a) acc[a] = v4d{0.0, 0.0, 0.0, 0.0};
}

// P = X^T W in place of W: a wavefront reads and writes its own columns of P
__device__ __forceinline__ void panel_in_place(const double *__restrict__ X,
                                               double *__restrict__ P) {
  const int w = threadIdx.x >> 6;
  v4d acc[4];
  strip_zero(acc);
  strip_mul<true, 1>(acc, X, P, w, 1.0);
  wave_sync_lds();
#pragma unroll
  for (int a = 0; a < 4; ++a) tile_put(P + 16 * a * kLd + 16 * w, kLd, acc[a]);
}

__global__ __launch_bounds__(kTh) void k_chol_first(const double *__restrict__ W, int64_t d,
                                                    double *__restrict__ R,
                                                    double *__restrict__ X,
                                                    int *__restrict__ flag) {
  __shared__ CholSmem S;
  const int nb = (int)(d < 64 ? d : 64);
  Tile64 t;
  t.load(W, d, 0, 0, nb, nb);
  t.store(S.PJ);
  __syncthreads();
  factor_diag(S.PJ, S.X, S, nb, d, 0, R, X, flag);
}

__global__ __launch_bounds__(kTh) void k_chol_step(double *__restrict__ W, int64_t d,
                                                   int nblk, int j,
                                                   double *__restrict__ R,
                                                   double *__restrict__ X,
                                                   int *__restrict__ flag,
                                                   double *__restrict__ xpart) {
  __shared__ CholSmem S;
  const int p = j < nblk ? nblk - j - 1 : 0;
  const int ntrail = p * (p + 1) / 2;
  const int npart = (j >= 2 && j < nblk) ? (j - 1) * j / 2 : 0;
  const int cfin = j - 1;  // the X block column finished in this launch
  const int nfin = cfin >= 1 ? cfin : 0;
  int t = blockIdx.x;
  const int64_t j0 = (int64_t)j * 64;
  const int nbj = (int)((d - j0) < 64 ? (d - j0) : 64);
  const int w = threadIdx.x >> 6, li = threadIdx.x & 15, kq = (threadIdx.x >> 4) & 3;
  auto width = [&](int64_t c0) { return (int)(d - c0 < 64 ? d - c0 : 64); };
  if (t < ntrail) {
    // trailing tile (I, J), enumerated row by row of the upper block triangle
    int I = j + 1, rem = t;
    while (rem >= nblk - I) { rem -= nblk - I; ++I; }
    const int J = I + rem;
    const int64_t r0 = (int64_t)I * 64, c0 = (int64_t)J * 64;
    Tile64 tx, ti, tj;
    tx.load(X, d, j0, j0, nbj, nbj);
    ti.load(W, d, j0, r0, nbj, width(r0));
    if (I == J) {
      // a diagonal tile: the ten 16 x 16 blocks of its upper triangle, two
      // or three a wavefront
      constexpr int kA[4][3] = {{0, 0, 1}, {0, 1, 2}, {0, 1, 0}, {2, 3, 0}};
      constexpr int kB[4][3] = {{0, 1, 1}, {2, 2, 2}, {3, 3, 3}, {3, 3, 3}};
      const int cnt = w < 2 ? 3 : 2;
      int ba[3], bb[3];
      v4d acc[3];
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        ba[q] = w == 0 ? kA[0][q] : w == 1 ? kA[1][q] : w == 2 ? kA[2][q] : kA[3][q];
        bb[q] = w == 0 ? kB[0][q] : w == 1 ? kB[1][q] : w == 2 ? kB[2][q] : kB[3][q];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int64_t gi = r0 + 16 * ba[q] + kq + 4 * e, gj = c0 + 16 * bb[q] + li;
          const bool in = gi < d && gj < d;
          const double x = W[in ? gi * d + gj : 0];
          acc[q][e] = in ? x : 0.0;
        }
      }
      tx.store(S.X);
      ti.store(S.PI);
      __syncthreads();
      panel_in_place(S.X, S.PI);
      __syncthreads();
#pragma unroll
      for (int s = 0; s < 16; ++s) {
        const double *row = S.PI + (4 * s + kq) * kLd + li;
#pragma unroll
        for (int q = 0; q < 3; ++q)
          if (q < cnt) acc[q] = mfma16(-row[16 * ba[q]], row[16 * bb[q]], acc[q]);
      }
      if (I == j + 1) {
        // the next diagonal tile, whose last update this is: factored here
#pragma unroll
        for (int q = 0; q < 3; ++q)
          if (q < cnt) tile_put(S.PJ + 16 * ba[q] * kLd + 16 * bb[q], kLd, acc[q]);
        __syncthreads();
        factor_diag(S.PJ, S.X, S, width(r0), d, r0, R, X, flag);
      } else {
#pragma unroll
        for (int q = 0; q < 3; ++q)
          if (q < cnt) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const int64_t gi = r0 + 16 * ba[q] + kq + 4 * e, gj = c0 + 16 * bb[q] + li;
              if (gi < d && gj < d) W[gi * d + gj] = acc[q][e];
            }
          }
      }
      return;
    }
    tj.load(W, d, j0, c0, nbj, width(c0));
    v4d acc[4];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int64_t gi = r0 + 16 * a + kq + 4 * e, gj = c0 + 16 * w + li;
        const double x = W[gj < d ? gi * d + gj : 0];  // rows of block I < J are in range
        acc[a][e] = gj < d ? x : 0.0;
      }
    tx.store(S.X);
    ti.store(S.PI);
    tj.store(S.PJ);
    __syncthreads();
    panel_in_place(S.X, S.PI);
    panel_in_place(S.X, S.PJ);
    __syncthreads();
    strip_mul<true, 0>(acc, S.PI, S.PJ, w, -1.0);
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int64_t gi = r0 + 16 * a + kq + 4 * e, gj = c0 + 16 * w + li;
        if (gj < d) W[gi * d + gj] = acc[a][e];
      }
    return;
  }
  t -= ntrail;
  const int64_t half = (int64_t)(nblk - 2) * (nblk - 1) / 2 * 4096;  // tiles per parity
  if (t < npart) {
    // partial product P_j[I][K] = X[I, K] R[K, j] for I <= K <= j - 2
    int K = 0;
    while ((K + 1) * (K + 2) / 2 <= t) ++K;
    const int I = t - K * (K + 1) / 2;
    Tile64 tx, tr;
    tx.load(X, d, (int64_t)I * 64, (int64_t)K * 64, 64, 64);
    tr.load(R, d, (int64_t)K * 64, j0, 64, nbj);
    tx.store(S.PI);
    tr.store(S.PJ);
    __syncthreads();
    v4d acc[4];
    strip_zero(acc);
    strip_mul<false, 0>(acc, S.PI, S.PJ, w, 1.0);
    double *P = xpart + (j & 1) * half + (int64_t)t * 4096;
#pragma unroll
    for (int a = 0; a < 4; ++a) tile_put(P + 16 * a * 64 + 16 * w, 64, acc[a]);
    return;
  }
  t -= npart;
  if (t < nfin) {
    // X[I, c] = -(sum_{K=I}^{c-2} P_c[I][K] + X[I, c-1] R[c-1, c]) X_cc, c = cfin
    const int I = t, c = cfin;
    const int64_t r0 = (int64_t)I * 64, cm0 = (int64_t)(c - 1) * 64, c0 = (int64_t)c * 64;
    const int nbc = width(c0);
    Tile64 ta, tr, tx;
    ta.load(X, d, r0, cm0, 64, 64);
    tr.load(R, d, cm0, c0, 64, nbc);
    tx.load(X, d, c0, c0, nbc, nbc);
    const double *Pc = xpart + (c & 1) * half;
    v4d acc[4];
    strip_zero(acc);
#pragma unroll 4
    for (int K = I; K <= c - 2; ++K) {
      const double *pk = Pc + (int64_t)(K * (K + 1) / 2 + I) * 4096 + 16 * w;
#pragma unroll
      for (int a = 0; a < 4; ++a) acc[a] += tile_get(pk + 16 * a * 64, 64);
    }
    ta.store(S.PI);
    tr.store(S.PJ);
    tx.store(S.X);
    __syncthreads();
    strip_mul<false, 0>(acc, S.PI, S.PJ, w, 1.0);
    __syncthreads();  // PI is read by every wavefront
#pragma unroll
    for (int a = 0; a < 4; ++a) tile_put(S.PI + 16 * a * kLd + 16 * w, kLd, acc[a]);
    __syncthreads();
    strip_zero(acc);
    strip_mul<false, 2>(acc, S.PI, S.X, w, -1.0);
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int64_t gi = r0 + 16 * a + kq + 4 * e, gj = c0 + 16 * w + li;
        if (gj < d) X[gi * d + gj] = acc[a][e];
      }
    return;
  }
  t -= nfin;
  if (t < p) {
    // panel tile R[j, J] = X_jj^T W[j, J]
    const int64_t c0 = (int64_t)(j + 1 + t) * 64;
    Tile64 tx, tj;
    tx.load(X, d, j0, j0, nbj, nbj);
    tj.load(W, d, j0, c0, nbj, width(c0));
    tx.store(S.X);
    tj.store(S.PI);
    __syncthreads();
    v4d acc[4];
    strip_zero(acc);
    strip_mul<true, 1>(acc, S.X, S.PI, w, 1.0);
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int i = 16 * a + kq + 4 * e;
        const int64_t gj = c0 + 16 * w + li;
        if (i < nbj && gj < d) R[(j0 + i) * d + gj] = acc[a][e];
      }
  }
}

// ---------------------------------------------------------------------------
// Cholesky factor and inverse of a near-identity W = I + E by matrix products
// only (used for the second and third Cholesky-QR passes, whose Gram matrix
// is the identity up to a small E when the previous pass was accurate).
// With R = I + U (U upper triangular), R^T R = W reads U + U^T = E - U^T U,
// so U = Phi(E - U^T U) where Phi keeps the strict upper triangle and half
// the diagonal.  The fixed point iteration U_0 = Phi(E), U_{t+1} =
// Phi(E - U_t^T U_t) gains a factor ~||E|| per step; X = R^{-1} is the
// Neumann series I - U + U^2 - ..., evaluated as X_{t+1} = I - U X_t.  For
// ||E||_F <= kSeriesTol = 1e-4 two steps of each leave errors below 1e-16;
// smaller ||E|| needs fewer (series_depth).  ||E||_F is read back to the
// host (one stream synchronisation per pass), which picks the series or
// the blocked Cholesky and, after a second pass that took the series, ends
// the factorisation there.
// ---------------------------------------------------------------------------
constexpr double kSeriesTol = 1e-4;
// ||W - I||_F up to which a pass's Cholesky is the last: cond(Q)^2 is at most
// (1 + 1/2) / (1 - 1/2) = 3, and Cholesky-QR's loss of orthogonality, about
// cond(Q)^2 u, stays at rounding level.  The shift of the first pass leaves
// ||W - I|| at 1e-2 to 0.4 for sketches of condition number 1e3 to 1e4, which
// a bound of 1e-4 sent through a third pass (2048 x 256 at 1e3: 638 us a call,
// now 279 with the shorter products).
constexpr double kLastTol = 0.5;
constexpr int kParts = 64;

// part[b] = sum over a fixed slice of (W - I)^2, fixed reduction order
__global__ __launch_bounds__(256) void k_fro_partials(const double *__restrict__ W, int64_t d,
                                                      double *__restrict__ part) {
  __shared__ double red[4];
  const int64_t n = d * d;
  const int64_t chunk = ceil_div(n, kParts);
  const int64_t b0 = (int64_t)blockIdx.x * chunk;
  const int64_t b1 = b0 + chunk < n ? b0 + chunk : n;
  double s = 0.0;
  for (int64_t e = b0 + threadIdx.x; e < b1; e += 256) {
    const int64_t i = e / d, jj = e - i * d;
    const double v = W[e] - (i == jj ? 1.0 : 0.0);
    s = fma(v, v, s);
  }
  s = wave_sum(s);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) part[blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
}

// U = Phi(W - I) (the whole matrix: zero below the diagonal)
__global__ __launch_bounds__(256) void k_series_u0(const double *__restrict__ W, int64_t d,
                                                   double *__restrict__ U) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= d * d) return;
  const int64_t i = e / d, jj = e - i * d;
  U[e] = jj > i ? W[e] : (jj == i ? 0.5 * (W[e] - 1.0) : 0.0);
}

// U = Phi(W - I - T), T = U_prev^T U_prev
__global__ __launch_bounds__(256) void k_series_phi(const double *__restrict__ W,
                                                    const double *__restrict__ T, int64_t d,
                                                    double *__restrict__ U) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= d * d) return;
  const int64_t i = e / d, jj = e - i * d;
  const double m = W[e] - (i == jj ? 1.0 : 0.0) - T[e];
  U[e] = jj > i ? m : (jj == i ? 0.5 * m : 0.0);
}

// R = I + U, X = I - U (whole matrices)
__global__ __launch_bounds__(256) void k_series_rx(const double *__restrict__ U, int64_t d,
                                                   double *__restrict__ R,
                                                   double *__restrict__ X) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= d * d) return;
  const int64_t i = e / d, jj = e - i * d;
  const double id = (i == jj) ? 1.0 : 0.0;
  R[e] = id + U[e];
  X[e] = id - U[e];
}

// X = I - T on and above the diagonal, 0 below (T = U X_prev, upper)
__global__ __launch_bounds__(256) void k_series_x(const double *__restrict__ T, int64_t d,
                                                  double *__restrict__ X) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= d * d) return;
  const int64_t i = e / d, jj = e - i * d;
  X[e] = jj >= i ? (i == jj ? 1.0 : 0.0) - T[e] : 0.0;
}

// Upper Cholesky of W + coef trace(W) I (W is destroyed) into R, and X =
// R^{-1}; *flag (four ints) is cleared first with clear.
// xpart: scratch of at least d * d doubles for the partial products of the
// off-diagonal blocks of X (two block columns' worth, by parity).
__global__ void k_chol_small(const double *__restrict__ W, int64_t d, double coef,
                             double *__restrict__ R, double *__restrict__ X,
                             int *__restrict__ flag, int clear);

void chol_inv(double *W, int64_t d, double coef, double *R, double *X, int *flag, bool clear,
              double *xpart, hipStream_t st) {
  if (d <= 64) {
    k_chol_small<<<1, kTh, 0, st>>>(W, d, coef, R, X, flag, clear ? 1 : 0);
    return;
  }
  const int nblk = (int)ceil_div(d, 64);
  const int64_t pb = ceil_div(d * d, (int64_t)1024);
  k_chol_prep<<<(unsigned)(pb < 1024 ? pb : 1024), 256, 0, st>>>(W, d, coef, R, X,
                                                                 clear ? flag : nullptr);
  k_chol_first<<<1, kTh, 0, st>>>(W, d, R, X, flag);
  // launch j = nblk only finishes the last block column of X
  for (int j = 0; j <= nblk; ++j) {
    const int p = j < nblk ? nblk - j - 1 : 0;
    const int npart = (j >= 2 && j < nblk) ? (j - 1) * j / 2 : 0;
    const int nfin = j - 1 >= 1 ? j - 1 : 0;
    const int tiles = p * (p + 1) / 2 + npart + nfin + p;
    if (tiles > 0)
      k_chol_step<<<tiles, kTh, 0, st>>>(W, d, nblk, j, R, X, flag, xpart);
  }
}

// ||W - I||_F^2, summed on the host in a fixed order from kParts device
// partials (synchronises the stream).
int fro_dist_identity_sq(const double *W, int64_t d, double *part, hipStream_t st,
                         double *out) {
  k_fro_partials<<<kParts, 256, 0, st>>>(W, d, part);
  double h[kParts];
  int rc;
  if ((rc = read_back(h, part, sizeof(h), st))) return rc;
  double sum = 0.0;
  for (int b = 0; b < kParts; ++b) sum += h[b];
  *out = sum;
  return 0;
}

// Products of the series for ||E||_F = eps: after t fixed-point steps U is
// off by about 2^t eps^(t+2), and I - U + ... + (-U)^(t+1) by eps^(t+2).
__host__ __device__ inline int series_depth(double eps) {
  if (eps <= 1e-8) return 0;
  if (eps <= 3e-6) return 1;
  return 2;
}

// The whole of a first pass's Cholesky for d <= 64 in one launch: W + coef
// trace(W) I factored in LDS into R and X = R^{-1} (*flag cleared first with
// clear).
__global__ __launch_bounds__(kTh) void k_chol_small(const double *__restrict__ W, int64_t d,
                                                    double coef, double *__restrict__ R,
                                                    double *__restrict__ X,
                                                    int *__restrict__ flag, int clear) {
  __shared__ CholSmem S;
  __shared__ double shift;
  if (clear && threadIdx.x < 4) atomicExch(&flag[threadIdx.x], 0);
  Tile64 t;
  t.load(W, d, 0, 0, (int)d, (int)d);
  t.store(S.PJ);
  __threadfence();  // the cleared flag, ahead of what the factorization reports
  __syncthreads();
  if (threadIdx.x < 64) {
    const int i = threadIdx.x;
    const double tr = wave_sum(i < d ? S.PJ[i * kLd + i] : 0.0);
    if (i == 0) shift = coef * tr;
  }
  __syncthreads();
  if (coef != 0.0 && threadIdx.x < (unsigned)d) S.PJ[threadIdx.x * (kLd + 1)] += shift;
  __syncthreads();
  factor_diag(S.PJ, S.X, S, (int)d, d, 0, R, X, flag);
}

// A pass after the first for d <= 64 in one launch: from W = Q^T Q and the
// factors R1, X1 = R1^{-1} so far, R = R2 R1 and X = X1 X2 with R2 the
// Cholesky factor of W and X2 its inverse, by the series where ||W - I||_F <=
// kSeriesTol (as series_chol) and by factor_diag otherwise; dist = ||W -
// I||_F.  R2 and X2 are written by the second way only.  The d x d steps and
// products were up to 13 launches with nothing to do but start (a solve of 1e4
// x 32: 334 us with them, 309 now).
__global__ __launch_bounds__(kTh) void k_later_small(
    const double *__restrict__ W, int64_t d, const double *__restrict__ R1,
    const double *__restrict__ X1, double *__restrict__ R, double *__restrict__ X,
    double *__restrict__ R2, double *__restrict__ X2, double *__restrict__ dist,
    int *__restrict__ flag) {
  __shared__ CholSmem S;
  __shared__ double red[4];
  const int nb = (int)d;
  const int w = threadIdx.x >> 6, li = threadIdx.x & 15, kq = (threadIdx.x >> 4) & 3;
  const int j = threadIdx.x & 63, i0 = threadIdx.x >> 6;
  Tile64 t, r1, x1;
  t.load(W, d, 0, 0, nb, nb);
  r1.load(R1, d, 0, 0, nb, nb);
  x1.load(X1, d, 0, 0, nb, nb);
  double s = 0.0;
#pragma unroll
  for (int p = 0; p < 16; ++p) {
    const int i = i0 + 4 * p;
    const double v = i < nb && j < nb ? t.v[p] - (i == j ? 1.0 : 0.0) : 0.0;
    s = fma(v, v, s);
  }
  s = wave_sum(s);
  if (j == 0) red[i0] = s;
  t.store(S.PJ);
  __syncthreads();
  const double eps = sqrt((red[0] + red[1]) + (red[2] + red[3]));
  if (threadIdx.x == 0) dist[0] = eps;
  v4d acc[4];
  // element e of block a of this wavefront's strip
  auto each = [&](auto f) __attribute__((always_inline)) {
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int e = 0; e < 4; ++e) f(a, e, 16 * a + kq + 4 * e, 16 * w + li);
  };
  if (eps <= kSeriesTol) {
    const int depth = series_depth(eps);
    // U = Phi(W - I - T) in PI (W is zero outside d; so is U there)
    auto phi = [&](bool first) __attribute__((always_inline)) {
      each([&](int a, int e, int i, int c) {
        const double id = i == c && i < nb ? 1.0 : 0.0;
        const double m = S.PJ[i * kLd + c] - id - (first ? 0.0 : acc[a][e]);
        S.PI[i * kLd + c] = c > i ? m : (c == i ? 0.5 * m : 0.0);
      });
      __syncthreads();
    };
    phi(true);
    for (int q = 0; q < depth; ++q) {
      strip_zero(acc);
      strip_mul<true, 0>(acc, S.PI, S.PI, w, 1.0);
      __syncthreads();
      phi(false);
    }
    // X2 = I - U, then I - U X2
    each([&](int, int, int i, int c) {
      S.X[i * kLd + c] = (i == c ? 1.0 : 0.0) - S.PI[i * kLd + c];
    });
    __syncthreads();
    for (int q = 0; q < depth; ++q) {
      strip_zero(acc);
      strip_mul<false, 2>(acc, S.PI, S.X, w, 1.0);
      __syncthreads();
      each([&](int a, int e, int i, int c) {
        S.X[i * kLd + c] = c >= i ? (i == c ? 1.0 : 0.0) - acc[a][e] : 0.0;
      });
      __syncthreads();
    }
    // R2 = I + U
    if (threadIdx.x < 64) S.PI[threadIdx.x * (kLd + 1)] += 1.0;
  } else {
    factor_diag(S.PJ, S.X, S, nb, d, 0, R2, X2, flag);
    __syncthreads();
    each([&](int, int, int i, int c) {
      S.PI[i * kLd + c] = c >= i ? S.PJ[i * kLd + c] : 0.0;
      if (c < i) S.X[i * kLd + c] = 0.0;
    });
  }
  __syncthreads();
  auto put = [&](double *__restrict__ out) __attribute__((always_inline)) {
    each([&](int a, int e, int i, int c) {
      if (i < nb && c < nb) out[i * d + c] = c >= i ? acc[a][e] : 0.0;
    });
  };
  r1.store(S.PJ);
  __syncthreads();
  strip_zero(acc);
  strip_mul<false, 2>(acc, S.PI, S.PJ, w, 1.0);
  put(R);
  __syncthreads();
  x1.store(S.PJ);
  __syncthreads();
  strip_zero(acc);
  strip_mul<false, 2>(acc, S.PJ, S.X, w, 1.0);
  put(X);
}

// R = I + U, X = R^{-1} of W = I + E with ||E||_F <= kSeriesTol: U_0 =
// Phi(E), U_{t+1} = Phi(E - U_t^T U_t), X_1 = I - U, X_{t+1} = I - U X_t,
// `depth` steps of each.  B0, B1, B2: d x d scratch.
int series_chol(const double *W, int64_t d, int depth, double *R, double *X, double *B0,
                double *B1, double *B2, Arena &ws, hipStream_t st) {
  const bool run = !ws.dry();
  const unsigned ew = (unsigned)ceil_div(d * d, 256);
  const size_t mk = ws.mark();
  int rc;
  if (run) k_series_u0<<<ew, 256, 0, st>>>(W, d, B0);
  double *u = B0, *v = B1;
  for (int t = 0; t < depth; ++t) {
    if ((rc = dgemm(true, false, d, d, d, 1.0, u, d, u, d, 0.0, B2, d, ws, st, kTriAT | kTriB)))
      return rc;
    ws.release(mk);
    if (run) k_series_phi<<<ew, 256, 0, st>>>(W, B2, d, v);
    double *tmp = u; u = v; v = tmp;
  }
  if (run) k_series_rx<<<ew, 256, 0, st>>>(u, d, R, X);
  for (int t = 0; t < depth; ++t) {
    if ((rc = dgemm(false, false, d, d, d, 1.0, u, d, X, d, 0.0, B2, d, ws, st, kTriA | kTriB)))
      return rc;
    ws.release(mk);
    if (run) k_series_x<<<ew, 256, 0, st>>>(B2, d, X);
  }
  return 0;
}

// R, X of the Gram matrix W = Q^T Q of a pass after the first: the series
// when ||W - I||_F <= kSeriesTol, else the blocked Cholesky.  In a planning
// run (no data) both are planned.  *dist: ||W - I||_F.
int later_pass_chol(double *W, int64_t d, double *R, double *X, double *B0, double *B1,
                    double *B2, double *part, int *flag, double *dist, Arena &ws,
                    hipStream_t st) {
  int rc;
  if (ws.dry()) {
    *dist = INFINITY;
    return series_chol(W, d, 2, R, X, B0, B1, B2, ws, st);
  }
  double e2;
  if ((rc = fro_dist_identity_sq(W, d, part, st, &e2))) return rc;
  *dist = sqrt(e2);
  if (*dist <= kSeriesTol) return series_chol(W, d, series_depth(*dist), R, X, B0, B1, B2, ws, st);
  chol_inv(W, d, 0.0, R, X, flag, false, B2, st);
  return 0;
}

}  // namespace

int chol_factor(double *W, int64_t d, double *R, double *X, int *flag, Arena &ws,
                hipStream_t st) {
  if (d > 4096) return fail(PSK_EUNSUPPORTED, "the Cholesky factorization supports d <= 4096");
  double *xpart = ws.take<double>((size_t)d * d);
  if (ws.dry()) return 0;
  if (!ws.ok()) return fail(PSK_ENOMEM, "workspace too small for the Cholesky factorization");
  chol_inv(W, d, 0.0, R, X, flag, true, xpart, st);
  PSK_HIP_TRY(hipGetLastError());
  return 0;
}

int sketch_qr_impl(const double *C, int64_t m, int64_t d, double *R, double *Rinv,
                   Arena &ws, hipStream_t st, int **flag_out) {
  if (d > 4096) return fail(PSK_EUNSUPPORTED, "sketch_qr supports d <= 4096");
  double *Qa = ws.take<double>((size_t)m * d);
  double *Qb = ws.take<double>((size_t)m * d);
  double *W = ws.take<double>((size_t)d * d);
  double *R1 = ws.take<double>((size_t)d * d);
  double *R2 = ws.take<double>((size_t)d * d);
  double *R3 = ws.take<double>((size_t)d * d);
  double *X1 = ws.take<double>((size_t)d * d);
  double *X2 = ws.take<double>((size_t)d * d);
  double *X3 = ws.take<double>((size_t)d * d);
  double *T = ws.take<double>((size_t)d * d);
  double *B0 = ws.take<double>((size_t)d * d);
  double *B1 = ws.take<double>((size_t)d * d);
  double *B2 = ws.take<double>((size_t)d * d);
  double *part = ws.take<double>(kParts);
  int *flag = ws.take<int>(4);
  const bool run = !ws.dry();
  if (run && !ws.ok()) return fail(PSK_ENOMEM, "workspace too small for sketch_qr");
  const size_t mk = ws.mark();
  int rc;
  KTimer timer("sketch_qr", st, run);
  // flag[0]: a Cholesky pivot failed
  if (flag_out) *flag_out = flag;
  // W = Q^T Q, its partial sums in a copy of Q not in use at the time (too
  // small for dgram's tiles only below 32 or so columns)
  auto gram_of = [&](const double *Q, double *idle) -> int {
    if (m * d >= dgram_room(d)) return run ? dgram(Q, m, d, W, idle, m * d, st) : 0;
    const int e = dgemm(true, false, d, d, m, 1.0, Q, d, Q, d, 0.0, W, d, ws, st);
    ws.release(mk);
    return e;
  };
  // pass 1 (shifted): W = C^T C + s I, blocked Cholesky
  if ((rc = gram_of(C, Qb))) return rc;
  const double u = 1.1102230246251565e-16;
  const double coef = 11.0 * ((double)m * d + (double)d * (d + 1)) * u;
  if (run) chol_inv(W, d, coef, R1, X1, flag, true, B0, st);  // B0 is not in use yet
  // out = a * b for upper triangular b (m or d rows) or a and b (d x d)
  auto times = [&](const double *a, const double *b, int64_t rows, int tri, double *out) -> int {
    const int e = dgemm(false, false, rows, d, d, 1.0, a, d, b, d, 0.0, out, d, ws, st, tri);
    ws.release(mk);
    return e;
  };
  if ((rc = times(C, X1, m, kTriB, Qa))) return rc;
  // pass 2: W = Qa^T Qa
  if ((rc = gram_of(Qa, Qb))) return rc;
  double dist2 = 0.0, dist3 = 0.0;
  if (d <= 64) {
    // (planned by what follows, whose scratch is larger)
    if (run) {
      k_later_small<<<1, kTh, 0, st>>>(W, d, R1, X1, R, Rinv, R2, X2, part, flag);
      if ((rc = read_back(&dist2, part, sizeof(double), st))) return rc;
      if (dist2 <= kLastTol) return 0;
      if ((rc = times(Qa, X2, m, kTriB, Qb))) return rc;
      if ((rc = gram_of(Qb, Qa))) return rc;
      // so far R2 R1 = R and X1 X2 = Rinv, both replaced by the last pass's
      PSK_HIP_TRY(hipMemcpyAsync(T, R, (size_t)d * d * sizeof(double), hipMemcpyDeviceToDevice,
                                 st));
      PSK_HIP_TRY(hipMemcpyAsync(B0, Rinv, (size_t)d * d * sizeof(double),
                                 hipMemcpyDeviceToDevice, st));
      k_later_small<<<1, kTh, 0, st>>>(W, d, T, B0, R, Rinv, R3, X3, part, flag);
      PSK_HIP_TRY(hipGetLastError());
      return 0;
    }
  }
  if ((rc = later_pass_chol(W, d, R2, X2, B0, B1, B2, part, flag, &dist2, ws, st)))
    return rc;
  ws.release(mk);
  // When pass 2's W was near the identity, Q is orthonormal to rounding level
  // after it and a third pass would change R only at that level: R = R2 R1,
  // R^{-1} = X1 X2.
  if (dist2 <= kLastTol) {
    if ((rc = times(R2, R1, d, kTriA | kTriB, R))) return rc;
    if ((rc = times(X1, X2, d, kTriA | kTriB, Rinv))) return rc;
    if (run) PSK_HIP_TRY(hipGetLastError());
    return 0;
  }
  if ((rc = times(Qa, X2, m, kTriB, Qb))) return rc;
  // pass 3: W = Qb^T Qb
  if ((rc = gram_of(Qb, Qa))) return rc;
  if ((rc = later_pass_chol(W, d, R3, X3, B0, B1, B2, part, flag, &dist3, ws, st)))
    return rc;
  ws.release(mk);
  // R = R3 R2 R1, R^{-1} = X1 X2 X3
  if ((rc = times(R2, R1, d, kTriA | kTriB, T))) return rc;
  if ((rc = times(R3, T, d, kTriA | kTriB, R))) return rc;
  if ((rc = times(X1, X2, d, kTriA | kTriB, T))) return rc;
  if ((rc = times(T, X3, d, kTriA | kTriB, Rinv))) return rc;
  if (run) PSK_HIP_TRY(hipGetLastError());
  return 0;
}

}  // namespace psk
