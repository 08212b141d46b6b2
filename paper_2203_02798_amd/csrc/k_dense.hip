// FP64 dense products on the gfx950 matrix cores (v_mfma_f64_16x16x4f64):
// a general row-major GEMM with optional transposes and K splitting, the
// Gram matrix of a dense A (upper tiles only, mirrored), and the fused
// product-and-row-norm of a dense A times B.
//
// Paper mapping (arXiv 2203.02798): Algorithm gram (row-partitioned Gram:
// private partial Grams of row blocks, then a reduction) becomes the K split
// of A^T*A over row blocks of A followed by a fixed-order reduction kernel;
// rmsqn ("memory efficient" squared row norms of A*B for dense A) becomes a
// GEMM whose epilogue squares and sums each output row, so A*B is never
// stored.
//
// One kernel template covers all three.  A workgroup is 4 wavefronts laid
// out WM x WN; each owns MB x NB blocks of 16 x 16 FP64 accumulators.  K
// advances 16 at a time through LDS tiles kept k-major (As[k][i], Bs[k][j]),
// with the next chunk prefetched into registers while the current one is
// multiplied.  FP32 inputs are widened to FP64 when staged.
#include <type_traits>

#include <algorithm>

#include "internal.hpp"

namespace psk {
namespace {

typedef double v4d __attribute__((ext_vector_type(4)));
constexpr int kBK = 16;

enum { EPI_PARTIAL = 0, EPI_ROWNORM = 1, EPI_DIRECT = 2 };

template <typename T, bool KMAJOR, int BX>
struct TileLoader {
  // Loads a kBK x BX k-major tile of a logical operand Op[k][x]:
  //   KMAJOR: Op[k][x] = P[k*ld + x] (rows of P are k)
  //   else:   Op[k][x] = P[x*ld + k] (rows of P are x)
  static constexpr int kPer = (kBK * BX) / 256;
  double v[kPer];
  __device__ __forceinline__ void load(const T *__restrict__ P, int64_t ld, int64_t x0,
                                       int64_t xlim, int64_t k0, int64_t klim) {
#pragma unroll
    for (int p = 0; p < kPer; ++p) {
      const int e = threadIdx.x + 256 * p;
      int kk, xx;
      if (KMAJOR) {
        kk = e / BX;
        xx = e % BX;
      } else {
        kk = e % kBK;
        xx = e / kBK;
      }
      const int64_t k = k0 + kk, x = x0 + xx;
      v[p] = (k < klim && x < xlim) ? (double)(KMAJOR ? P[k * ld + x] : P[x * ld + k])
                                    : 0.0;
    }
  }
  __device__ __forceinline__ void store(double (*S)[BX + 4]) const {
#pragma unroll
    for (int p = 0; p < kPer; ++p) {
      const int e = threadIdx.x + 256 * p;
      int kk, xx;
      if (KMAJOR) {
        kk = e / BX;
        xx = e % BX;
      } else {
        kk = e % kBK;
        xx = e / kBK;
      }
      S[kk][xx] = v[p];
    }
  }
};

// Tile scheduling: tile t of the (tiles_m x tiles_n [upper only]) grid,
// split ks.  Blocks are renumbered so one XCD gets consecutive tiles.
struct TileCoord {
  int mt, nt, ks;
};

__device__ __forceinline__ TileCoord tile_of(int tiles_m, int tiles_n, bool upper) {
  const int64_t nblk = (int64_t)gridDim.x;
  int64_t lin = blockIdx.x;
  if ((nblk & 7) == 0) lin = (lin & 7) * (nblk >> 3) + (lin >> 3);
  TileCoord c;
  if (!upper) {
    c.mt = (int)(lin % tiles_m);
    const int64_t rest = lin / tiles_m;
    c.nt = (int)(rest % tiles_n);
    c.ks = (int)(rest / tiles_n);
  } else {
    // upper-triangular tiles (mt <= nt) of a square grid, row-major order
    const int64_t nup = (int64_t)tiles_m * (tiles_m + 1) / 2;
    int64_t t = lin % nup;
    c.ks = (int)(lin / nup);
    int mt = 0;
    int64_t rowlen = tiles_m;
    while (t >= rowlen) {
      t -= rowlen;
      ++mt;
      --rowlen;
    }
    c.mt = mt;
    c.nt = mt + (int)t;
  }
  return c;
}

template <typename TA, typename TB, bool TRA, bool TRB, int WM, int WN, int MB, int NB,
          int EPI, bool UPPER>
__global__ __launch_bounds__(256, 2) void k_dgemm(
    int64_t M, int64_t N, int64_t K, const TA *__restrict__ A, int64_t lda,
    const TB *__restrict__ B, int64_t ldb, int tiles_m, int tiles_n, int64_t kper, int tri,
    double *__restrict__ out, int64_t ldo, double alpha, double beta) {
  constexpr int BM = WM * MB * 16;
  constexpr int BN = WN * NB * 16;
  __shared__ double As[kBK][BM + 4];
  __shared__ double Bs[kBK][BN + 4];

  const TileCoord tc = tile_of(tiles_m, tiles_n, UPPER);
  const int64_t m0 = (int64_t)tc.mt * BM;
  const int64_t n0 = (int64_t)tc.nt * BN;
  int64_t kb = (int64_t)tc.ks * kper;
  int64_t ke = kb + kper;
  if (ke > K) ke = K;
  // the zero part of a triangular operand is not walked
  if ((tri & kTriB) && ke > n0 + BN) ke = n0 + BN;
  if ((tri & kTriAT) && ke > m0 + BM) ke = m0 + BM;
  if ((tri & kTriA) && kb < m0) kb = m0;

  const int tid = threadIdx.x;
  const int wave = tid >> 6;
  const int lane = tid & 63;
  const int kq = lane >> 4;
  const int li = lane & 15;
  const int wm = wave / WN;
  const int wn = wave % WN;

  v4d acc[MB][NB];
#pragma unroll
  for (int a = 0; a < MB; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[a][b] = v4d{0.0, 0.0, 0.0, 0.0};

  // Op_A[i][k]: TRA -> A is K x M (A[k*lda+i]) which is k-major
  TileLoader<TA, TRA, BM> la;
  TileLoader<TB, !TRB, BN> lb;
  const int64_t nchunks = (ke > kb) ? ceil_div(ke - kb, kBK) : 0;
  if (nchunks > 0) {
    la.load(A, lda, m0, M, kb, ke);
    lb.load(B, ldb, n0, N, kb, ke);
  }
  for (int64_t c = 0; c < nchunks; ++c) {
    __syncthreads();
    la.store(As);
    lb.store(Bs);
    __syncthreads();
    if (c + 1 < nchunks) {
      const int64_t k1 = kb + (c + 1) * kBK;
      la.load(A, lda, m0, M, k1, ke);
      lb.load(B, ldb, n0, N, k1, ke);
    }
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      double av[MB], bv[NB];
#pragma unroll
      for (int a = 0; a < MB; ++a) av[a] = As[4 * s + kq][(wm * MB + a) * 16 + li];
#pragma unroll
      for (int b = 0; b < NB; ++b) bv[b] = Bs[4 * s + kq][(wn * NB + b) * 16 + li];
#pragma unroll
      for (int a = 0; a < MB; ++a)
#pragma unroll
        for (int b = 0; b < NB; ++b)
          acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[a], bv[b], acc[a][b], 0, 0, 0);
    }
  }

  if (EPI == EPI_DIRECT) {
    // no K split: out = alpha * acc + beta * out (beta == 0 ignores out)
#pragma unroll
    for (int a = 0; a < MB; ++a)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int64_t row = m0 + (wm * MB + a) * 16 + kq + 4 * e;
        if (row >= M) continue;
#pragma unroll
        for (int b = 0; b < NB; ++b) {
          const int64_t col = n0 + (wn * NB + b) * 16 + li;
          if (col < N) {
            double *po = out + row * ldo + col;
            *po = beta != 0.0 ? alpha * acc[a][b][e] + beta * *po : alpha * acc[a][b][e];
          }
        }
      }
  } else if (EPI == EPI_PARTIAL && UPPER) {
    // whole tiles, packed: [split][tile][BM][BN]
    const int64_t nup = (int64_t)tiles_m * (tiles_m + 1) / 2;
    const int64_t t = (int64_t)tc.mt * tiles_m - (int64_t)tc.mt * (tc.mt - 1) / 2 + tc.nt - tc.mt;
    double *o = out + ((int64_t)tc.ks * nup + t) * (BM * BN);
#pragma unroll
    for (int a = 0; a < MB; ++a)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int b = 0; b < NB; ++b)
          o[((wm * MB + a) * 16 + kq + 4 * e) * BN + (wn * NB + b) * 16 + li] = acc[a][b][e];
  } else if (EPI == EPI_PARTIAL) {
    double *o = out + (int64_t)tc.ks * M * ldo;
#pragma unroll
    for (int a = 0; a < MB; ++a)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int64_t row = m0 + (wm * MB + a) * 16 + kq + 4 * e;
        if (row >= M) continue;
#pragma unroll
        for (int b = 0; b < NB; ++b) {
          const int64_t col = n0 + (wn * NB + b) * 16 + li;
          if (col < N) o[row * ldo + col] = acc[a][b][e];
        }
      }
  } else {
    // squared row norms over this tile's columns: out[nt][row]
    __shared__ double red[WN][BM];
#pragma unroll
    for (int a = 0; a < MB; ++a)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        double s2 = 0.0;
#pragma unroll
        for (int b = 0; b < NB; ++b) s2 += acc[a][b][e] * acc[a][b][e];
#pragma unroll
        for (int off = 1; off < 16; off <<= 1) s2 += __shfl_xor(s2, off, 64);
        if (li == 0) red[wn][(wm * MB + a) * 16 + kq + 4 * e] = s2;
      }
    __syncthreads();
    for (int i = tid; i < BM; i += 256) {
      const int64_t row = m0 + i;
      if (row >= M) continue;
      double s2 = 0.0;
#pragma unroll
      for (int q = 0; q < WN; ++q) s2 += red[q][i];
      out[(int64_t)tc.nt * ldo + row] = s2;
    }
  }
}

// C = alpha * sum_s part[s] + beta * C; part is [splits][M][ldp]
__global__ __launch_bounds__(256) void k_splitk_reduce(
    const double *__restrict__ part, int64_t M, int64_t N, int64_t ldp, int splits,
    double alpha, double beta, double *__restrict__ C, int64_t ldc) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= M * N) return;
  const int64_t i = e / N, j = e % N;
  double acc = part[i * ldp + j];
  for (int s = 1; s < splits; ++s) acc += part[(int64_t)s * M * ldp + i * ldp + j];
  double v = alpha * acc;
  if (beta != 0.0) v += beta * C[i * ldc + j];
  C[i * ldc + j] = v;
}

// W = sum_s of the packed upper tiles (nup of them, BT x BT), s in order; both
// triangles written
template <int BT>
__global__ __launch_bounds__(256) void k_sym_reduce(const double *__restrict__ part, int64_t d,
                                                    int64_t nup, int T, int splits,
                                                    double *__restrict__ W) {
  int I = 0;
  int64_t t = blockIdx.y;
  while (t >= T - I) {
    t -= T - I;
    ++I;
  }
  const int J = I + (int)t;
  const int e = blockIdx.x * 256 + threadIdx.x;
  const int64_t i = (int64_t)I * BT + e / BT, j = (int64_t)J * BT + e % BT;
  if (i >= d || j >= d) return;
  const double *p = part + (int64_t)blockIdx.y * (BT * BT) + e;
  double acc = p[0];
#pragma unroll 4
  for (int s = 1; s < splits; ++s) acc += p[(int64_t)s * nup * (BT * BT)];
  W[i * d + j] = acc;
  if (I != J) W[j * d + i] = acc;
}

__global__ __launch_bounds__(256) void k_rownorm_reduce(const double *__restrict__ part,
                                                        int64_t n, int tiles,
                                                        double alpha, double beta,
                                                        double *__restrict__ x) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  double s = part[i];
  for (int t = 1; t < tiles; ++t) s += part[(int64_t)t * n + i];
  double v = alpha * s;
  if (beta != 0.0) v += beta * x[i];
  x[i] = v;
}

// K splits of a product with few tiles; from 512 tiles on none
int64_t pick_splits(int64_t tiles, int64_t K, int64_t target_blocks) {
  if (tiles >= 512) return 1;
  const int64_t kchunks = ceil_div(K, kBK);
  int64_t s = ceil_div(target_blocks, tiles);
  int64_t smax = kchunks / 16;
  if (smax < 1) smax = 1;
  if (s > smax) s = smax;
  return s < 1 ? 1 : s;
}

template <bool TRA, bool TRB, int MB, int NB>
int gemm_launch(int64_t M, int64_t N, int64_t K, const double *A, int64_t lda, const double *B,
                int64_t ldb, double alpha, double beta, double *C, int64_t ldc, int tri, Arena &ws,
                hipStream_t st) {
  constexpr int BM = 32 * MB, BN = 32 * NB;
  const int tm = (int)ceil_div(M, BM), tn = (int)ceil_div(N, BN);
  const int64_t tiles = (int64_t)tm * tn;
  int64_t splits = pick_splits(tiles, K, 1024);
  const int64_t kper = ceil_div(ceil_div(K, kBK), splits) * kBK;
  splits = K > 0 ? ceil_div(K, kper) : 1;
  if (splits == 1) {
    if (ws.dry()) return 0;
    k_dgemm<double, double, TRA, TRB, 2, 2, MB, NB, EPI_DIRECT, false>
        <<<(unsigned)tiles, 256, 0, st>>>(M, N, K, A, lda, B, ldb, tm, tn, kper, tri, C, ldc,
                                          alpha, beta);
    PSK_HIP_TRY(hipGetLastError());
    return 0;
  }
  double *part = ws.take<double>((size_t)splits * M * N);
  if (ws.dry()) return 0;
  if (!ws.ok()) return fail(PSK_ENOMEM, "workspace too small for a GEMM");
  k_dgemm<double, double, TRA, TRB, 2, 2, MB, NB, EPI_PARTIAL, false>
      <<<(unsigned)(tiles * splits), 256, 0, st>>>(M, N, K, A, lda, B, ldb, tm, tn, kper, tri,
                                                   part, N, 1.0, 0.0);
  k_splitk_reduce<<<(unsigned)ceil_div(M * N, 256), 256, 0, st>>>(part, M, N, N, (int)splits,
                                                                  alpha, beta, C, ldc);
  PSK_HIP_TRY(hipGetLastError());
  return 0;
}

// Groups of four consecutive elements of a row, 16 apart, in 16-byte loads
// that need no more than the element's own alignment, as loaded (raw, in the
// dtype of A: widened when used, so the loads stay in flight meanwhile).
template <typename TA, int KW>
__device__ __forceinline__ void row_load(const TA *p, TA (&x)[KW]) {
  constexpr int VE = 16 / sizeof(TA);
  typedef TA vec __attribute__((ext_vector_type(VE), aligned(sizeof(TA))));
#pragma unroll
  for (int s = 0; s < KW; s += VE) {
    const vec v = *reinterpret_cast<const vec *>(p + 16 * (s / 4) + s % 4);
#pragma unroll
    for (int e = 0; e < VE; ++e) x[s + e] = v[e];
  }
}

// Fused row norms with a column tile of B resident in LDS.  A workgroup
// works on tiles p and T - 1 - p of the T = ceil(k / 32) 32-column tiles of B
// (one when they coincide): both at once when they fit in LDS (PAIR true),
// else one after the other, or on one tile only (tn = T) where that ends
// sooner.  Its B columns (rows padded to a multiple of the K chunk with zeros,
// row stride BNC + 4) are staged; the 8 wavefronts then stream
// row tiles of A (kBresMB blocks of 16 rows) straight from memory into the
// MFMA operand registers (no LDS round trip and no barrier in the main loop)
// and keep kBresMB x BNC/16 accumulator blocks.
// While staging, the workgroup finds each tile's row extent: one past the
// last row of B holding a nonzero in the tile's columns.  K chunks at or past
// a tile's extent only add exact zeros to its products, so they are skipped:
// for B = R^{-1} upper triangular, tile t needs its first 32 (t + 1) rows,
// and pairing tile t with tile T - 1 - t gives every workgroup the same
// work.  (Skipped products are a * 0 with a finite: the sums are the same
// bits as the full product's.)
// What bounds it: the FP64 matrix cores and the vector instructions between
// their products, which do not run beside them (about 64 + 4 v cycles for a
// product and v vector instructions).  So a chunk inside d is loaded in
// vector loads of whatever alignment the rows have and multiplied unmasked;
// RAG holds the code for the last chunk of a d that is not a multiple of 32
// (without it 1e6 x 256 takes 1226 us, with it 1278).  The first chunk of a
// phase or row tile is loaded while the one before it is multiplied.  Two
// wavefronts per SIMD: with three (168 registers each) the paired form spilled
// 30 to 130 of them (FP64 1e6 x 256: 1815 us at three, 1263 at two).
// Measured in us, before (masked element loads, three wavefronts, single
// tiles unpaired) and now: FP64 20,000 x 50 36 -> 18, 300,007 x 97 253 ->
// 134, 1e6 x 128 738 -> 427, 1e6 x 256 2696 -> 1214, 200,000 x 500 3175 ->
// 1032; FP32 1e6 x 128 383 -> 349, 4e6 x 256 4769 -> 4563 (2.9e11 flops: 62
// TF/s of the 76 that bare products reach).
// Inside a K chunk of 32 columns, lane (li, kq) feeds column k0 + 16 (s / 4) +
// 4 kq + s % 4 of A at step s = 0 .. 7, and that row of B: the same permutation
// of the chunk on both operands.  A lane reads four consecutive elements at a
// time and the four lanes of a row 16 in a row, so a load touches a cache line
// a row, and the chunk's first 16 rows are steps 0 .. 3 (with eight
// consecutive elements a lane it touched four lines, and a diagonal chunk
// needed lane halves swapped: 300,007 x 97 140 us, now 134; 200,000 x 256 in
// FP64 269, now 260).
// The diagonal 32 x 32 block of a triangular B is half zeros.  When the
// staging finds the lower-left 16 x 16 quarter of a tile's diagonal block
// zero (its rows 16 .. 31 in the tile's first 16 columns) and that block is
// the tile's last chunk (and inside the d columns), the products of the tile's
// first column block skip steps 4 .. 7, which are that chunk's last 16 rows.
// part[slot * n + row] = the row's squared norm over the slot's columns.
// Workgroups form row groups of tn (one per slot) that sit on one XCD
// (linear ids equal mod 8) and walk the same rows, so A is fetched into that
// XCD's L2 about once for all tn slots.
constexpr int kBresThreads = 512;  // 8 wavefronts: two per SIMD
constexpr int kBresWaves = kBresThreads / 64;
constexpr int kBresMB = 2;  // 16-row blocks per wavefront tile
constexpr int kBresRows = 16 * kBresMB;
constexpr int kBresKW = 8;
constexpr int kBresTile = 32;  // columns of B per tile

template <typename TA, bool PAIR, bool RAG>
__global__ __launch_bounds__(kBresThreads) void k_rownorm_bres(
    const TA *__restrict__ A, int64_t ld, int64_t n, int64_t d, const double *__restrict__ B,
    int64_t k, int tn, double *__restrict__ part) {
  extern __shared__ double Bs[];
  __shared__ int ext[2];
  __shared__ int nzq[2];  // a nonzero in the lower-left quarter of the tile's diagonal block
  constexpr int BNC = PAIR ? 2 * kBresTile : kBresTile;
  constexpr int LDB = BNC + 4;
  constexpr int NB = BNC / 16;
  constexpr int NBH = kBresTile / 16;  // blocks per tile
  constexpr int MB = kBresMB;
  constexpr int KW = kBresKW;  // consecutive elements of a row per lane per chunk
  constexpr int CK = 4 * KW;   // K chunk width
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int li = lane & 15, kq = lane >> 4;
  const int64_t lin = blockIdx.x, nblk = gridDim.x;
  const int64_t slot = lin >> 3;
  const int nt = (int)(slot % tn);
  const int64_t ngroups = nblk / tn;
  const int64_t group = (slot / tn) * 8 + (lin & 7);
  const int64_t ntile = ceil_div(k, (int64_t)kBresTile);
  const int64_t kch = (d + CK - 1) / CK;
  const int64_t drows = kch * CK;
  const int64_t ntiles = (n + kBresRows - 1) / kBresRows;
  const int64_t t0 = wave * ngroups + group, tstep = ngroups * kBresWaves;
  for (int pass = 0; pass < (PAIR || tn == ntile ? 1 : 2); ++pass) {
    const int64_t ta = pass ? ntile - 1 - nt : nt;  // the tile, or the first of the two
    if (pass) {
      if (ta == nt) break;
      __syncthreads();  // the first pass is done with the LDS tile
    }
    // first columns of the (one or two) tiles; -1: no second tile
    const int64_t c0a = ta * kBresTile;
    const int64_t tb = PAIR ? ntile - 1 - nt : -1;
    const int64_t c0b = (PAIR && tb != nt) ? tb * kBresTile : -1;
    if (tid < 2) {
      ext[tid] = 0;
      nzq[tid] = 0;
    }
    __syncthreads();
    int exa = 0, exb = 0;
    bool qa = false, qb = false;
    // four loads at once (clamped address, then a select): one after another
    // they would cost a memory latency each
    for (int64_t e0 = tid; e0 < drows * BNC; e0 += 4 * kBresThreads) {
      double bv[4];
      bool in[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int64_t e = e0 + u * kBresThreads;
        const int64_t kk = e / BNC;
        const int jj = (int)(e - kk * BNC);
        const int64_t cb = jj >= kBresTile ? c0b : c0a;
        const int64_t col = cb + (jj & (kBresTile - 1));
        in[u] = cb >= 0 && kk < d && col < k;
        bv[u] = B[in[u] ? kk * k + col : 0];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int64_t e = e0 + u * kBresThreads;
        if (e >= drows * BNC) break;
        const int64_t kk = e / BNC;
        const int jj = (int)(e - kk * BNC);
        const bool hb = jj >= kBresTile;
        const int64_t cb = hb ? c0b : c0a;
        const int jt = jj & (kBresTile - 1);
        const double v = in[u] ? bv[u] : 0.0;
        Bs[kk * LDB + jj] = v;
        if (v != 0.0) {  // NaN counts as nonzero
          const bool quarter = jt < 16 && kk >= cb + 16 && kk < cb + kBresTile;
          if (hb) {
            exb = (int)kk + 1;
            qb = qb || quarter;
          } else {
            exa = (int)kk + 1;
            qa = qa || quarter;
          }
        }
      }
    }
    if (exa) atomicMax(&ext[0], exa);
    if (exb) atomicMax(&ext[1], exb);
    if (qa) atomicOr(&nzq[0], 1);
    if (qb) atomicOr(&nzq[1], 1);
    __syncthreads();
    // K chunks each tile needs (uniform over the workgroup)
    const int64_t kca = __builtin_amdgcn_readfirstlane((ext[0] + CK - 1) / CK);
    const int64_t kcb = __builtin_amdgcn_readfirstlane((ext[1] + CK - 1) / CK);
    // the diagonal chunk of each tile (chunk index = tile index, a chunk
    // spanning one tile's rows) when its quarter is zero and its columns of A
    // are inside d; -1: none
    static_assert(CK == kBresTile, "a K chunk spans one tile's rows");
    const int64_t dga =
        (__builtin_amdgcn_readfirstlane(nzq[0]) || c0a + kBresTile > d) ? -1 : ta;
    const int64_t dgb =
        (c0b < 0 || __builtin_amdgcn_readfirstlane(nzq[1]) || c0b + kBresTile > d) ? -1 : tb;
    // The chunks of a row tile, in the order they are taken: the phase that
    // feeds both tiles (HM 3; the only one of a single tile is HM 1), then the
    // rest of the tile with the larger extent (HM 1 or 2).  A phase's last chunk
    // comes first when it is a special one: the diagonal chunk of the phase's
    // tile (of its first tile in HM 3), or the ragged end of d (never a
    // diagonal chunk: those are inside d).
    const int64_t kone = PAIR && kcb < kca ? kcb : kca;  // end of the first phase
    const int64_t k1 = PAIR ? kone : kca;
    const int64_t k2 = PAIR ? (kca > kcb ? kca : kcb) : k1;
    const bool hb2 = PAIR && kcb > kca;  // the second phase is the second tile's
    const bool dg1 = k1 > 0 && k1 - 1 == dga;
    const bool dg2 = k2 > k1 && k2 - 1 == (hb2 ? dgb : dga);
    const bool sp1 = dg1 || (RAG && k1 * CK > d), sp2 = dg2 || (RAG && k2 * CK > d);
    const int64_t f1 = sp1 ? k1 - 1 : 0, f2 = sp2 ? k2 - 1 : k1;  // first chunk of each phase
    const int64_t ffirst = k1 > 0 ? f1 : f2;
    // KW elements of each of the lane's rows, as loaded: a whole chunk in
    // vector loads; of the ragged chunk the columns inside d (the others read
    // the row's first element or four and are masked when used).  A row past n reads
    // row 0 and feeds only its own outputs, which are not stored.
    typedef TA RawChunk[MB][KW];
    auto load_whole = [&](const TA *const (&row)[MB], int64_t c, RawChunk &a)
                          __attribute__((always_inline)) {
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) row_load<TA, KW>(row[mb] + c * CK, a[mb]);
    };
    auto load = [&](const TA *const (&row)[MB], int64_t c, RawChunk &a)
                    __attribute__((always_inline)) {
      if (!RAG || (c + 1) * CK <= d) {
        load_whole(row, c, a);
      } else {
        const int64_t left = d - (c * CK + 4 * kq);  // this lane's columns inside d
        // Groups of four are inside or past d as a whole where d is a multiple of
        // four (FP32, k = 16, element / vector loads: 300,000 x 28 51.5 / 46.2 us,
        // 300,000 x 100 80.7 / 78.5).
        if (d % 4 == 0) {
          typedef TA Four[4];
#pragma unroll
          for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int g = 0; g < KW / 4; ++g)
              row_load<TA, 4>(row[mb] + (16 * g < left ? c * CK + 16 * g : -(int64_t)(4 * kq)),
                              *reinterpret_cast<Four *>(&a[mb][4 * g]));
        } else {
#pragma unroll
          for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int s = 0; s < KW; ++s) {
              const int k = 16 * (s / 4) + s % 4;
              a[mb][s] = row[mb][k < left ? c * CK + k : -(int64_t)(4 * kq)];
            }
        }
      }
    };
    auto rows_of = [&](int64_t t, const TA *(&row)[MB]) __attribute__((always_inline)) {
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) {
        const int64_t r = t * kBresRows + mb * 16 + li;
        row[mb] = A + (r < n ? r : 0) * ld + 4 * kq;
      }
    };
    // a0: the chunk taken next, loading since the one before it was multiplied
    // (across phases and row tiles)
    RawChunk a0, a1;
    const TA *arow[MB], *nrow[MB];
    rows_of(t0 < ntiles ? t0 : 0, arow);
    if (k2 > 0) load(arow, ffirst, a0);
    for (int64_t t = t0; t < ntiles; t += tstep) {
      const int64_t r0 = t * kBresRows;
      rows_of(t + tstep < ntiles ? t + tstep : t, nrow);
      v4d acc[MB][NB];
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) acc[mb][nb] = v4d{0.0, 0.0, 0.0, 0.0};
      using D0 = std::integral_constant<int, 0>;
      // one K chunk for the blocks of the tiles in HM (bit 0: first tile,
      // bit 1: second tile); DG 1 / 2: a diagonal chunk, the first
      // column block of the first / second tile skipping steps 4 .. 7
      auto step = [&](auto hm, auto dg, int64_t c, const RawChunk &raw)
                      __attribute__((always_inline)) {
        constexpr int HM = decltype(hm)::value;
        constexpr int DG = decltype(dg)::value;
        double a[MB][KW];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
          for (int s = 0; s < KW; ++s) a[mb][s] = (double)raw[mb][s];
#pragma unroll
        for (int s = 0; s < KW; ++s) {
          const int64_t kr = c * CK + 16 * (s / 4) + 4 * kq + s % 4;
          const double *brow = Bs + kr * LDB + li;
          auto on = [&](int nb) {
            return ((HM >> (nb / NBH)) & 1) && !(DG && s >= 4 && nb == (DG - 1) * NBH);
          };
          double bv[NB];
#pragma unroll
          for (int nb = 0; nb < NB; ++nb)
            if (on(nb)) bv[nb] = brow[nb * 16];
#pragma unroll
          for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
              if (on(nb))
                acc[mb][nb] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[mb][s], bv[nb], acc[mb][nb],
                                                                   0, 0, 0);
        }
      };
      // chunks c0 .. c1 - 1, the next chunk's A loaded while one is multiplied:
      // unconditional loads, so that with the same loads in flight on every path
      // a step waits for its own chunk only, not for the one loading behind it.
      // After the last comes chunk cn of the rows in rn.
      auto run = [&](auto hm, bool dg, bool special, int64_t c0, int64_t c1,
                     const TA *const (&rn)[MB], int64_t cn) __attribute__((always_inline)) {
        constexpr int HM = decltype(hm)::value;
        using DGT = std::integral_constant<int, HM == 2 ? 2 : 1>;
        if (c0 >= c1) return;
        int64_t ce = c1;
        if (special) {
          --ce;
          if (c0 < ce) load_whole(arow, c0, a1);
          else load(rn, cn, a1);
          if (!RAG || dg) {
            step(hm, DGT{}, ce, a0);
          } else {
            const int64_t left = d - (ce * CK + 4 * kq);
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
              for (int s = 0; s < KW; ++s)
                a0[mb][s] = 16 * (s / 4) + s % 4 < left ? a0[mb][s] : (TA)0;
            step(hm, D0{}, ce, a0);
          }
#pragma unroll
          for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int s = 0; s < KW; ++s) a0[mb][s] = a1[mb][s];
        }
        int64_t c = c0;
        for (; c + 2 < ce; c += 2) {
          load_whole(arow, c + 1, a1);
          __builtin_amdgcn_sched_barrier(0);  // keep the next chunk's loads ahead of this step
          step(hm, D0{}, c, a0);
          load_whole(arow, c + 2, a0);
          __builtin_amdgcn_sched_barrier(0);
          step(hm, D0{}, c + 1, a1);
        }
        if (c >= ce) return;
        if (c + 1 < ce) {
          load_whole(arow, c + 1, a1);
          __builtin_amdgcn_sched_barrier(0);
          step(hm, D0{}, c, a0);
          load(rn, cn, a0);
          __builtin_amdgcn_sched_barrier(0);
          step(hm, D0{}, c + 1, a1);
        } else {
          load(rn, cn, a1);
          __builtin_amdgcn_sched_barrier(0);
          step(hm, D0{}, c, a0);
#pragma unroll
          for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int s = 0; s < KW; ++s) a0[mb][s] = a1[mb][s];
        }
      };
      using HBoth = std::integral_constant<int, 3>;
      using HA = std::integral_constant<int, 1>;
      using HB = std::integral_constant<int, 2>;
      if constexpr (PAIR) {
        const bool two = k2 > k1;
        const TA *prow[MB];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) prow[mb] = two ? arow[mb] : nrow[mb];
        run(HBoth{}, dg1, sp1, 0, k1, prow, two ? f2 : ffirst);
        if (two && !hb2) run(HA{}, dg2, sp2, k1, k2, nrow, ffirst);
        if (two && hb2) run(HB{}, dg2, sp2, k1, k2, nrow, ffirst);
      } else {
        run(HA{}, dg1, sp1, 0, k1, nrow, ffirst);
      }
      // lane (li, kq) holds rows kq + 4 e, column li of each 16 x 16 block
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          double s2 = 0.0;
#pragma unroll
          for (int nb = 0; nb < NB; ++nb) s2 += acc[mb][nb][e] * acc[mb][nb][e];
#pragma unroll
          for (int off = 1; off < 16; off <<= 1) s2 += __shfl_xor(s2, off, 64);
          const int64_t row = r0 + mb * 16 + kq + 4 * e;
          if (li == 0 && row < n) part[(PAIR ? nt : ta) * n + row] = s2;
        }
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) arow[mb] = nrow[mb];
    }
  }
}

// LDS-resident form for d: 2 paired tiles (64 columns) when k > 32 and they
// fit, else 1 tile of 32 columns; 0: the tile does not fit.
int bres_width(int64_t d, int64_t k) {
  const int64_t drows = ceil_div(d, (int64_t)(4 * kBresKW)) * (4 * kBresKW);
  if (k > kBresTile && drows * (2 * kBresTile + 4) * 8 <= 163840) return 2;
  if (drows * (kBresTile + 4) * 8 <= 163840) return 1;
  return 0;
}

// Row groups of tn workgroups: one workgroup per CU (the LDS tile), so that each
// XCD holds whole groups.
int64_t bres_groups(int64_t n, int tn) {
  const int64_t tiles = ceil_div(n, (int64_t)kBresRows);
  int64_t groups = 256 / tn;
  if (groups < 8) groups = 8;
  groups = (groups / 8) * 8;
  const int64_t need = ceil_div(tiles, (int64_t)kBresWaves);  // row tiles per wavefront round
  // fewer groups for few rows, still whole eights (the kernel deals groups to
  // XCDs by linear id mod 8; 80 halved to 20 or 10 left rows without a group)
  while (groups > 8 && groups / 16 * 8 >= need) groups = groups / 16 * 8;
  return groups;
}

// Workgroups per row group, single tiles (bw 1): a workgroup takes two tiles in
// turn, T / 2 workgroups a group, or one, T a group and so fewer groups.  The
// costs compared are rounds of row tiles times the tiles' extents: two tiles of a
// B with fewer columns than rows are two whole ones, those of a square B are
// taken for a triangular one's, which together are one and a little (T + 1) / T.
// Few rows leave CUs idle when paired (FP64, k = 64, two / one in us: 3000 x 320
// 75.8 / 49.7, 30,000 x 320 80.0 / 52.7), many are the same either way (100,000 x
// 320: 125.9).
int bres_single_tn(int64_t n, int64_t d, int64_t k) {
  const int64_t ntile = ceil_div(k, (int64_t)kBresTile);
  const int pair = (int)ceil_div(ntile, (int64_t)2);
  const int64_t tiles = ceil_div(n, (int64_t)kBresRows);
  auto rounds = [&](int tn) { return ceil_div(tiles, bres_groups(n, tn) * kBresWaves); };
  const int64_t two = rounds(pair) * (k < d ? 2 * ntile : ntile + 1);
  return rounds((int)ntile) * ntile < two ? (int)ntile : pair;
}

template <typename TA, bool PAIR, bool RAG>
int bres_launch_as(const psk_mat &Am, const double *B, int64_t k, double *part, int tn,
                hipStream_t st) {
  const int64_t n = Am.n, d = Am.d;
  constexpr int BNC = PAIR ? 2 * kBresTile : kBresTile;
  const size_t lds =
      (size_t)ceil_div(d, (int64_t)(4 * kBresKW)) * (4 * kBresKW) * (BNC + 4) * sizeof(double);
  PSK_HIP_TRY(hipFuncSetAttribute((const void *)k_rownorm_bres<TA, PAIR, RAG>,
                                  hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  const unsigned nblk = (unsigned)(bres_groups(n, tn) * tn);
  KTimer timer("rownorm", st);
  k_rownorm_bres<TA, PAIR, RAG><<<nblk, kBresThreads, lds, st>>>(
      (const TA *)Am.values, Am.ld, n, d, B, k, tn, part);
  return 0;
}

template <typename TA, bool PAIR>
int bres_launch(const psk_mat &Am, const double *B, int64_t k, double *part, int tn,
                hipStream_t st) {
  return Am.d % (4 * kBresKW) ? bres_launch_as<TA, PAIR, true>(Am, B, k, part, tn, st)
                              : bres_launch_as<TA, PAIR, false>(Am, B, k, part, tn, st);
}

template <typename TA>
int rownorm_launch(const psk_mat &Am, const double *B, int64_t k, double alpha,
                   double beta, double *x, Arena &ws, hipStream_t st) {
  const int64_t n = Am.n, d = Am.d;
  const TA *A = (const TA *)Am.values;
  const int bw = bres_width(d, k);
  if (bw > 0) {
    // a workgroup's two 32-column tiles give one sum per row together (bw 2,
    // both in LDS at once) or one each (bw 1, one after the other)
    const int64_t ntile = ceil_div(k, (int64_t)kBresTile);
    const int tn = bw == 2 ? (int)ceil_div(ntile, (int64_t)2) : bres_single_tn(n, d, k);
    const int slots = bw == 2 ? tn : (int)ntile;  // sums per row
    double *part = ws.take<double>((size_t)slots * n);
    if (ws.dry()) return 0;
    if (!ws.ok()) return fail(PSK_ENOMEM, "workspace too small for row norms");
    const int rc = bw == 2 ? bres_launch<TA, true>(Am, B, k, part, tn, st)
                           : bres_launch<TA, false>(Am, B, k, part, tn, st);
    if (rc) return rc;
    k_rownorm_reduce<<<(unsigned)ceil_div(n, 256), 256, 0, st>>>(part, n, slots, alpha, beta, x);
  } else if (k <= 64) {
    constexpr int BM = 32, BN = 64;
    const int tm = (int)ceil_div(n, BM), tn = (int)ceil_div(k, BN);
    double *part = ws.take<double>((size_t)tn * n);
    if (ws.dry()) return 0;
    if (!ws.ok()) return fail(PSK_ENOMEM, "workspace too small for row norms");
    {
      KTimer timer("rownorm", st);
      k_dgemm<TA, double, false, false, 2, 2, 1, 2, EPI_ROWNORM, false>
          <<<(unsigned)((int64_t)tm * tn), 256, 0, st>>>(n, k, d, A, Am.ld, B, k, tm, tn, d,
                                                         0, part, n, 1.0, 0.0);
    }
    k_rownorm_reduce<<<(unsigned)ceil_div(n, 256), 256, 0, st>>>(part, n, tn, alpha,
                                                                  beta, x);
  } else {
    constexpr int BM = 32, BN = 256;
    const int tm = (int)ceil_div(n, BM), tn = (int)ceil_div(k, BN);
    double *part = ws.take<double>((size_t)tn * n);
    if (ws.dry()) return 0;
    if (!ws.ok()) return fail(PSK_ENOMEM, "workspace too small for row norms");
    {
      KTimer timer("rownorm", st);
      k_dgemm<TA, double, false, false, 2, 2, 1, 8, EPI_ROWNORM, false>
          <<<(unsigned)((int64_t)tm * tn), 256, 0, st>>>(n, k, d, A, Am.ld, B, k, tm, tn, d,
                                                         0, part, n, 1.0, 0.0);
    }
    k_rownorm_reduce<<<(unsigned)ceil_div(n, 256), 256, 0, st>>>(part, n, tn, alpha,
                                                                  beta, x);
  }
  PSK_HIP_TRY(hipGetLastError());
  return 0;
}


// ---------------------------------------------------------------------------
// Gram matrix of a dense tall A: C = A^T A as a sum over row slabs
// ---------------------------------------------------------------------------
// A work item is one 64 x 64 tile (I, J), I <= J, of the upper block triangle
// of C and one slab of consecutive rows of A.  WPT wavefronts share it, each
// accumulating every WPT-th group of the slab's rows in registers (4 x 4
// blocks of 16 x 16 FP64 accumulators); with four (a whole workgroup) the
// sums are added in LDS, in wavefront order, before the tile is written.
// Lane (li, kq) = (lane % 16, lane / 16) reads, of row k0 + kq, element li of
// each 16-column block.  On a diagonal tile (I = J) only the
// blocks a <= b are multiplied (10 of 16).  The last tile of a d that is not
// a multiple of 64 has fewer blocks (NBT of 4): the blocks past d are neither
// read nor multiplied (d = 97: 28 blocks a step, not 36).
// What bounds it: the FP64 matrix cores and next to them every vector
// instruction, since the two do not run side by side (a 16 x 16 x 4 product
// takes 64 cycles, each vector instruction about 4 more).  So the loop holds
// little else than loads, FP32 conversions and products: addresses are one
// addition per row and side, columns past d are clamped to column d - 1 (they
// reach only outputs past d, which nobody reads) and rows are counted, so no
// element is masked except in a slab's last rows; and two wavefronts per SIMD
// are stated to the compiler, which then keeps the accumulators where the
// products use them (without it they moved between the two register files on
// every step).
// Past that it waits for its rows in the vector L1 (FP64 1e6 x 256: 55 TF/s
// whatever the instruction count, before the wavefronts kept step; FP32, half
// the bytes: 65).
// Two arrangements.  WPT = 4, d <= 112 and many rows: as above, a partial per
// workgroup; narrow products are short of work, and the fewer partials matter
// most.  WPT = 1, wider or few rows: every wavefront has a tile and a slab of
// its own and writes its own partial, so that the workgroup's wavefronts, mostly tiles of
// one slab, find each other's rows in the L1; a barrier every group of rows
// keeps the off-diagonal ones in step, without which they drift apart and
// find nothing (us, without / with: FP64 1e6 x 256 1267 / 1190, 200,000 x 500
// 913 / 865; FP32 1e6 x 256 1076 / 1025, 300,000 x 200 302 / 274).  Measured
// in us, before / one wavefront, out of step / four: FP64 300,000 x 64: 91 /
// 55 / 48, 300,007 x 97: 162 / 116 / 97, 1e6 x 128: 456 / 416 / 547, 1e6 x
// 256: 1290 / 1266 / 1728; FP32 1e6 x 128: 390 / 306 / 309, 1e6 x 256: 1255 /
// 1076 / 1104.  Before, the loads were masked element by element, the
// accumulators moved every step and a small A was cut into 2048 partials
// whatever its size (20,000 x 50: 34 us with its reduction, now 21; 20,000 x
// 256: 111, now 46).
// Work items: the classes of tiles (off-diagonal, off-diagonal in the last
// tile column, diagonal, last diagonal) take 16, 4 NBT, 10 and
// NBT (NBT + 1) / 2 block products a row step, and each class gets slabs in
// proportion, so that every item costs about the same and all of them run in
// one round, two wavefronts per SIMD.  Slab-major order inside a class, and
// workgroups of one XCD (linear ids equal mod 8) take consecutive items: the
// tiles of one slab read its rows through one L2.  No atomics.
constexpr int kGramWaves = 4;
// Row steps whose loads are in flight: six where a wavefront has its item to
// itself (FP64 300,000 x 129: 239 us at four, 206 at six; 244 registers, 252
// with FP32 rows, so kernels of another stream run before and after it rather
// than beside it: 4e6 x 256 in FP32 with its sketch on a second stream takes
// 10.50 ms a step, 10.59 on one stream; 11.05 and 11.98 while it held 208 and
// ran slower), four where the workgroup shares it and the rows are few (20,000
// x 97: 25 us at four, 30 at six).
constexpr int gram_prefetch(int wpt) { return wpt == 1 ? 6 : 4; }
constexpr int kGramLds = 64 + 16;  // row stride of the LDS sum: rows kq and kq + 1 in other banks

// The four tile classes of a T-tile-wide upper triangle: count of tiles and
// slabs of each, in item order.
struct GramPlan {
  int T;        // tiles across
  int nbt;      // 16-column blocks of the last tile
  int cnt[4];   // tiles: off-diagonal, off-diagonal last column, diagonal, last diagonal
  int slabs[4];
  int64_t rows[4];   // rows of a slab
  int64_t first[5];  // first item of each class; [4]: items in all
};

// class of tile (I, J) and its index in the class
__device__ __forceinline__ int gram_class(const GramPlan &p, int I, int J, int &idx) {
  const bool tail = p.cnt[3] != 0 && J == p.T - 1;
  if (I == J) {
    idx = tail ? 0 : I;
    return tail ? 3 : 2;
  }
  idx = tail ? I : J * (J - 1) / 2 + I;
  return tail ? 1 : 0;
}

// One wavefront's share of the rows [k0, k1) of a tile (every kGramWaves-th
// group of rows, the last rows to wavefront 0): NI x NJ blocks (DG: NI = NJ,
// the upper ones).  CLAMP: the tile is the last one of a ragged d, whose last
// block holds columns past d: they read column d - 1.
template <typename TA, int WPT, bool DG, bool CLAMP, int NI, int NJ>
__device__ __forceinline__ void gram_rows(const TA *__restrict__ A, int64_t ld, int64_t d,
                                          int64_t k0, int64_t k1, int wave, int I, int J,
                                          int64_t stepped, v4d (&acc)[4][4]) {
  constexpr bool kStepped = WPT == 1;
  constexpr int PF = gram_prefetch(WPT);
  const int lane = threadIdx.x & 63;
  const int li = lane & 15, kq = lane >> 4;
  const TA *pi = A + (int64_t)kq * ld + 64 * (int64_t)I + li;
  const TA *pj = A + (int64_t)kq * ld + 64 * (int64_t)J + li;
  // the last block of the J columns, relative to pj
  int64_t lastj = 16 * (NJ - 1);
  if (CLAMP) {
    const int64_t left = d - 1 - 64 * (int64_t)J - li;
    if (left < lastj) lastj = left;
  }
  auto load = [&](const TA *p, bool isj, int nb, TA (&x)[4]) __attribute__((always_inline)) {
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      if (b >= nb) continue;
      x[b] = CLAMP && isj && b == nb - 1 ? p[lastj] : p[16 * b];
    }
  };
  auto mul = [&](const TA (&xi)[4], const TA (&xj)[4]) __attribute__((always_inline)) {
    double av[4], bv[4];
#pragma unroll
    for (int a = 0; a < NI; ++a) av[a] = (double)xi[a];
#pragma unroll
    for (int b = 0; b < NJ; ++b) bv[b] = DG ? av[b] : (double)xj[b];
#pragma unroll
    for (int a = 0; a < NI; ++a)
#pragma unroll
      for (int b = 0; b < NJ; ++b)
        if (!DG || a <= b)
          acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[a], bv[b], acc[a][b], 0, 0, 0);
  };
  TA xi[PF][4], xj[PF][4];
  auto fetch = [&](int p, int64_t row) __attribute__((always_inline)) {
    load(pi + row * ld, DG, NI, xi[p]);
    if constexpr (!DG) load(pj + row * ld, true, NJ, xj[p]);
  };
  // this wavefront's groups of PF steps, WPT groups apart; the
  // loads past its last group repeat that group (in bounds, unused)
  constexpr int64_t kGroup = 4 * PF;
  const int64_t groups = (k1 - k0) / kGroup;
  if (wave < groups) {
#pragma unroll
    for (int p = 0; p < PF; ++p) fetch(p, k0 + kGroup * wave + 4 * p);
    for (int64_t g = wave; g < groups; g += WPT) {
      const int64_t next = k0 + kGroup * (g + WPT < groups ? g + WPT : g);
#pragma unroll
      for (int p = 0; p < PF; ++p) {
        TA ci[4], cj[4];
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          ci[b] = xi[p][b];
          cj[b] = xj[p][b];
        }
        mul(ci, cj);
        fetch(p, next + 4 * p);
      }
      if (kStepped && stepped) __builtin_amdgcn_s_barrier();
    }
  }
  // (a shorter slab waits out its fellows' groups: every wavefront meets the
  // barrier `stepped` times)
  if (kStepped)
    for (int64_t g = groups; g < stepped; ++g) __builtin_amdgcn_s_barrier();
  if (wave) return;
  // the rest (fewer than 4 PF rows, at the end of A only): rows past k1 as zero
  for (int64_t k = k0 + groups * kGroup; k < k1; k += 4) {
    const bool ok = k + kq < k1;
    const int64_t row = ok ? k : k1 - 1 - kq;  // relative to this lane's row kq
    fetch(0, row);
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      xi[0][b] = ok && b < NI ? xi[0][b] : (TA)0;
      if constexpr (!DG) xj[0][b] = ok && b < NJ ? xj[0][b] : (TA)0;
    }
    mul(xi[0], xj[0]);
  }
}

template <typename TA, int WPT>
__global__ __launch_bounds__(64 * kGramWaves, 2) void k_gram_syrk(const TA *__restrict__ A,
                                                                  int64_t ld, int64_t n,
                                                                  int64_t d, GramPlan pl,
                                                                  double *__restrict__ part) {
  static_assert(WPT == 1 || WPT == kGramWaves, "one wavefront or the workgroup per item");
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int li = lane & 15, kq = lane >> 4;
  const int64_t nblk = gridDim.x;
  int64_t g = blockIdx.x;
  if ((nblk & 7) == 0) g = (g & 7) * (nblk >> 3) + (g >> 3);
  if (WPT == 1) g = g * kGramWaves + wave;
  if (g >= pl.first[4]) return;
  int cls = 0;
  while (g >= pl.first[cls + 1]) ++cls;
  const int64_t local = g - pl.first[cls];
  const int64_t slab = local / pl.cnt[cls];
  const int idx = (int)(local - slab * pl.cnt[cls]);
  int I, J;
  if (cls == 0) {
    J = 1;
    while (J * (J + 1) / 2 <= idx) ++J;
    I = idx - J * (J - 1) / 2;
  } else {
    I = cls == 3 ? pl.T - 1 : idx;
    J = cls == 2 ? idx : pl.T - 1;
  }
  const int64_t k0 = slab * pl.rows[cls];
  int64_t k1 = k0 + pl.rows[cls];
  if (k1 > n) k1 = n;
  v4d acc[4][4];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[a][b] = v4d{0.0, 0.0, 0.0, 0.0};
  const int wt = WPT == 1 ? 0 : wave;  // wavefront of the item
  // The groups that the workgroup's wavefronts take in step, 0: none.  In step
  // where all four are tiles of one off-diagonal class, so that a step costs
  // them the same, and three or more of those share a slab: the first one's
  // slab is the longest.
  int64_t stepped = 0;
  const int64_t g0 = g - wave;
  if (WPT == 1 && cls < 2 && g0 >= pl.first[cls] && g0 + kGramWaves <= pl.first[cls + 1] &&
      pl.cnt[cls] >= 3) {
    const int64_t r0 = (g0 - pl.first[cls]) / pl.cnt[cls] * pl.rows[cls];
    stepped = (n - r0 < pl.rows[cls] ? n - r0 : pl.rows[cls]) / (4 * gram_prefetch(1));
  }
#define PSK_GR(DG, CL, NI, NJ) gram_rows<TA, WPT, DG, CL, NI, NJ>(A, ld, d, k0, k1, wt, I, J, stepped, acc)
  if (cls == 0) PSK_GR(false, false, 4, 4);
  else if (cls == 2) PSK_GR(true, false, 4, 4);
  else if (cls == 1) {
    if (pl.nbt == 4) PSK_GR(false, true, 4, 4);
    else if (pl.nbt == 3) PSK_GR(false, true, 4, 3);
    else if (pl.nbt == 2) PSK_GR(false, true, 4, 2);
    else PSK_GR(false, true, 4, 1);
  } else {
    if (pl.nbt == 4) PSK_GR(true, true, 4, 4);
    else if (pl.nbt == 3) PSK_GR(true, true, 3, 3);
    else if (pl.nbt == 2) PSK_GR(true, true, 2, 2);
    else PSK_GR(true, true, 1, 1);
  }
#undef PSK_GR
  // lane (li, kq) holds rows kq + 4 e, column li of each block; the blocks
  // not multiplied hold zeros and are not read from the sum
  double *o = part + g * 4096;
  if constexpr (WPT == 1) {
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int e = 0; e < 4; ++e) o[(16 * a + kq + 4 * e) * 64 + 16 * b + li] = acc[a][b][e];
  } else {
    __shared__ __align__(16) double sum[64][kGramLds];
#pragma unroll 1
    for (int w = 0; w < kGramWaves; ++w) {
      if (wave == w) {
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
          for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              double *s = &sum[16 * a + kq + 4 * e][16 * b + li];
              *s = w ? *s + acc[a][b][e] : acc[a][b][e];
            }
      }
      __syncthreads();
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int e = 2 * (threadIdx.x + 256 * q);
      *reinterpret_cast<double2 *>(o + e) =
          *reinterpret_cast<const double2 *>(&sum[e >> 6][e & 63]);
    }
  }
}

// C = alpha * sum over a tile's slabs + beta * C (beta == 0 ignores C): one
// workgroup per tile row of 64 columns, blockDim.y groups of slabs summed
// side by side (eight loads at once) and then in order.  The element (p, c),
// p <= c, of the tile also gives (c, p).
constexpr int kGramGroups = 16;

template <typename TO>
__global__ __launch_bounds__(64 * kGramGroups) void k_gram_reduce(
    const double *__restrict__ part, int64_t d, GramPlan pl, double alpha, double beta,
    TO *__restrict__ C) {
  __shared__ double sum[kGramGroups][64];
  const int x = threadIdx.x, y = threadIdx.y, ny = blockDim.y;
  const int row = blockIdx.x & 63, tile = blockIdx.x >> 6;
  int J = 0;
  while ((J + 1) * (J + 2) / 2 <= tile) ++J;
  const int I = tile - J * (J + 1) / 2;
  const int64_t p = 64 * (int64_t)I + row, c = 64 * (int64_t)J + x;
  if (p >= d) return;  // the whole workgroup
  int idx;
  const int cls = gram_class(pl, I, J, idx);
  const int64_t slabs = pl.slabs[cls], step = (int64_t)pl.cnt[cls] * 4096;
  const int64_t s0 = slabs * y / ny, s1 = slabs * (y + 1) / ny;
  const bool on = c < d && (I != J || row / 16 <= x / 16);
  double acc = 0.0;
  if (on) {
    const double *q = part + (pl.first[cls] + idx) * 4096 + row * 64 + x;
    int64_t s = s0;
    for (; s + 8 <= s1; s += 8) {
      double v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = q[(s + u) * step];
#pragma unroll
      for (int u = 0; u < 8; ++u) acc += v[u];
    }
    for (; s < s1; ++s) acc += q[s * step];
  }
  if (ny > 1) {
    sum[y][x] = acc;
    __syncthreads();
    if (y) return;
    for (int u = 1; u < ny; ++u) acc += sum[u][x];
  }
  if (!on || y) return;
  double v = alpha * acc;
  const int64_t e = p * d + c, m = c * d + p;
  // the mirrored element; inside a diagonal 16 x 16 block both are computed
  const bool mirror = I != J || row / 16 < x / 16;
  if (mirror) C[m] = (TO)(beta != 0.0 ? v + beta * (double)C[m] : v);
  if (beta != 0.0) v += beta * (double)C[e];
  C[e] = (TO)v;
}

// Wavefronts that share an item, for d <= 112 as said beside the kernel.  Up to
// 2000 rows such a product is a launch, a few groups of rows and the reduction,
// and summing four wavefronts in LDS is most of it (us, four / one: 100 x 64
// 34.8 / 29.9, 500 x 112 37.3 / 33.5).  Past that one is little faster (16,000 x
// 97 44.0 / 41.8) and holds 2.5 times the partials, which narrow requests in a
// small server pool would run fewer at once for (20,000 x 50 in 20 MB: 384 us
// each, not 143).  A lean workspace has no room for them at all.
int gram_wpt(int64_t n, int64_t d, bool lean) {
  return d <= 112 && (n > 2000 || lean) ? kGramWaves : 1;
}

GramPlan gram_plan(int64_t n, int64_t d, int wpt, bool f64, bool lean) {
  GramPlan p{};
  p.T = (int)ceil_div(d, (int64_t)64);
  p.nbt = (int)ceil_div(d - 64 * (int64_t)(p.T - 1), (int64_t)16);
  const bool tail = d % 64 != 0;
  const int F = tail ? p.T - 1 : p.T;  // full tiles across
  p.cnt[0] = F * (F - 1) / 2;
  p.cnt[1] = tail ? F : 0;
  p.cnt[2] = F;
  p.cnt[3] = tail ? 1 : 0;
  // a step costs its block products, or twice the blocks it loads where those
  // are more: a narrow last tile waits for its rows (300,000 x 200 in FP64,
  // whose last tile is one block wide: 605 us by products alone, 302 by this
  // rule).  The last diagonal tile of a wavefront of its own waits longest, its
  // loads are all it does: two more in FP64, one in FP32 past 256 columns
  // (without them 120,000 x 836 in FP64 took 2397 us, its last tile alone in two
  // slabs of 60,000 rows, now 1428; 200,000 x 452 1068 and 765, 300,000 x 220 375
  // and 323)
  const double nbt = p.nbt, wait = wpt > 1 ? 0.0 : f64 ? 2.0 : p.T > 4 ? 1.0 : 0.0;
  const double cost[4] = {16.0, std::max(4.0 * nbt, 2.0 * (4.0 + nbt)), 10.0,
                          std::max(0.5 * nbt * (nbt + 1.0), 2.0 * nbt + wait)};
  double total = 0.0;
  for (int c = 0; c < 4; ++c) total += p.cnt[c] * cost[c];
  // two wavefronts per SIMD in one round (a lean workspace: one), at least
  // two groups of rows each
  const int64_t kRound = 4 * gram_prefetch(wpt) * wpt;
  const double slots = (lean ? 256.0 : 512.0) * kGramWaves / wpt;
  for (int c = 0; c < 4; ++c) {
    if (!p.cnt[c]) continue;
    int64_t s = (int64_t)(slots * cost[c] / total);
    if (s < 2) s = 2;
    int64_t rows = ceil_div(ceil_div(n, s), kRound) * kRound;
    if (rows < 2 * kRound) rows = 2 * kRound;
    p.rows[c] = rows;
    p.slabs[c] = (int)ceil_div(n, rows);
    if (p.slabs[c] < 1) p.slabs[c] = 1;
  }
  for (int c = 0; c < 4; ++c)
    p.first[c + 1] = p.first[c] + (int64_t)p.cnt[c] * p.slabs[c];
  return p;
}

template <typename TA>
int gram_syrk_launch(double alpha, const psk_mat &Am, double beta, void *C, bool out_f32,
                     Arena &ws, hipStream_t st) {
  const int64_t n = Am.n, d = Am.d;
  const int wpt = gram_wpt(n, d, ws.lean);
  const GramPlan pl = gram_plan(n, d, wpt, sizeof(TA) == 8, ws.lean);
  const int64_t items = pl.first[4];
  double *part = ws.take<double>((size_t)items * 4096);
  if (ws.dry()) return 0;
  if (!ws.ok()) return fail(PSK_ENOMEM, "workspace too small for the Gram matrix");
  // whole XCD rounds for the remap
  const int64_t nblk = ceil_div(ceil_div(items * wpt, (int64_t)kGramWaves), (int64_t)8) * 8;
  {
    KTimer timer("gram", st);
    if (wpt == 1)
      k_gram_syrk<TA, 1><<<(unsigned)nblk, 64 * kGramWaves, 0, st>>>((const TA *)Am.values, Am.ld,
                                                                    n, d, pl, part);
    else
      k_gram_syrk<TA, kGramWaves><<<(unsigned)nblk, 64 * kGramWaves, 0, st>>>(
          (const TA *)Am.values, Am.ld, n, d, pl, part);
  }
  KTimer rtimer("gram_reduce", st);
  int most = 1, groups = 1;
  for (int c = 0; c < 4; ++c) most = pl.slabs[c] > most ? pl.slabs[c] : most;
  while (groups < kGramGroups && groups * 8 < most) groups *= 2;
  const unsigned rgrid = (unsigned)(pl.T * (pl.T + 1) / 2 * 64);
  if (out_f32)
    k_gram_reduce<float><<<rgrid, dim3(64, groups), 0, st>>>(part, d, pl, alpha, beta,
                                                             (float *)C);
  else
    k_gram_reduce<double><<<rgrid, dim3(64, groups), 0, st>>>(part, d, pl, alpha, beta,
                                                              (double *)C);
  PSK_HIP_TRY(hipGetLastError());
  return 0;
}

}  // namespace

int dgemm(bool ta, bool tb, int64_t M, int64_t N, int64_t K, double alpha,
          const double *A, int64_t lda, const double *B, int64_t ldb, double beta,
          double *C, int64_t ldc, Arena &ws, hipStream_t st, int tri) {
  if (M <= 0 || N <= 0) return 0;
  if (K <= 0) return fail(PSK_EINVAL, "internal GEMM with K <= 0");
  // up to 1024 x 1024 outputs (the d x d products of the factorizations),
  // 32 x 32 tiles give the chip four times the workgroups of 64 x 64 ones
#define PSK_DG(TRA, TRB)                                                                       \
  return (M * N <= 1024 * 1024)                                                                \
      ? gemm_launch<TRA, TRB, 1, 1>(M, N, K, A, lda, B, ldb, alpha, beta, C, ldc, tri, ws, st) \
      : gemm_launch<TRA, TRB, 2, 2>(M, N, K, A, lda, B, ldb, alpha, beta, C, ldc, tri, ws, st)
  if (ta && tb) PSK_DG(true, true);
  if (ta) PSK_DG(true, false);
  if (tb) PSK_DG(false, true);
  PSK_DG(false, false);
#undef PSK_DG
}

int dgram(const double *C, int64_t m, int64_t d, double *W, double *scratch, int64_t room,
          hipStream_t st) {
  // 64 x 64 tiles where they and their K splits (eight 16-row chunks or more
  // each) fill the chip, else 32 x 32 ones: a wavefront then has one block a
  // step, a quarter of the matrix work per operand read
  const int64_t kch = ceil_div(m, (int64_t)kBK);
  const int64_t smax = kch / 8 > 0 ? kch / 8 : 1;
  auto run = [&](auto mb) -> int {
    constexpr int MB = decltype(mb)::value, BT = 32 * MB;
    const int T = (int)ceil_div(d, (int64_t)BT);
    const int64_t nup = (int64_t)T * (T + 1) / 2;
    int64_t splits = 768 / nup;
    if (splits > smax) splits = smax;
    if (splits > room / (nup * BT * BT)) splits = room / (nup * BT * BT);
    if (splits < 1) splits = 1;
    const int64_t kper = ceil_div(kch, splits) * kBK;
    splits = ceil_div(m, kper);
    k_dgemm<double, double, true, false, 2, 2, MB, MB, EPI_PARTIAL, true>
        <<<(unsigned)(nup * splits), 256, 0, st>>>(d, d, m, C, d, C, d, T, T, kper, 0, scratch,
                                                   d, 1.0, 0.0);
    k_sym_reduce<BT><<<dim3(BT * BT / 256, (unsigned)nup), 256, 0, st>>>(scratch, d, nup, T,
                                                                        (int)splits, W);
    PSK_HIP_TRY(hipGetLastError());
    return 0;
  };
  const int64_t T64 = ceil_div(d, (int64_t)64), n64 = T64 * (T64 + 1) / 2;
  const bool wide = n64 * smax >= 256 && n64 * 4096 <= room;
  return wide ? run(std::integral_constant<int, 2>{}) : run(std::integral_constant<int, 1>{});
}

int64_t dgram_room(int64_t d) {
  const int64_t T = ceil_div(d, (int64_t)32);  // one split of whole 32 x 32 tiles
  return T * (T + 1) / 2 * 1024;
}

int gram_dense(double alpha, const psk_mat &A, double beta, void *C, Arena &ws,
               hipStream_t st, bool out_f64) {
  if (A.dtype == PSK_F32) return gram_syrk_launch<float>(alpha, A, beta, C, !out_f64, ws, st);
  return gram_syrk_launch<double>(alpha, A, beta, C, false, ws, st);
}

int rownorms_dense(double alpha, const psk_mat &A, const double *B, int64_t k,
                   double beta, double *x, Arena &ws, hipStream_t st) {
  if (A.dtype == PSK_F32) return rownorm_launch<float>(A, B, k, alpha, beta, x, ws, st);
  return rownorm_launch<double>(A, B, k, alpha, beta, x, ws, st);
}

}  // namespace psk
