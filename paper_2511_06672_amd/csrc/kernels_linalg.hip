// Dense FP64 complex linear algebra for the MPS factorisations (§2.4: truncation by SVD).
//
// * k_zgemm_s / k_zgemm: C = alpha op(A) op(B) on 16x16 or 32x32 tiles with v_mfma_f64_16x16x4 (a
//   complex product is four real MFMAs into a real and an imaginary accumulator).
// * Hermitian eigen-decomposition by two-sided Jacobi rotations: a single-workgroup kernel that
//   keeps the whole matrix in LDS (m <= kSmallEig) and a block-Jacobi scheme for larger m
//   (pairs of 16-blocks solved as 32x32 sub-problems in LDS, the rotations applied to the matrix
//   and the eigenvector accumulator as 32x32 MFMA tile products).
// * k_trunc: descending sort of squared singular values and the truncation rule.
// * k_emit: writes the two factors of a split in the requested orientation.
#include <cfloat>
#include <cstring>

#include "jacobi.h"
#include "kernels.h"

namespace gc {

namespace {

// ===================================================================================== GEMM
// Two forms: k_zgemm_s on 16 x 16 output tiles with operands straight from memory, and k_zgemm on 32 x 32 tiles
// staged through LDS for products of many tiles (launch_zgemm has the line).  In k_zgemm, K advances in chunks
// of 16; each chunk is fetched into registers while the previous one is multiplied, then stored into
// the other LDS stage (one barrier per chunk).  In both a complex product is four real MFMAs into a real
// and an imaginary accumulator, and Hermitian products (herm: M == N and op(B) = op(A)^H) compute
// the upper triangle, diagonal included, and write its mirror.
constexpr int GT = 32, GK = 16, GLD = GT + 4;

// Output element (row, col) of a Hermitian or general product, with alpha and accumulate.
__device__ __forceinline__ void gemm_store(z64* __restrict__ C, int ldc, int M, int N, int row, int col, double sr,
                                           double si, z64 alpha, int accumulate, int herm) {
  if (row >= M || col >= N || (herm && row > col)) return;
  z64 v = {alpha.re * sr - alpha.im * si, alpha.re * si + alpha.im * sr};
  if (accumulate) v = cadd(v, C[(size_t)row * ldc + col]);
  C[(size_t)row * ldc + col] = v;
  if (herm && row < col) C[(size_t)col * ldc + row] = cconj(v);
}

// Element e of a 32-row (or 32-column) operand tile times KC k values, as (row or column, k):
// k fastest when LAYOUT is 0, the row or column fastest when it is 1.  Each operand takes the
// order in which consecutive threads read consecutive addresses: A as is and B transposed are
// contiguous along k (layout 0), A transposed and B as is along the row or column (layout 1).
template <int LAYOUT, int KC>
__device__ __forceinline__ void tile_elem(int e, int& rc, int& kk) {
  if (LAYOUT == 0) {
    rc = e / KC;
    kk = e % KC;
  } else {
    rc = e % GT;
    kk = e / GT;
  }
}
template <int OP>
__device__ __forceinline__ z64 load_a(const z64* __restrict__ A, int lda, int M, int K, int gr, int gk) {
  z64 v = {0.0, 0.0};
  if (gr < M && gk < K) {
    if (OP == 0) {
      v = A[(size_t)gr * lda + gk];
    } else {
      v = A[(size_t)gk * lda + gr];
      v.im = -v.im;
    }
  }
  return v;
}
template <int OP>
__device__ __forceinline__ z64 load_b(const z64* __restrict__ B, int ldb, int N, int K, int gc, int gk) {
  z64 v = {0.0, 0.0};
  if (gc < N && gk < K) {
    if (OP == 0) {
      v = B[(size_t)gk * ldb + gc];
    } else {
      v = B[(size_t)gc * ldb + gk];
      v.im = -v.im;
    }
  }
  return v;
}

// Four waves, each a 16 x 16 quadrant of the tile, over every K chunk.
template <int OPA, int OPB>
__global__ __launch_bounds__(256) void k_zgemm(int M, int N, int K, const z64* __restrict__ A, int lda,
                                               const z64* __restrict__ B, int ldb, z64* __restrict__ C, int ldc,
                                               z64 alpha, int accumulate, int herm) {
  const int m0 = blockIdx.y * GT, n0 = blockIdx.x * GT;
  if (herm && m0 >= n0 + GT) return;  // entirely below the diagonal
  __shared__ double As[2][2][GK][GLD];  // [stage][re, im][k][row]
  __shared__ double Bs[2][2][GK][GLD];  // [stage][re, im][k][col]
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int wr = (w >> 1) * 16, wc = (w & 1) * 16;
  d4 accr = {0, 0, 0, 0}, acci = {0, 0, 0, 0};
  z64 ra[2], rb[2];
  auto fetch = [&](int k0) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      int r, kk;
      tile_elem<OPA, GK>(t + 256 * i, r, kk);
      ra[i] = load_a<OPA>(A, lda, M, K, m0 + r, k0 + kk);
      tile_elem<OPB == 0 ? 1 : 0, GK>(t + 256 * i, r, kk);
      rb[i] = load_b<OPB>(B, ldb, N, K, n0 + r, k0 + kk);
    }
  };
  auto stash = [&](int s) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      int r, kk;
      tile_elem<OPA, GK>(t + 256 * i, r, kk);
      As[s][0][kk][r] = ra[i].re;
      As[s][1][kk][r] = ra[i].im;
      tile_elem<OPB == 0 ? 1 : 0, GK>(t + 256 * i, r, kk);
      Bs[s][0][kk][r] = rb[i].re;
      Bs[s][1][kk][r] = rb[i].im;
    }
  };
  const int nch = (K + GK - 1) / GK;
  fetch(0);
  stash(0);
  __syncthreads();
  for (int c = 0; c < nch; ++c) {
    const int s = c & 1;
    if (c + 1 < nch) fetch((c + 1) * GK);
#pragma unroll
    for (int kk = 0; kk < GK; kk += 4) {
      const int ka = kk + (lane >> 4);
      const double ar = As[s][0][ka][wr + (lane & 15)], ai = As[s][1][ka][wr + (lane & 15)];
      const double br = Bs[s][0][ka][wc + (lane & 15)], bi = Bs[s][1][ka][wc + (lane & 15)];
      accr = __builtin_amdgcn_mfma_f64_16x16x4f64(ar, br, accr, 0, 0, 0);
      accr = __builtin_amdgcn_mfma_f64_16x16x4f64(-ai, bi, accr, 0, 0, 0);
      acci = __builtin_amdgcn_mfma_f64_16x16x4f64(ar, bi, acci, 0, 0, 0);
      acci = __builtin_amdgcn_mfma_f64_16x16x4f64(ai, br, acci, 0, 0, 0);
    }
    if (c + 1 < nch) stash(s ^ 1);
    __syncthreads();
  }
  for (int q = 0; q < 4; ++q)
    gemm_store(C, ldc, M, N, m0 + wr + mfma_row_f64(lane, q), n0 + wc + (lane & 15), accr[q], acci[q], alpha,
               accumulate, herm);
}

// One 16 x 16 tile per workgroup: the eight waves take eight k values each in turn, straight from memory into
// MFMA operands (the next ones while the current are multiplied), and their sums are added in a fixed
// order through LDS.  Bound by the MFMA pipe of one CU per tile (K / 4 steps of four MFMAs on four SIMDs) where the
// tiles are fewer than CUs, by the operands' L2 traffic (4 flop a byte) where they are many, and for small
// products by the launch, one load latency and the reduction.  Against 32 x 32 tiles staged through LDS, the K range
// split over two groups of four waves: 81 x 81 x 81 4.1 and 7.0 us (back to back, so mostly the launch), the Gram
// of 243 x 729 12.4 and 38.6, 128 x 128 x 1152 18.0 and 58.2, 384^3 16.2 and 20.3, 768 x 256 x 768 28.2 and
// 36.6, the Gram of 729 x 729 52 and 99 us.
constexpr int ST = 16, SLD = ST + 1;
template <int OPA, int OPB>
__global__ __launch_bounds__(512) void k_zgemm_s(int M, int N, int K, const z64* __restrict__ A, int lda,
                                                 const z64* __restrict__ B, int ldb, z64* __restrict__ C, int ldc,
                                                 z64 alpha, int accumulate, int herm) {
  const int m0 = blockIdx.y * ST, n0 = blockIdx.x * ST;
  if (herm && m0 > n0) return;  // entirely below the diagonal
  __shared__ z64 part[8][ST * SLD];
  const int t = threadIdx.x, lane = t & 63, col = lane & 15, quad = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  d4 accr = {0, 0, 0, 0}, acci = {0, 0, 0, 0};
  z64 a[2], b[2];
  auto fetch = [&](int k0) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      a[j] = load_a<OPA>(A, lda, M, K, m0 + col, k0 + 4 * j + quad);
      b[j] = load_b<OPB>(B, ldb, N, K, n0 + col, k0 + 4 * j + quad);
    }
  };
  fetch(w * 8);
  for (int k0 = w * 8; k0 < K; k0 += 64) {
    const z64 a0 = a[0], a1 = a[1], b0 = b[0], b1 = b[1];
    if (k0 + 64 < K) fetch(k0 + 64);
    mma4(a0, b0, accr, acci);
    mma4(a1, b1, accr, acci);
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) part[w][mfma_row_f64(lane, q) * SLD + col] = z64{accr[q], acci[q]};
  __syncthreads();
  const bool act = t < ST * ST;
  const int i = t / ST, j = t % ST, row = m0 + i, cc = n0 + j;
  if (act) {
    z64 s = part[0][i * SLD + j];
    const int used = min(8, (K + 7) / 8);
    for (int x = 1; x < used; ++x) s = cadd(s, part[x][i * SLD + j]);
    s = z64{alpha.re * s.re - alpha.im * s.im, alpha.re * s.im + alpha.im * s.re};
    const bool in = row < M && cc < N;
    if (accumulate && in) s = cadd(s, C[(size_t)row * ldc + cc]);
    if (in && !(herm && row > cc)) C[(size_t)row * ldc + cc] = s;
    if (herm) part[0][i * SLD + j] = s;
  }
  if (!herm) return;
  __syncthreads();
  // the mirror of the tile, by rows of the mirror
  const int mr = n0 + i, mc = m0 + j;
  if (act && mr < M && mc < mr) C[(size_t)mr * ldc + mc] = cconj(part[0][j * SLD + i]);
}

// ===================================================================================== Jacobi
// Single-workgroup Jacobi: G (m x m, m <= 2 HM) -> U (m x m), lam (m), all in LDS; 2 HM^2 threads.
template <int HM, bool REL>
__global__ __launch_bounds__(2 * HM * HM) void k_jacobi_small(const z64* __restrict__ G, int ldg_in, int m,
                                                              z64* __restrict__ U, int ldu, double* __restrict__ lam,
                                                              JacobiCrit cr, DevStatus* st) {
  constexpr int LD = 2 * HM;
  __shared__ __align__(16) z64 hs[2 * LD * LD], v[LD * LD];
  __shared__ int pending[2];
  __shared__ double trace;
  const int t = threadIdx.x, nt = blockDim.x;
  for (int idx = t; idx < LD * LD; idx += nt) {
    const int i = idx / LD, j = idx % LD;
    z64 x = (i < m && j < m) ? G[(size_t)i * ldg_in + j] : z64{0.0, 0.0};
    if (i == j) x.im = 0.0;
    hs[idx] = x;
    v[idx] = z64{(i == j) ? 1.0 : 0.0, 0.0};
  }
  if (t < 2) pending[t] = 0;
  __syncthreads();
  jacobi_trace<LD>(hs, m, &trace);
  __syncthreads();
  const JacobiThr jt = jacobi_thr(trace, cr.tol, cr.skip_rel, REL, cr.floor_rel);
  int sweeps;
  bool conv;
  const z64* h = jacobi_sweeps<HM, REL>(hs, v, m, jt, cr.max_sweeps, pending, &sweeps, &conv);
  for (int i = t; i < m; i += nt) lam[i] = h[i * (LD + 1)].re;
  for (int idx = t; idx < m * m; idx += nt) {
    const int i = idx / m, j = idx - (idx / m) * m;
    U[(size_t)i * ldu + j] = v[i * LD + j];
  }
  if (t == 0 && st) {
    st->converged = conv ? 1 : 0;
    st->sweeps = sweeps;
  }
}

// ----------------------------------------------------------------------- block Jacobi
constexpr int BJ = kBlk;      // block size (16)
constexpr int kSolveThreads = 512;  // threads per 32x32 sub-problem (block and V updates split)
static_assert(kSolveThreads == 2 * BJ * BJ, "the inter-block steps give each thread one block or one V item");
constexpr int BJ2 = 2 * kBlk; // pair size (32)

// The pair holding block b at outer step s and b's offset in it (0: first block, BJ: second):
// the inverse of rr_pair over nb blocks.  Block 0 stays in pair 0; another block b sits at
// position x = (b - 1 - s) mod (nb - 1) of the rotating circle, which is the first slot of pair
// x + 1 for x < nb / 2 - 1 and the second slot of pair nb - 2 - x otherwise.
__device__ __forceinline__ void block_home(int b, int s, int nb, int& pair, int& off) {
  if (b == 0) {
    pair = 0;
    off = 0;
    return;
  }
  int x = b - 1 - s;  // in (-(nb - 1), nb - 1)
  if (x < 0) x += nb - 1;
  pair = (x <= nb / 2 - 2) ? x + 1 : nb - 2 - x;
  int I, J;
  rr_pair(pair, s, nb, I, J);
  off = (b == I) ? 0 : BJ;
}

// The tile updates: four waves per 32 x 32 tile (one 16 x 16 quadrant each), two tiles per block,
// operands straight from global memory into MFMA registers.  Only the first product of a G tile
// passes through LDS, so that each wave can read both row halves of it.  A tile per block staged
// through LDS and multiplied by half of the block's waves bound a round from about m = 600 on
// (15 us there); one wave per 16-column half bound it at every size (13.5 us at m = 243: 128
// dependent MFMAs per wave).
constexpr int kTilesPerBlock = kSolveThreads / 256;

// Quadrant product: acc = A(16 x 32) B(32 x 16) with B in b (b[j]: row 4 j + l / 16) and A's element
// (row, kk) at a0[row * lda + kk] for kk < 16, a1[row * lda + kk - 16] otherwise.
__device__ __forceinline__ void tile_mul(const z64* __restrict__ a0, const z64* __restrict__ a1, size_t lda,
                                         const z64* b, d4& xr, d4& xi) {
  const int lane = threadIdx.x & 63, lo = lane & 15, hi = lane >> 4;
  z64 a[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) a[j] = (j < 4 ? a0 : a1)[lo * lda + 4 * (j & 3) + hi];
#pragma unroll
  for (int j = 0; j < 8; ++j) mma4(a[j], b[j], xr, xi);
}

// Column half ch of V_Q as an operand (v[j]: row 4 j + l / 16, column l % 16 of the half), or the
// identity's when the pair did not rotate.
__device__ __forceinline__ void load_vhalf(const z64* __restrict__ V, int Q, int flag, int ch, z64* v) {
  const int lane = threadIdx.x & 63, lo = lane & 15, hi = lane >> 4;
#pragma unroll
  for (int j = 0; j < 8; ++j) v[j] = V[(size_t)Q * BJ2 * BJ2 + (4 * j + hi) * BJ2 + ch * BJ + lo];
  if (!flag)
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = z64{(4 * j + hi == ch * BJ + lo) ? 1.0 : 0.0, 0.0};
}

// Row tile (R, Q), tile = R half + Q, of U <- U V_Q, in place: all of a tile is read before any of
// it is written (the barrier).
__device__ void u_tile(z64* __restrict__ Up, int mp, int nb, int step, const z64* __restrict__ V,
                       const int* __restrict__ pair_flag, int tile, int ntiles) {
  const int half = nb / 2, lane = threadIdx.x & 63, lo = lane & 15, wv = threadIdx.x >> 6, ch = wv & 1,
            rh = (wv >> 1) & 1;
  const int R = tile / half, Q = tile % half;
  const bool run = tile < ntiles && pair_flag[Q];  // uniform over the tile's waves
  d4 xr = {0, 0, 0, 0}, xi = {0, 0, 0, 0};
  int q0, q1;
  rr_pair(Q, step, nb, q0, q1);
  z64* u = Up + (size_t)(R * BJ2 + rh * BJ) * mp;
  if (run) {
    z64 b[8];
    load_vhalf(V, Q, 1, ch, b);
    tile_mul(u + q0 * BJ, u + q1 * BJ, mp, b, xr, xi);
  }
  __syncthreads();
  if (run)
#pragma unroll
    for (int q = 0; q < 4; ++q) {  // streamed: no later block of this round reads them
      const d2 x = {xr[q], xi[q]};
      __builtin_nontemporal_store(
          x, reinterpret_cast<d2*>(u + (size_t)mfma_row_f64(lane, q) * mp + (ch ? q1 : q0) * BJ + lo));
    }
}

// Tile (P, Q), P <= Q (numbered along the rows of the upper triangle), of the round's update
// Gd = V^H Gs V; the (Q, P) tile is written as the conjugate transpose.  A pair that did not rotate
// contributes the identity; a tile whose two pairs both did not rotate is copied as it is (with its
// mirror), and a diagonal tile is the pair's solved sub-problem.  xs: 1024 elements of LDS per tile.
__device__ void g_tile(const z64* __restrict__ Gs, z64* __restrict__ Gd, int mp, int nb, int step,
                       const z64* __restrict__ V, const z64* __restrict__ D, const int* __restrict__ pair_flag,
                       int tile, int ntiles, z64* __restrict__ xs) {
  const int half = nb / 2, lane = threadIdx.x & 63, lo = lane & 15, hi = lane >> 4, wv = threadIdx.x >> 6, ch = wv & 1,
            rh = (wv >> 1) & 1;
  const bool live = tile < ntiles;  // uniform over the tile's waves, as all conditions below
  int P = 0, rem = live ? tile : 0;
  while (rem >= half - P) {
    rem -= half - P;
    ++P;
  }
  const int Q = P + rem;
  int p0, p1, q0, q1;
  rr_pair(P, step, nb, p0, p1);
  rr_pair(Q, step, nb, q0, q1);
  const int gr0 = (rh ? p1 : p0) * BJ, gc = (ch ? q1 : q0) * BJ + lo;  // the quadrant's rows, this lane's column
  const int fP = pair_flag[P], fQ = pair_flag[Q];
  const bool mul = live && P != Q && (fP || fQ);
  z64 vp[8];
  if (mul) {
    z64 b[8];
    d4 xr = {0, 0, 0, 0}, xi = {0, 0, 0, 0};
    load_vhalf(V, Q, fQ, ch, b);
    load_vhalf(V, P, fP, rh, vp);
    tile_mul(Gs + (size_t)gr0 * mp + q0 * BJ, Gs + (size_t)gr0 * mp + q1 * BJ, mp, b, xr, xi);  // X = T V_Q
#pragma unroll
    for (int q = 0; q < 4; ++q) xs[ch * 512 + (rh * BJ + mfma_row_f64(lane, q)) * BJ + lo] = z64{xr[q], xi[q]};
  }
  __syncthreads();
  if (mul) {  // Y = V_P^H X
    d4 yr = {0, 0, 0, 0}, yi = {0, 0, 0, 0};
#pragma unroll
    for (int j = 0; j < 8; ++j) mma4(cconj(vp[j]), xs[ch * 512 + (4 * j + hi) * BJ + lo], yr, yi);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int gr = gr0 + mfma_row_f64(lane, q);
      Gd[(size_t)gr * mp + gc] = z64{yr[q], yi[q]};
      Gd[(size_t)gc * mp + gr] = z64{yr[q], -yi[q]};
    }
  } else if (live) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = 4 * i + hi, gr = gr0 + r;
      if (P == Q) {
        Gd[(size_t)gr * mp + gc] = D[(size_t)P * BJ2 * BJ2 + (rh * BJ + r) * BJ2 + ch * BJ + lo];
      } else {
        const z64 x = Gs[(size_t)gr * mp + gc];
        Gd[(size_t)gr * mp + gc] = x;
        Gd[(size_t)gc * mp + gr] = cconj(x);
      }
    }
  }
}

// The 32x32 sub-problem of blocks (I, J) after the previous round's update, from the matrix before
// that update (Gs) and that round's results (rotations V, solved sub-problems D, flags pf, outer
// step ps), into h (32 x 32).  With P and Q the previous pairs of I and J (offsets oI and oJ in
// them; P != Q, since consecutive rounds pair no two blocks twice), the diagonal blocks are those
// that P's and Q's solves left, and the off-diagonal block is the (oI, oJ) quadrant of
// V_P^H G_PQ V_Q: the only product a round's critical path has to wait for.  Waves 0..3 form it
// straight from global memory into MFMA operands, X = G_PQ V_Q[:, oJ..] by row and K halves and
// then V_P[:, oI..]^H X by K quarters; waves 4..7 fetch the diagonal blocks.  xs and ys are
// scratch of 1024 elements.  A product over the whole (P, Q) tile, with the diagonal tiles
// multiplied as well, took 5.5 us per round at m = 768.
__device__ void rebuild_pair(int I, int J, const z64* __restrict__ Gs, int mp, int nb, int ps,
                             const z64* __restrict__ V, const z64* __restrict__ D, const int* __restrict__ pf,
                             z64* __restrict__ xs, z64* __restrict__ ys, z64* __restrict__ h) {
  const int t = threadIdx.x, lane = t & 63, w = t >> 6, lo = lane & 15, hi = lane >> 4;
  int P, oI, Q, oJ;
  block_home(I, ps, nb, P, oI);
  block_home(J, ps, nb, Q, oJ);
  z64 vp[2];
  if (w < 4) {
    const int rh = w & 1, kh = w >> 1;
    int p0, p1, q0, q1;
    rr_pair(P, ps, nb, p0, p1);
    rr_pair(Q, ps, nb, q0, q1);
    const z64* g = Gs + (size_t)((rh ? p1 : p0) * BJ + lo) * mp + (kh ? q1 : q0) * BJ + hi;
    const z64* vq = V + (size_t)Q * BJ2 * BJ2 + (kh * BJ + hi) * BJ2 + oJ + lo;
    const z64* vpp = V + (size_t)P * BJ2 * BJ2 + (w * 8 + hi) * BJ2 + oI + lo;
    z64 a[4], b[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      a[j] = g[4 * j];
      b[j] = vq[4 * j * BJ2];
    }
    vp[0] = vpp[0];
    vp[1] = vpp[4 * BJ2];
    const int fP = pf[P], fQ = pf[Q];
    // a pair that did not rotate left no V: its rotation is the identity
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (!fQ) b[j] = z64{(kh * BJ + 4 * j + hi == oJ + lo) ? 1.0 : 0.0, 0.0};
#pragma unroll
    for (int j = 0; j < 2; ++j)
      if (!fP) vp[j] = z64{(w * 8 + 4 * j + hi == oI + lo) ? 1.0 : 0.0, 0.0};
    d4 accr = {0, 0, 0, 0}, acci = {0, 0, 0, 0};
#pragma unroll
    for (int j = 0; j < 4; ++j) mma4(a[j], b[j], accr, acci);
#pragma unroll
    for (int q = 0; q < 4; ++q)
      xs[kh * 512 + (rh * BJ + mfma_row_f64(lane, q)) * BJ + lo] = z64{accr[q], acci[q]};
  } else {
    // upper elements, mirrored: the rotations leave the two triangles equal only to rounding, and
    // what differs would add up from round to round
    const int e = t - 256, i = e >> 4, j = e & 15, r = min(i, j), c = max(i, j);
    z64 x = D[(size_t)P * BJ2 * BJ2 + (oI + r) * BJ2 + oI + c];
    z64 y = D[(size_t)Q * BJ2 * BJ2 + (oJ + r) * BJ2 + oJ + c];
    const double sg = i < j ? 1.0 : i > j ? -1.0 : 0.0;
    x.im *= sg;
    y.im *= sg;
    h[i * BJ2 + j] = x;
    h[(BJ + i) * BJ2 + BJ + j] = y;
  }
  __syncthreads();
  if (w < 4) {
    d4 accr = {0, 0, 0, 0}, acci = {0, 0, 0, 0};
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int kk = w * 8 + 4 * j + hi;
      mma4(cconj(vp[j]), cadd(xs[kk * BJ + lo], xs[512 + kk * BJ + lo]), accr, acci);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) ys[w * 256 + mfma_row_f64(lane, q) * BJ + lo] = z64{accr[q], acci[q]};
  }
  __syncthreads();
  if (t < 256) {
    const z64 x = cadd(cadd(ys[t], ys[256 + t]), cadd(ys[512 + t], ys[768 + t]));
    const int i = t >> 4, j = t & 15;
    h[i * BJ2 + BJ + j] = x;
    h[(BJ + j) * BJ2 + i] = cconj(x);
  }
}

// Solve step of a round: pair k of outer step `step` solves its 32x32 sub-problem (blocks I, J)
// and writes the accumulated rotation to V + k*32*32 (row-major, only when it rotated, as the pair's
// flag says) and the rotated sub-problem to D + k*32*32.  The first step of an outer sweep also covers the
// pairs inside each block; later steps rotate only the 16 x 16 inter-block pairs.  Over one outer sweep every index pair is visited
// once.  With ps < 0 the sub-problem is read from Gs; otherwise it is rebuilt from the matrix before
// the previous round's update (rebuild_pair), that update running beside this solve.
// pool: 3 x 1024 elements of LDS.
template <bool REL>
__device__ void solve_pair(int k, const z64* __restrict__ Gs, int mp, int nb, int step, int ps,
                           const z64* __restrict__ Vp, const z64* __restrict__ Dp, const int* __restrict__ pfp,
                           const JacobiThr& jt, z64* __restrict__ Vout, z64* __restrict__ Dout,
                           int* __restrict__ pair_flag, int* __restrict__ any_flag, const int* __restrict__ prev_any,
                           z64* __restrict__ pool, int& need) {
  const int t = threadIdx.x;
  const int live = prev_any ? *prev_any : 1;  // tested after the loads below are on their way
  z64 *h0 = pool, *h1 = pool + BJ2 * BJ2, *v = pool + 2 * BJ2 * BJ2;
  int I, J;
  rr_pair(k, step, nb, I, J);
  const bool full = (step == 0);
  if (t == 0) need = 0;
  if (ps < 0) {
    for (int idx = t; idx < BJ2 * BJ2; idx += kSolveThreads) {
      const int i = idx / BJ2, j = idx % BJ2;
      const int gi = (i < BJ ? I * BJ + i : J * BJ + (i - BJ));
      const int gj = (j < BJ ? I * BJ + j : J * BJ + (j - BJ));
      z64 x = Gs[(size_t)gi * mp + gj];
      if (i == j) x.im = 0.0;
      h0[idx] = x;
    }
  } else {
    rebuild_pair(I, J, Gs, mp, nb, ps, Vp, Dp, pfp, h1, v, h0);
  }
  if (!live) return;
  __syncthreads();
  bool hit = false;
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int idx = t + u * kSolveThreads, i = idx / BJ2, j = idx % BJ2;
    if (i < j && (full || (i < BJ && j >= BJ)))
      hit = hit || rot_needed<REL>(h0[i * (BJ2 + 1)].re, h0[j * (BJ2 + 1)].re, cabs2(h0[idx]), jt);
    if (full) v[idx] = z64{(i == j) ? 1.0 : 0.0, 0.0};
  }
  if (hit) need = 1;
  __syncthreads();
  const int run = need;  // then some pair rotates: the first one met above the threshold at the latest
  const z64* res = h0;
  if (run) {
    z64* vo = Vout + (size_t)k * BJ2 * BJ2;
    if (full) {
      jacobi_intra_steps<REL, true>(h0, h1, v, jt);
      res = h1;
    }
    jacobi_ib_steps<REL>(full ? h1 : h0, full ? h0 : h1, full ? v : nullptr, vo, jt);
  }
  for (int idx = t; idx < BJ2 * BJ2; idx += kSolveThreads) Dout[(size_t)k * BJ2 * BJ2 + idx] = res[idx];
  if (t == 0) {
    pair_flag[k] = run;
    if (run) atomicOr(any_flag, 1);
  }
}

// One round of the block Jacobi sweep in one launch.  Blocks 0..half-1 (when step >= 0) solve the
// sub-problems of outer step `step` (rotations to Vout, solved sub-problems to Dout, flags to
// pair_flag, any rotation to *any_flag); when ps >= 0 the previous round (outer step ps, rotations
// Vp, solved sub-problems Dp, flags pfp) is applied beside them: the next blocks form
// the half(half+1)/2 tiles of Gd = V^H Gs V, the remaining ones the (mp/32) half row tiles of U <- U V.  The solves rebuild their sub-problems from Gs, so no
// block waits for another; Gs and Gd alternate between rounds.  512 threads.  With a non-null
// prev_any that holds 0 (the sweep before rotated nothing) the round does nothing: rounds may be
// launched before the host knows that the sweeps have converged.
//
// What bounds it: a round is as long as one solve.  At m = 243 a round takes 12.0 us (20.1 with one
// refined rotation per thread and scalar LDS accesses): the launch and the loads 4 to 5 us (what a round
// without rotations takes), the two small products of the rebuild and 16 steps of 0.3 to 0.4 us; the
// rounds that start a sweep 20 us.  At m = 384 with the relative criterion 13.4 us.
// Launched with kJroundPad bytes of (unused) dynamic LDS, a block holds more than half of a CU's
// 160 KB, so a solve never shares its SIMDs with tile updates.  That pays while the updates are few
// (m = 768: 16.6 against 17.9 ms per decomposition) and costs once they dominate (m = 1024: 29.8
// against 27.6 ms; m = 1536: 82.0 against 70.5 ms), where the rounds go without the pad.
constexpr int kJroundPad = 36 * 1024;
constexpr int kPadMaxM = 896;
template <bool REL>
__global__ __launch_bounds__(512) void k_jround(const z64* __restrict__ Gs, z64* __restrict__ Gd,
                                                z64* __restrict__ Up, int mp, int nb, int step, int ps,
                                                const double* __restrict__ trace, double tol, double skip_rel,
                                                double floor_rel, z64* __restrict__ Vout, z64* __restrict__ Dout,
                                                int* __restrict__ pair_flag, int* __restrict__ any_flag,
                                                const int* __restrict__ prev_any, const z64* __restrict__ Vp,
                                                const z64* __restrict__ Dp, const int* __restrict__ pfp,
                                                SweepReport* report, Ticket ticket) {
  __shared__ __align__(16) z64 pool[3 * BJ2 * BJ2];
  __shared__ int need;
  const int half = nb / 2, nsolve = step >= 0 ? half : 0, ngt = half * (half + 1) / 2;
  int b = blockIdx.x;
  if (report && b == 0 && threadIdx.x == 0) {
    report->rotated = *prev_any;
    announce(&report->ticket, ticket);
  }
  if (b < nsolve) {
    // thresholds from the trace on the device (read by no host sync)
    const JacobiThr jt = jacobi_thr(*trace, tol, skip_rel, REL, floor_rel);
    solve_pair<REL>(b, Gs, mp, nb, step, ps, Vp, Dp, pfp, jt, Vout, Dout, pair_flag, any_flag, prev_any, pool, need);
    return;
  }
  if (prev_any && !*prev_any) return;
  b -= nsolve;
  const int sub = threadIdx.x >> 8, ngb = (ngt + kTilesPerBlock - 1) / kTilesPerBlock;
  if (b < ngb)
    g_tile(Gs, Gd, mp, nb, ps, Vp, Dp, pfp, b * kTilesPerBlock + sub, ngt, pool + sub * BJ2 * BJ2);
  else
    u_tile(Up, mp, nb, ps, Vp, pfp, (b - ngb) * kTilesPerBlock + sub, (mp / BJ2) * half);
}

__global__ void k_pad_copy(const z64* __restrict__ G, int m, int ldg, z64* __restrict__ Gp, int mp,
                           z64* __restrict__ Up) {
  size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (size_t)mp * mp) return;
  int i = (int)(idx / mp), j = (int)(idx % mp);
  Gp[idx] = (i < m && j < m) ? G[(size_t)i * ldg + j] : z64{0.0, 0.0};
  Up[idx] = (i == j) ? z64{1.0, 0.0} : z64{0.0, 0.0};
}

// The pre-check's bounds.  A Rayleigh-Ritz matrix is diagonal to the rounding of its products, a few 1e-16 of the
// trace, so the sweeps' bound of 3e-16 for every pair calls for a sweep each time (m = 600: 0.7 ms).  Between
// directions that are all kept, or all dropped, entries up to kPrecheckTol may stay: they change neither space and
// leave B's rows orthogonal to kPrecheckTol / discardable (5e-13 at 256 kept).  One that may be kept and one that may be
// dropped are held to the sweeps' bound, unless what stays tilts them by no more than the rounding of the
// rotations that made them (m 2^-53 = 8.5e-14 at m = 768).
constexpr double kPrecheckTol = 2e-15, kPrecheckTilt = 1e-13;
constexpr int kSweepFlags = 128;  // one rotation flag per sweep

__global__ void k_trace(const z64* __restrict__ Gp, int m, int mp, double* out, int* __restrict__ sweep_flags) {
  __shared__ double red[256];
  double s = 0.0;
  for (int i = threadIdx.x; i < m; i += blockDim.x) s += fabs(Gp[(size_t)i * mp + i].re);
  red[threadIdx.x] = s;
  __syncthreads();
  for (int off = 128; off > 0; off >>= 1) {
    if ((int)threadIdx.x < off) red[threadIdx.x] += red[threadIdx.x + off];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    out[0] = red[0];
    reinterpret_cast<int*>(out + 1)[0] = 0;  // pre-check flag, set by k_offdiag_check
  }
  if (threadIdx.x < kSweepFlags) sweep_flags[threadIdx.x] = 0;
}

// Pre-check of a decomposition: sets *flag when some pair (i < j < m) of Gp has an entry g above kPrecheckTol of the
// trace (in *trace_in, from k_trace), or one above tol of it and above kPrecheckTilt of the difference of the
// diagonal entries where the smaller of these is at most discardable of the trace.
__global__ void k_offdiag_check(const z64* __restrict__ Gp, int m, int mp, const double* __restrict__ trace_in,
                                double tol, double discardable, int* __restrict__ flag) {
  const JacobiThr strict = jacobi_thr(*trace_in, tol, 0.0, 0, 0.0), kept = jacobi_thr(*trace_in, kPrecheckTol, 0.0, 0, 0.0);
  const double may_drop = discardable * *trace_in;
  const size_t total = (size_t)m * m;
  int hit = 0;
  for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (size_t)gridDim.x * blockDim.x) {
    const int i = (int)(e / m), j = (int)(e % m);
    if (i < j) {
      const double h2 = cabs2(Gp[(size_t)i * mp + j]);
      const double a = Gp[(size_t)i * mp + i].re, b = Gp[(size_t)j * mp + j].re;
      const bool mixes = fmin(a, b) <= may_drop && h2 > kPrecheckTilt * kPrecheckTilt * (a - b) * (a - b);
      if (rot_needed<false>(a, b, h2, mixes ? strict : kept)) hit = 1;
    }
  }
  if (hit) atomicOr(flag, 1);
}

__global__ void k_unpad(const z64* __restrict__ Gp, const z64* __restrict__ Up, int m, int mp, z64* __restrict__ U,
                        int ldu, double* __restrict__ lam) {
  size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (size_t)m * m) return;
  int i = (int)(idx / m), j = (int)(idx % m);
  U[(size_t)i * ldu + j] = Up[(size_t)i * mp + j];
  if (j == 0) lam[i] = Gp[(size_t)i * mp + i].re;
}

// ===================================================================================== misc
__global__ void k_rownorm2(const z64* __restrict__ B, int m, int k, int ldb, double* __restrict__ out) {
  __shared__ double red[256];
  const int r = blockIdx.x;
  double s = 0.0;
  for (int c = threadIdx.x; c < k; c += blockDim.x) s += cabs2(B[(size_t)r * ldb + c]);
  red[threadIdx.x] = s;
  __syncthreads();
  for (int off = 128; off > 0; off >>= 1) {
    if ((int)threadIdx.x < off) red[threadIdx.x] += red[threadIdx.x + off];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[r] = red[0];
}

// Truncation rule on squared values sig2 (any order).  Sorted descending (ties by index).
//   w_j = sig2_j / sum sig2;  tail[k] = sum_{j >= k} w_j  (sums of values from k on alone, added from the end)
//   k_cut = smallest k >= 1 with tail[k] <= cutoff; k_floor = #{sigma_j > 1e-13 sigma_0}
//   k = min(k_cut, k_floor, chi_max); degeneracy guard as in the truncation rule.
// mode 1 keeps k_floor (exact moves).  need_pass2 when a kept value is below 1e-12 sig2_0.
// force_k > 0 replaces the rule by that rank (frozen-decision replay; never flagged).
// Bound by the barriers of the sort.  With the sums and counts by one thread m = 243 took 39 us and m = 768 88 us,
// this way 16.6 and 26.6 us.
constexpr int TRUNC_MAX = 4096;
__global__ __launch_bounds__(1024) void k_trunc(const double* __restrict__ sig2, int m, double cutoff, int chi_max,
                                                int mode, int force_k, int* __restrict__ perm,
                                                double* __restrict__ sig_sorted, DevStatus* st,
                                                const double* __restrict__ extra) {
  __shared__ double key[TRUNC_MAX];
  __shared__ int idx[TRUNC_MAX];
  __shared__ double wsum[16], tail_k;
  __shared__ int above, over, below;
  int P2 = 1;
  while (P2 < m) P2 <<= 1;
  const int t = threadIdx.x, nt = blockDim.x;
  for (int i = t; i < P2; i += nt) {
    key[i] = (i < m) ? fmax(sig2[i], 0.0) : -1.0;
    idx[i] = i;
  }
  __syncthreads();
  // bitonic sort: descending key, ascending index on ties
  for (int size = 2; size <= P2; size <<= 1) {
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      for (int i = t; i < P2; i += nt) {
        int j = i ^ stride;
        if (j > i) {
          bool desc = ((i & size) == 0);
          double ki = key[i], kj = key[j];
          int ii = idx[i], ij = idx[j];
          bool i_before_j = (ki > kj) || (ki == kj && ii < ij);
          bool swap = desc ? !i_before_j : i_before_j;
          if (swap) {
            key[i] = kj;
            key[j] = ki;
            idx[i] = ij;
            idx[j] = ii;
          }
        }
      }
      __syncthreads();
    }
  }
  for (int i = t; i < m; i += nt) {
    perm[i] = idx[i];
    sig_sorted[i] = sqrt(key[i]);
  }
  // E consecutive values a thread; tail[e]: the weight of value e and all after it and outside the list
  // (always discarded), by suffix sums within the threads, the waves and over them.
  const int E = (P2 + nt - 1) / nt, i0 = t * E, lane = t & 63, w = t >> 6;
  double tail[TRUNC_MAX / 1024], sum = 0.0;
#pragma unroll
  for (int e = TRUNC_MAX / 1024 - 1; e >= 0; --e) {
    if (e < E && i0 + e < m) sum += key[i0 + e];
    tail[e] = sum;
  }
  double after = sum;  // of this thread and the later lanes of its wave
  for (int off = 1; off < 64; off <<= 1) {
    const double o = __shfl_down(after, off, 64);
    if (lane + off < 64) after += o;
  }
  // of the later lanes alone: after - sum would lose them where this thread holds both sides of a gap
  const double next = __shfl_down(after, 1, 64), later = lane < 63 ? next : 0.0;
  if (lane == 0) wsum[w] = after;
  if (t == 0) {
    above = over = below = 0;
    tail_k = 0.0;
  }
  __syncthreads();
  const double ex = extra ? fmax(*extra, 0.0) : 0.0;
  double rest = ex;
  for (int x = nt / 64 - 1; x > w; --x) rest += wsum[x];
  rest += later;
  double total = ex;
  for (int x = nt / 64 - 1; x >= 0; --x) total += wsum[x];
  const double s0 = sqrt(key[0]);
  auto apart = [&](int i) { return !(sqrt(key[i]) >= sqrt(key[i - 1]) * (1.0 - 1e-10)); };
  int my_above = 0, my_over = 0;
#pragma unroll
  for (int e = 0; e < TRUNC_MAX / 1024; ++e) {
    const int i = i0 + e;
    tail[e] += rest;
    if (e >= E || i >= m) continue;
    if (sqrt(key[i]) > 1e-13 * s0) ++my_above;
    if (i >= 1 && tail[e] / total > cutoff) ++my_over;
  }
  if (my_above) atomicAdd(&above, my_above);
  if (my_over) atomicAdd(&over, my_over);
  __syncthreads();
  const int kcut = over + 1, kfloor = above;  // the tails descend: the first at or below the cutoff
  int k, flagged = 0;
  if (mode == 1) {
    k = max(kfloor, 1);
  } else {
    k = max(min(min(kcut, kfloor), chi_max), 1);
    // a cut inside a degenerate block drops the whole block
    if (k < m && sqrt(key[k]) > 1e-13 * s0 && !apart(k)) {
      for (int i = t; i < k; i += nt)
        if (i >= 1 && apart(i)) atomicMax(&below, i);
      __syncthreads();  // k, and with it the branch, is the same for every thread
      if (below == 0)
        flagged = 1;
      else
        k = below;
    }
  }
  if (force_k > 0) {
    k = min(force_k, m);
    flagged = 0;
  }
#pragma unroll
  for (int e = 0; e < TRUNC_MAX / 1024; ++e)
    if (e < E && i0 + e == k && k < m) tail_k = tail[e];
  __syncthreads();
  if (t == 0) {
    st->kept = k;
    st->eps = (k < m ? tail_k : ex) / total;
    st->flagged = flagged;
    st->need_pass2 = (key[k - 1] < 1e-12 * key[0]) ? 1 : 0;
    st->lam_max = key[0];
  }
}

// Factor emission.  W is the wide orientation of the split matrix M (p x q): wide = 1 when
// W = M (p <= q, m = p, kW = q), wide = 0 when W = M^H (m = q, kW = p).  With U (m x m) the
// eigenvectors of W W^H, B = U^H W (m x kW), perm the sorted order (null: sorted already) and sig the row norms of B:
//   wide, left_ortho : L = U[:, perm],            R = B[perm, :] * rn
//   wide, right_ortho: L = U[:, perm] * sig * rn, R = B[perm, :] / sig
//   tall, left_ortho : L = B[perm, :]^H / sig,    R = sig * rn * U[:, perm]^H
//   tall, right_ortho: L = B[perm, :]^H * rn,     R = U[:, perm]^H
// rn = 1 / sqrt(sum_kept sig^2) when renorm, else 1.
__global__ void k_emit(int wide, int left_ortho, int renorm, int p, int q, int kept, const z64* __restrict__ U,
                       int ldu, const z64* __restrict__ B, int ldb, const int* __restrict__ perm,
                       const double* __restrict__ sig, z64* __restrict__ L, z64* __restrict__ R) {
  __shared__ double part[4];
  double sq = 0.0;
  for (int j = threadIdx.x; j < kept; j += 256) sq += sig[j] * sig[j];
  for (int off = 32; off > 0; off >>= 1) sq += __shfl_xor(sq, off, 64);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = sq;
  __syncthreads();
  const double rn = renorm ? 1.0 / sqrt(part[0] + part[1] + part[2] + part[3]) : 1.0;
  size_t nl = (size_t)p * kept, nr = (size_t)kept * q;
  size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx < nl) {
    int i = (int)(idx / kept), j = (int)(idx % kept);
    int pj = perm ? perm[j] : j;
    z64 v;
    if (wide) {
      v = U[(size_t)i * ldu + pj];
      if (!left_ortho) v = cscale(v, sig[j] * rn);
    } else {
      v = cconj(B[(size_t)pj * ldb + i]);
      v = left_ortho ? cscale(v, 1.0 / sig[j]) : cscale(v, rn);
    }
    L[idx] = v;
  } else if (idx < nl + nr) {
    size_t e = idx - nl;
    int j = (int)(e / q), c = (int)(e % q);
    int pj = perm ? perm[j] : j;
    z64 v;
    if (wide) {
      v = B[(size_t)pj * ldb + c];
      v = left_ortho ? cscale(v, rn) : cscale(v, 1.0 / sig[j]);
    } else {
      v = cconj(U[(size_t)c * ldu + pj]);
      if (left_ortho) v = cscale(v, sig[j] * rn);
    }
    R[e] = v;
  }
}

__global__ void k_copy(z64* __restrict__ dst, const z64* __restrict__ src, size_t count) {
  size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx < count) dst[idx] = src[idx];
}

__global__ void k_fill_identity(z64* U, int m, int ld) {
  size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (size_t)m * m) return;
  int i = (int)(idx / m), j = (int)(idx % m);
  U[(size_t)i * ld + j] = (i == j) ? z64{1.0, 0.0} : z64{0.0, 0.0};
}

inline unsigned blocks_for(size_t n, int bs) { return (unsigned)((n + bs - 1) / bs); }

}  // namespace

// ===================================================================================== launchers
void linalg_set_attributes() {
  // the rounds' optional LDS pad is dynamic shared memory; static plus dynamic exceeds 64 KB
  for (const void* f : {reinterpret_cast<const void*>(k_jround<false>), reinterpret_cast<const void*>(k_jround<true>)})
    (void)hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, kJroundPad);
  (void)hipGetLastError();
}

void launch_zgemm(hipStream_t s, int opa, int opb, int M, int N, int K, const z64* A, int lda, const z64* B,
                  int ldb, z64* C, int ldc, z64 alpha, int accumulate, int herm) {
  if (M <= 0 || N <= 0) return;
  // Below 4096 16 x 16 tiles (Hermitian: counting the upper ones) the form without staging is the faster one
  // (768^3: 74 against 98 us), above it the 32 x 32 tiles, which read half as much (1024^3: 172 us both;
  // Hermitian 1536 x 512: 156 against 174 us).
  const dim3 grid((N + GT - 1) / GT, (M + GT - 1) / GT), sgrid((N + ST - 1) / ST, (M + ST - 1) / ST);
  const bool small = (herm ? (long)sgrid.x * (sgrid.x + 1) / 2 : (long)sgrid.x * sgrid.y) < 4096;
#define GC_ZGEMM(OA, OB)                                                                                         \
  do {                                                                                                           \
    if (small)                                                                                                   \
      hipLaunchKernelGGL((k_zgemm_s<OA, OB>), sgrid, dim3(512), 0, s, M, N, K, A, lda, B, ldb, C, ldc, alpha,    \
                         accumulate, herm);                                                                      \
    else                                                                                                         \
      hipLaunchKernelGGL((k_zgemm<OA, OB>), grid, dim3(256), 0, s, M, N, K, A, lda, B, ldb, C, ldc, alpha,       \
                         accumulate, herm);                                                                      \
  } while (0)
  if (opa == 0 && opb == 0)
    GC_ZGEMM(0, 0);
  else if (opa == 0 && opb == 1)
    GC_ZGEMM(0, 1);
  else if (opa == 1 && opb == 0)
    GC_ZGEMM(1, 0);
  else
    GC_ZGEMM(1, 1);
#undef GC_ZGEMM
  GC_LAUNCH_CHECK();
}

void eig_hermitian(hipStream_t s, const z64* G, int m, int ldg, z64* U, int ldu, double* lam, int rel, EigWork& w,
                   DevStatus* st, int* host_sweeps, double discardable) {
  const JacobiCrit cr = jacobi_crit(m, rel);
  const double tol = cr.tol, skip = cr.skip_rel, floor_rel = cr.floor_rel;
  const int max_sweeps = cr.max_sweeps;
  if (m <= kSmallEig) {
#define GC_JSMALL(HM, REL)                                                                                           \
  hipLaunchKernelGGL((k_jacobi_small<HM, REL>), dim3(1), dim3(2 * HM * HM), 0, s, G, ldg, m, U, ldu, lam, cr, st)
    if (m <= 16 && rel)
      GC_JSMALL(8, true);
    else if (m <= 16)
      GC_JSMALL(8, false);
    else if (rel)
      GC_JSMALL(16, true);
    else
      GC_JSMALL(16, false);
#undef GC_JSMALL
    GC_LAUNCH_CHECK();
    if (host_sweeps) *host_sweeps = -1;
    return;
  }
  const int mp = ((m + BJ2 - 1) / BJ2) * BJ2;
  const int nb = mp / BJ;
  GC_CHECK(mp <= w.m_pad, GCAMPS_ECAPACITY, "eigensolver workspace too small");
  z64* Gp = w.G;
  z64* Up = w.G + (size_t)w.m_pad * w.m_pad;
  z64* Gp1 = w.G + 2 * (size_t)w.m_pad * w.m_pad;
  hipLaunchKernelGGL(k_pad_copy, dim3(blocks_for((size_t)mp * mp, 256)), dim3(256), 0, s, G, m, ldg, Gp, mp, Up);
  GC_LAUNCH_CHECK();
  double* d_trace = reinterpret_cast<double*>(w.flags + 512);
  int* sweep_flags = w.flags + 300;  // rotation flag of each sweep, cleared by k_trace
  GC_CHECK(max_sweeps < kSweepFlags, GCAMPS_ECAPACITY, "more sweeps than rotation flags");
  hipLaunchKernelGGL(k_trace, dim3(1), dim3(256), 0, s, Gp, m, mp, d_trace, sweep_flags);
  GC_LAUNCH_CHECK();
  if (discardable >= 0.0) {
    GC_CHECK(!rel, GCAMPS_EINVAL, "eigensolver: the pre-check has the absolute criterion only");
    hipLaunchKernelGGL(k_offdiag_check, dim3(blocks_for((size_t)m * m, 256)), dim3(256), 0, s, Gp, m, mp, d_trace, tol,
                       discardable, reinterpret_cast<int*>(d_trace + 1));
    GC_LAUNCH_CHECK();
    // the flag sits after the trace; the rounds read the trace themselves
    double* tr_flag = w.host_rb;
    GC_HIP(hipMemcpyAsync(tr_flag, d_trace, 2 * sizeof(double), hipMemcpyDeviceToHost, s));
    GC_HIP(hipStreamSynchronize(s));
    int pre_hit = 1;
    std::memcpy(&pre_hit, &tr_flag[1], sizeof(int));
    if (!pre_hit) {  // nothing to rotate: U = I (set by k_pad_copy), lam = diag(G)
      hipLaunchKernelGGL(k_unpad, dim3(blocks_for((size_t)m * m, 256)), dim3(256), 0, s, Gp, Up, m, mp, U, ldu,
                         lam);
      GC_LAUNCH_CHECK();
      if (host_sweeps) *host_sweeps = 0;
      return;
    }
  }
  const int half = nb / 2;
  int sweeps = 0;
  bool conv = false;
  // rotation, solved-sub-problem and flag buffers of round r: V and D + (r & 1) * half * 32 * 32,
  // flags + 1 + (r & 1) * 128 (half <= m_pad / 32 <= 128; the V and D regions hold m_pad / 16 blocks of
  // 32 x 32 and more)
  GC_CHECK(half <= 128, GCAMPS_ECAPACITY, "eigensolver: matrix side exceeds 4096");
  auto vbuf = [&](long r) { return w.V + (size_t)(r & 1) * half * BJ2 * BJ2; };
  auto dbuf = [&](long r) { return w.D + (size_t)(r & 1) * half * BJ2 * BJ2; };
  auto fbuf = [&](long r) { return w.flags + 1 + (r & 1) * 128; };
  // the matrix after round r - 1's update lives in gbuf(r): round r (r >= 1) solves from gbuf(r - 1)
  // and the previous round's rotations while it writes gbuf(r)
  auto gbuf = [&](long r) { return (r & 1) ? Gp1 : Gp; };
  auto tile_blocks = [](int tiles) { return (tiles + kTilesPerBlock - 1) / kTilesPerBlock; };
  const int gtiles = tile_blocks(half * (half + 1) / 2), utiles = tile_blocks((mp / BJ2) * half);
  // a whole CU per block while the tile updates are few (see k_jround)
  const size_t pad = mp <= kPadMaxM ? kJroundPad : 0;
  // A sweep is launched before the host knows whether the one before it rotated anything: its first round
  // reports that, and if nothing was rotated it does nothing (prev_any).  So the queue never runs dry, where a
  // read-back of the flags left it empty for 15 us after every one or two sweeps; the sweep too many
  // costs 3 us a round.
  long round = 0;  // rounds launched so far
  int prev_step = -1;
  auto sweep = [&](int sw) {
    for (int step = 0; step < nb - 1; ++step, ++round) {
      const bool upd = round > 0, tell = sw > 0 && step == 0;
      if (tell) ++*w.ticket;
#define GC_JROUND(REL)                                                                                               \
  hipLaunchKernelGGL((k_jround<REL>), dim3(half + (upd ? gtiles + utiles : 0)), dim3(kSolveThreads), pad, s,         \
                     upd ? gbuf(round - 1) : Gp, gbuf(round), Up, mp, nb, step, upd ? prev_step : -1, d_trace, tol,  \
                     skip, floor_rel, vbuf(round), dbuf(round), fbuf(round), sweep_flags + sw,                       \
                     sw > 0 ? sweep_flags + sw - 1 : nullptr, upd ? vbuf(round - 1) : nullptr,                       \
                     upd ? dbuf(round - 1) : nullptr, upd ? fbuf(round - 1) : nullptr, tell ? w.report_dev : nullptr, \
                     *w.ticket)
      if (rel)
        GC_JROUND(true);
      else
        GC_JROUND(false);
#undef GC_JROUND
      GC_LAUNCH_CHECK();
      prev_step = step;
    }
  };
  sweep(0);
  while (!conv && sweeps < max_sweeps) {
    sweep(++sweeps);
    await_ticket(s, w.report->ticket, *w.ticket);
    conv = w.report->rotated == 0;
  }
  // The last sweep rotated nothing, so its last round has nothing to apply: the matrix is what that
  // round's launch wrote.
  const z64* Gf = gbuf((long)sweeps * (nb - 1) - 1);
  hipLaunchKernelGGL(k_unpad, dim3(blocks_for((size_t)m * m, 256)), dim3(256), 0, s, Gf, Up, m, mp, U, ldu, lam);
  GC_LAUNCH_CHECK();
  GC_CHECK(conv, GCAMPS_ENUMERIC,
           std::string("block Jacobi eigensolver did not converge (m = ") + std::to_string(m) +
               (rel ? ", relative-accuracy pass)" : ", first pass)"));
  if (host_sweeps) *host_sweeps = sweeps;
}

void launch_rownorm2(hipStream_t s, const z64* B, int m, int k, int ldb, double* out) {
  if (m <= 0) return;
  hipLaunchKernelGGL(k_rownorm2, dim3(m), dim3(256), 0, s, B, m, k, ldb, out);
  GC_LAUNCH_CHECK();
}

void launch_trunc(hipStream_t s, const double* sig2, int m, double cutoff, int chi_max, int mode, int force_k,
                  int* perm, double* sig_sorted, DevStatus* st, const double* extra) {
  GC_CHECK(m <= TRUNC_MAX, GCAMPS_ECAPACITY, "truncation: matrix side exceeds 4096");
  hipLaunchKernelGGL(k_trunc, dim3(1), dim3(1024), 0, s, sig2, m, cutoff, chi_max, mode, force_k, perm, sig_sorted,
                     st, extra);
  GC_LAUNCH_CHECK();
}

void launch_emit(hipStream_t s, int wide, int left_ortho, int renorm, int p, int q, int kept, const z64* U, int ldu,
                 const z64* B, int ldb, const int* perm, const double* sig, z64* L, z64* R) {
  size_t total = (size_t)p * kept + (size_t)kept * q;
  hipLaunchKernelGGL(k_emit, dim3(blocks_for(total, 256)), dim3(256), 0, s, wide, left_ortho, renorm, p, q, kept, U,
                     ldu, B, ldb, perm, sig, L, R);
  GC_LAUNCH_CHECK();
}

void launch_copy(hipStream_t s, z64* dst, const z64* src, size_t count) {
  if (!count) return;
  hipLaunchKernelGGL(k_copy, dim3(blocks_for(count, 256)), dim3(256), 0, s, dst, src, count);
  GC_LAUNCH_CHECK();
}

void launch_fill_identity(hipStream_t s, z64* U, int m, int ld) {
  hipLaunchKernelGGL(k_fill_identity, dim3(blocks_for((size_t)m * m, 256)), dim3(256), 0, s, U, m, ld);
  GC_LAUNCH_CHECK();
}

}  // namespace gc
