// Exact moves of the orthogonality centre (§2.4) without an eigen-decomposition.
//
// A move M = L R that keeps every direction only needs one orthonormal factor, in any gauge.  With m
// the smaller side, W the wide orientation of M and G = W W^H = K K^H (Cholesky, blocks of 32
// columns), all pivots well above rounding say that M has full rank m.  Then
//   - the factor on the smaller side may be the identity: L = I, R = M (or L = M, R = I);
//   - the factor on the larger side is X K^-H with X the tall orientation: X's rows ride along below
//     G through the elimination (the panel solves divide them by K^H as they go), and two
//     Newton-Schulz steps remove the rounding that the condition number has amplified.
// The host falls back to the eigen-decomposition when a pivot is small (rank deficiency, or a
// spectrum too wide for the Gram) or X K^-H is too far from orthonormal for those two steps, by a bound of
// the norm of its defect: its largest entry may be m times smaller.
//
// The eigen-decomposition that a move took before ran 5 to 10 sweeps: per move (averaged over a qutrit
// circuit, device time) 0.63 ms at m = 81, 1.87 at 243 and 2.86 at 384, now 0.20, 0.43 and 0.72.  The
// splits that follow start from a basis that is no longer sorted by weight and take about a sweep
// more (11.8 against 10.5 at m = 243), a fifth of what the moves save.
//
// What bounds it: per 32 columns one panel launch, whose 32 pivot steps are a dependent chain (22 us),
// and one rank-32 update on MFMA.
#include <algorithm>

#include "jacobi.h"
#include "kernels.h"

namespace gc {

namespace {

constexpr int CB = 32;  // columns per panel

__global__ __launch_bounds__(256) void k_chol_init(const z64* __restrict__ G, int m, CholState* __restrict__ st) {
  __shared__ double red[256];
  double s = 0.0;
  for (int i = threadIdx.x; i < m; i += blockDim.x) s = fmax(s, G[(size_t)i * m + i].re);
  red[threadIdx.x] = s;
  __syncthreads();
  for (int off = 128; off > 0; off >>= 1) {
    if ((int)threadIdx.x < off) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + off]);
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    st->dmax = st->dmin = red[0];
    st->emax = 0.0;
  }
}

// Panel of columns j0..j0 + nb of A (rows x m, rows 0..m the Hermitian matrix, its lower part live).  Every
// block factors the diagonal block K K^H on its own (the same arithmetic in each), running the
// identity's rows through the same elimination, which turns them into K^-H, and then multiplies its
// 128 rows below by K^-H on MFMA.  Block 0 records the smallest pivot.  (One row per thread, by
// substitution from LDS, spilled registers: 130 us per panel.)
constexpr int kCholRows = 128;
__global__ __launch_bounds__(512) void k_chol_panel(z64* __restrict__ A, int lda, int rows, int j0, int nb,
                                                    CholState* __restrict__ st) {
  __shared__ __align__(16) z64 kinv[CB * CB];      // K^-H, row-major
  __shared__ __align__(16) z64 col[2][2][CB];      // [step parity][matrix, identity]: the pivot column
  __shared__ double piv[CB];
  const int t = threadIdx.x, k = t & 31, ib = t >> 5;
  const double dmax = st->dmax;
  z64 a[2], y[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) {  // elements (ib + 16 u, k); the identity times dmax beyond nb
    const int i = ib + 16 * u;
    a[u] = (i < nb && k < nb) ? A[(size_t)(j0 + i) * lda + j0 + k] : z64{i == k ? dmax : 0.0, 0.0};
    y[u] = z64{i == k ? 1.0 : 0.0, 0.0};
    if (k == 0) {
      col[0][0][i] = a[u];
      col[0][1][i] = y[u];
    }
  }
  __syncthreads();
  for (int j = 0; j < CB; ++j) {
    const z64* ca = col[j & 1][0];
    const z64* cy = col[j & 1][1];
    const double d0 = ca[j].re, d = d0 > 0.0 ? d0 : dmax;  // a pivot that is not positive: the host rejects
    if (t == 0) piv[j] = d0 > 0.0 ? d0 : 0.0;
    double r = __builtin_amdgcn_rcp(d);
    r = fma(fma(-d, r, 1.0), r, r);
    r = fma(fma(-d, r, 1.0), r, r);
    if (k > j) {  // element (i, k) -= (i, j) conj(k, j) / d
      const z64 f = cscale(cconj(ca[k]), r);
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int i = ib + 16 * u;
        a[u] = csub(a[u], cmul(ca[i], f));
        y[u] = csub(y[u], cmul(cy[i], f));
        if (k == j + 1) {
          col[(j + 1) & 1][0][i] = a[u];
          col[(j + 1) & 1][1][i] = y[u];
        }
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const double d = piv[k] > 0.0 ? piv[k] : dmax;
    kinv[(ib + 16 * u) * CB + k] = cscale(y[u], 1.0 / sqrt(d));
  }
  if (blockIdx.x == 0 && t < 64) {
    double v = t < nb ? piv[t] : dmax;
    for (int off = 32; off > 0; off >>= 1) v = fmin(v, __shfl_xor(v, off, 64));
    if (t == 0) st->dmin = fmin(st->dmin, v);
  }
  __syncthreads();
  const int lane = t & 63, lo = lane & 15, hi = lane >> 4;
  const int r0 = j0 + nb + blockIdx.x * kCholRows + (t >> 6) * 16;
  if (r0 >= rows) return;  // uniform over the wave, no barrier follows
  const bool live = r0 + lo < rows;
  z64 x[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int c = 4 * j + hi;
    x[j] = (live && c < nb) ? A[(size_t)(r0 + lo) * lda + j0 + c] : z64{0.0, 0.0};
  }
  d4 rr[2], ri[2];
#pragma unroll
  for (int ch = 0; ch < 2; ++ch) {
    rr[ch] = ri[ch] = d4{0, 0, 0, 0};
#pragma unroll
    for (int j = 0; j < 8; ++j) mma4(x[j], kinv[(4 * j + hi) * CB + 16 * ch + lo], rr[ch], ri[ch]);
  }
#pragma unroll
  for (int ch = 0; ch < 2; ++ch)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int row = r0 + mfma_row_f64(lane, q), c = 16 * ch + lo;
      if (row < rows && c < nb) A[(size_t)row * lda + j0 + c] = z64{rr[ch][q], ri[ch][q]};
    }
}

// Largest row sum of |S - I| (S m x m, Hermitian), a bound of its spectral norm, into st->emax; one workgroup
// per row, and a maximum over them, so that the result does not depend on their order.
__global__ __launch_bounds__(256) void k_identity_gap(const z64* __restrict__ S, int m, CholState* __restrict__ st) {
  __shared__ double part[4];
  const int i = blockIdx.x, t = threadIdx.x;
  double e = 0.0;
  for (int j = t; j < m; j += 256) {
    const z64 x = S[(size_t)i * m + j];
    e += fabs(x.re - (i == j ? 1.0 : 0.0)) + fabs(x.im);
  }
  for (int off = 32; off > 0; off >>= 1) e += __shfl_xor(e, off, 64);
  if ((t & 63) == 0) part[t >> 6] = e;
  __syncthreads();
  if (t != 0) return;
  e = part[0] + part[1] + part[2] + part[3];
  if (!(e < 1e30)) e = 1e30;  // NaN as well
  // non-negative doubles order as their bit patterns
  atomicMax(reinterpret_cast<unsigned long long*>(&st->emax), (unsigned long long)__double_as_longlong(e));
}

// dst (q x p) = src^H (src p x q).
__global__ __launch_bounds__(256) void k_conj_transpose(const z64* __restrict__ src, int p, int q,
                                                        z64* __restrict__ dst) {
  __shared__ z64 tile[32][33];
  const int p0 = blockIdx.y * 32, q0 = blockIdx.x * 32, tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  for (int i = ty; i < 32; i += 8)
    if (p0 + i < p && q0 + tx < q) tile[i][tx] = src[(size_t)(p0 + i) * q + q0 + tx];
  __syncthreads();
  for (int i = ty; i < 32; i += 8)
    if (q0 + i < q && p0 + tx < p) dst[(size_t)(q0 + i) * p + p0 + tx] = cconj(tile[tx][i]);
}

}  // namespace

void launch_cholesky(hipStream_t s, z64* A, int m, int rows, CholState* st) {
  GC_CHECK(m >= 1 && rows >= m, GCAMPS_EINVAL, "cholesky: fewer rows than columns");
  hipLaunchKernelGGL(k_chol_init, dim3(1), dim3(256), 0, s, A, m, st);
  GC_LAUNCH_CHECK();
  for (int j0 = 0; j0 < m; j0 += CB) {
    const int nb = std::min(CB, m - j0), j1 = j0 + nb;
    const int blocks = std::max(1, (rows - j1 + kCholRows - 1) / kCholRows);
    hipLaunchKernelGGL(k_chol_panel, dim3(blocks), dim3(512), 0, s, A, m, rows, j0, nb, st);
    GC_LAUNCH_CHECK();
    const z64* P = A + (size_t)j1 * m + j0;
    launch_zgemm(s, 0, 1, rows - j1, m - j1, nb, P, m, P, m, A + (size_t)j1 * m + j1, m, z64{-1.0, 0.0}, 1, 0);
  }
}

void launch_identity_gap(hipStream_t s, const z64* S, int m, CholState* st) {
  hipLaunchKernelGGL(k_identity_gap, dim3(m), dim3(256), 0, s, S, m, st);
  GC_LAUNCH_CHECK();
}

void launch_conj_transpose(hipStream_t s, const z64* src, int p, int q, z64* dst) {
  hipLaunchKernelGGL(k_conj_transpose, dim3((q + 31) / 32, (p + 31) / 32), dim3(256), 0, s, src, p, q, dst);
  GC_LAUNCH_CHECK();
}

}  // namespace gc
