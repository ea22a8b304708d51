// Candidate scoring through the two-site reduced density matrix (§3: the Rényi-2 entropy of Q_c Theta), for
// d = 2 and 3.
//
// Theta(a, t, b), t = (t1 t2) in [0, D), D = d^2; x is the smaller bond (a or b), y the other.  With
//   F(x t, x' t') = sum_y Theta(x t y) conj Theta(x' t' y),
// which no candidate enters, the reduced density matrix of a cut is
//   rho_c(x s, x' s') = sum_{t t'} T_c(s s', t t') F(x t, x' t'),
//   T_c(s s', t t') = sum_r Q_c((s r), t) conj Q_c((s' r), t')   (left cut, x = a; r s swapped on the right),
// so every candidate's entries for every pair (x, x') are one matrix product: the pairs' d^4 values of
// F against the rows T_c, d^2 per candidate, which depend on the candidate set alone.  The purity
// sum |rho_c|^2 is summed as it is formed (pairs x < x' twice), nothing is stored, and rho_c is the same
// matrix as before: the sum over y is done first, once instead of per candidate.  A candidate costs
// 4 X^2 d^6 flop (8 per complex multiply-add, half of the pairs) instead of the 4 m^2 k of its Gram product,
// m = X d, k = Y d.
//
// k_density: a block stages the F values of 32 pairs in LDS and each of its four waves multiplies them
// by 32 rows T_c (from L2) on MFMA.  What bounds it: the MFMA pipe (m = 729, 512 candidates, FP64: about
// 65 of 78.6 TFLOP/s).  Three blocks per CU hide each other's staging and loads; 64 pairs per block (one
// block per CU) took 1.94 against 1.71 ms there, 48 or 64 rows per wave 2.0 and 2.1.
// Scores of one bond of 512 qutrit candidates, call to host values, from rotated matrices and now:
// FP64 m = 81 343 and 65 us, m = 243 1160 and 252, m = 729 17570 and 1714; FP32 193 and 55, 617 and 152,
// 6981 and 932.  720 qubit candidates, m = 512: FP64 8023 and 384, FP32 3234 and 279, BF16 mode 1565 and 278.  Errors against 64 bits are those of
// the rotated form (6e-16 at m = 243) and a third of them in FP32 (1.7e-8 against 5.2e-8).
#include <algorithm>

#include "kernels.h"

namespace gc {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));

namespace {

constexpr int PT = 32;         // pairs per block step
constexpr int CT = 2;          // 16-row tiles of T per wave
constexpr int kColsPerBlock = 4 * CT * 16;
constexpr int kDensityBlocks = 768;

template <int DD>
struct Dim {
  static constexpr int D = DD * DD, S = DD * DD, K = D * D, KP = (K + 3) / 4 * 4;
};

__device__ __forceinline__ d4 mfma_t(double a, double b, d4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f4 mfma_t(float a, float b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
template <typename T>
struct Acc;
template <>
struct Acc<double> {
  typedef d4 type;
};
template <>
struct Acc<float> {
  typedef f4 type;
};

// One thread per (candidate, s s', k): the rows T_c of both cuts, zero beyond k = d^4.
template <int DD>
__global__ __launch_bounds__(256) void k_density_maps(int count, const z64* __restrict__ qm, z64* __restrict__ tab,
                                                      c32* __restrict__ tab32) {
  constexpr int D = Dim<DD>::D, S = Dim<DD>::S, K = Dim<DD>::K, KP = Dim<DD>::KP;
  const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x, per = (size_t)count * S * KP;
  if (e >= 2 * per) return;
  const bool left = e < per;
  const size_t r = left ? e : e - per;
  const int k = (int)(r % KP), ss = (int)(r / KP % S), c = (int)(r / KP / S);
  const int s = ss / DD, sp = ss % DD, t = k / D, tp = k % D;
  const z64* q = qm + (size_t)c * D * D;
  z64 acc = {0.0, 0.0};
  if (k < K)
    for (int o = 0; o < DD; ++o) {
      const int r1 = left ? s * DD + o : o * DD + s, r2 = left ? sp * DD + o : o * DD + sp;
      acc = cadd(acc, cmul(q[r1 * D + t], cconj(q[r2 * D + tp])));
    }
  tab[e] = acc;
  if (tab32) tab32[e] = c32{(float)acc.re, (float)acc.im};
}

// Pair (x, x') with x <= x' from its rank p in row-major order of the upper triangle.
__device__ __forceinline__ void unrank_pair(long long p, int X, int& x, int& xp) {
  const double b = 2.0 * X + 1.0;
  int g = (int)floor((b - sqrt(b * b - 8.0 * (double)p)) * 0.5);
  g = max(0, min(g, X - 1));
  auto off = [X](long long r) { return r * X - r * (r - 1) / 2; };
  while (g > 0 && off(g) > p) --g;
  while (g + 1 < X && off(g + 1) <= p) ++g;
  x = g;
  xp = g + (int)(p - off(g));
}

// partial[blockIdx.x][0][n] = sum over the block's pairs of w |rho|^2 for column n = (slot, s s'), and
// [1][n] the block's part of the trace (x = x', s = s'; taken from rho_c itself, so that what rounding
// leaves of Q_c's norm cancels in the score).  F: (X D) x (X D), entry (x t, x' t') at (x D + t) ld + x' D + t'
// when left, else the conjugate at (t X + x) ld + t' X + x'.  A block takes the pair tiles blockIdx.x,
// + gridDim.x, ... and, for each tile once staged, the column groups blockIdx.y, + gridDim.y, ...
// FP32 forms a complex product from three real ones (re = T1 - T2, im = T3 - T1 - T2 with
// T3 = (ar + ai)(br + bi)), FP64 from four.
template <typename T, int DD>
__global__ __launch_bounds__(256, 3) void k_density(int X, const z64* __restrict__ F, int ld, int left, long long npairs,
                                                 const int* __restrict__ list, const int* __restrict__ nlimit,
                                                 int count, const cx<T>* __restrict__ tab,
                                                 double* __restrict__ partial) {
  constexpr int D = Dim<DD>::D, S = Dim<DD>::S, K = Dim<DD>::K, KP = Dim<DD>::KP, LD = KP + 1, RT = PT / 16;
  constexpr bool M3 = sizeof(T) == 4;
  typedef typename Acc<T>::type acc_t;
  __shared__ __align__(16) cx<T> fs[PT * LD];
  __shared__ double wgt[PT];
  __shared__ int px[PT], pxp[PT];
  const int lim = nlimit ? min(*nlimit, count) : count;
  const int cols = lim * S, groups = (cols + kColsPerBlock - 1) / kColsPerBlock;
  if ((int)blockIdx.y >= groups) return;  // uniform over the block
  const int t = threadIdx.x, lane = t & 63, lo = lane & 15, hi = lane >> 4, wv = t >> 6;
  double* out = partial + (size_t)blockIdx.x * 2 * count * S;
  const long long ntiles = (npairs + PT - 1) / PT;
  for (long long pt = blockIdx.x; pt < ntiles; pt += gridDim.x) {
    if (t < PT) {
      const long long p = pt * PT + t;
      int x = 0, xp = 0;
      if (p < npairs) unrank_pair(p, X, x, xp);
      px[t] = x;
      pxp[t] = xp;
      wgt[t] = p < npairs ? (x == xp ? 1.0 : 2.0) : 0.0;
    }
    __syncthreads();
#pragma unroll 7
    for (int e = t; e < PT * KP; e += 256) {
      // left: runs of t' along a row of F; right: runs of pairs (mostly consecutive x')
      const int i = left ? e / KP : e % PT, k = left ? e % KP : e / PT;
      cx<T> v = {T(0), T(0)};
      if (k < K) {
        const int a = k / D, b = k % D;
        const z64 f = left ? F[(size_t)(px[i] * D + a) * ld + pxp[i] * D + b]
                           : F[(size_t)(a * X + px[i]) * ld + b * X + pxp[i]];
        v = cx<T>{T(f.re), T(left ? f.im : -f.im)};
      }
      fs[i * LD + k] = v;
    }
    __syncthreads();
    for (int g = blockIdx.y; g < groups; g += gridDim.y) {
      const cx<T>* rowp[CT];
      int col[CT];
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) {
        col[ct] = g * kColsPerBlock + (wv * CT + ct) * 16 + lo;
        const int n = min(col[ct], cols - 1), slot = n / S;
        const int c = list ? list[slot] : slot;
        rowp[ct] = tab + ((size_t)c * S + n % S) * KP + hi;
      }
      acc_t ar[RT][CT], ai[RT][CT], a3[M3 ? RT : 1][CT];
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) ar[rt][ct] = ai[rt][ct] = a3[M3 ? rt : 0][ct] = acc_t{0, 0, 0, 0};
      cx<T> b[CT], bn[CT];
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) b[ct] = rowp[ct][0];
#pragma unroll 3
      for (int k = 0; k < KP; k += 4) {
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) bn[ct] = rowp[ct][k + 4 < KP ? k + 4 : k];  // next step's rows
        cx<T> a[RT];
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) a[rt] = fs[(16 * rt + lo) * LD + k + hi];
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
          for (int ct = 0; ct < CT; ++ct) {
            ar[rt][ct] = mfma_t(a[rt].re, b[ct].re, ar[rt][ct]);
            ai[rt][ct] = mfma_t(M3 ? a[rt].im : a[rt].re, b[ct].im, ai[rt][ct]);
          }
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
          for (int ct = 0; ct < CT; ++ct) {
            if (M3) {
              a3[M3 ? rt : 0][ct] = mfma_t(a[rt].re + a[rt].im, b[ct].re + b[ct].im, a3[M3 ? rt : 0][ct]);
            } else {
              ar[rt][ct] = mfma_t(-a[rt].im, b[ct].im, ar[rt][ct]);
              ai[rt][ct] = mfma_t(a[rt].im, b[ct].re, ai[rt][ct]);
            }
          }
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) b[ct] = bn[ct];
      }
      double psum[CT], tsum[CT];
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) psum[ct] = tsum[ct] = 0.0;
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const double w = wgt[16 * rt + mfma_row<T>(lane, q)];
#pragma unroll
          for (int ct = 0; ct < CT; ++ct) {
            const T x1 = ar[rt][ct][q], x2 = ai[rt][ct][q];
            const double re = M3 ? x1 - x2 : x1, im = M3 ? a3[M3 ? rt : 0][ct][q] - x1 - x2 : x2;
            psum[ct] += w * (re * re + im * im);
            tsum[ct] += w == 1.0 ? re : 0.0;
          }
        }
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) {
        double v = psum[ct], tr = tsum[ct];
        v += __shfl_xor(v, 16, 64);
        v += __shfl_xor(v, 32, 64);
        tr += __shfl_xor(tr, 16, 64);
        tr += __shfl_xor(tr, 32, 64);
        if (hi == 0 && col[ct] < cols) {  // this block's own entries: added up over its tiles
          double* o = out + col[ct];
          o[0] = pt == blockIdx.x ? v : o[0] + v;
          o[(size_t)count * S] = pt == blockIdx.x ? tr : o[(size_t)count * S] + tr;
        }
      }
    }
    __syncthreads();  // the stage is overwritten next
  }
}

// S2 of one candidate per block from the partial sums (columns with s = s', e % S a multiple of d + 1, hold the
// trace).
__global__ __launch_bounds__(64) void k_density_reduce(int d, int nblk, int count, const int* __restrict__ nlimit,
                                                       const double* __restrict__ partial, double* __restrict__ s2) {
  const int slot = blockIdx.x, t = threadIdx.x, S = d * d;
  if (slot >= (nlimit ? min(*nlimit, count) : count)) return;
  double p = 0.0, tr = 0.0;
  for (int e = t; e < nblk * S; e += 64) {
    const double* at = partial + (size_t)(e / S) * 2 * count * S + slot * S + e % S;
    p += at[0];
    if (e % S % (d + 1) == 0) tr += at[(size_t)count * S];
  }
  for (int off = 32; off > 0; off >>= 1) {
    p += __shfl_xor(p, off, 64);
    tr += __shfl_xor(tr, off, 64);
  }
  if (t == 0) s2[slot] = -log(p / (tr * tr));
}

constexpr size_t table_elems_of(int d, int count) {
  return 2 * (size_t)count * d * d * (d == 3 ? Dim<3>::KP : Dim<2>::KP);
}

}  // namespace

size_t density_table_elems(int d, int count) { return d <= 3 ? table_elems_of(d, count) : 0; }

void launch_density_tables(hipStream_t s, int d, int count, const z64* qmats, z64* tab, c32* tab32) {
  const unsigned blocks = (unsigned)((table_elems_of(d, count) + 255) / 256);
  if (d == 3)
    hipLaunchKernelGGL(k_density_maps<3>, dim3(blocks), dim3(256), 0, s, count, qmats, tab, tab32);
  else
    hipLaunchKernelGGL(k_density_maps<2>, dim3(blocks), dim3(256), 0, s, count, qmats, tab, tab32);
  GC_LAUNCH_CHECK();
}

bool density_fits(int d, int chil, int chir, int count, size_t scratch_bytes) {
  const size_t xd = (size_t)std::min(chil, chir) * d * d;
  return align256(xd * xd * sizeof(z64)) + (size_t)count * 2 * d * d * sizeof(double) <= scratch_bytes;
}

void launch_density_gram(hipStream_t s, int d, int chil, int chir, const z64* theta, void* scratch) {
  const int D = d * d, xd = std::min(chil, chir) * D;
  z64* F = reinterpret_cast<z64*>(scratch);
  const z64 one = {1.0, 0.0};
  if (chil <= chir)
    launch_zgemm(s, 0, 1, xd, xd, chir, theta, chir, theta, chir, F, xd, one, 0, 1);
  else  // columns (t b) of theta: the conjugate of F, the bond fastest
    launch_zgemm(s, 1, 0, xd, xd, chil, theta, xd, theta, xd, F, xd, one, 0, 1);
}

void launch_density_score(hipStream_t s, int d, bool fp32, int chil, int chir, const z64* tab, const c32* tab32,
                          int set_count, const int* list, int count, const int* nlimit, double* s2, void* scratch,
                          size_t scratch_bytes, hipEvent_t ev0, hipEvent_t ev1) {
  const bool left = chil <= chir;
  const int D = d * d, S = D, X = left ? chil : chir, xd = X * D;
  const z64* F = reinterpret_cast<const z64*>(scratch);
  const size_t fbytes = align256((size_t)xd * xd * sizeof(z64));
  double* partial = reinterpret_cast<double*>(reinterpret_cast<char*>(scratch) + fbytes);
  const long long npairs = (long long)X * (X + 1) / 2, ntiles = (npairs + PT - 1) / PT;
  // one pair tile per block where the partial sums fit, and column groups dealt to about three blocks per
  // CU in all (staging a tile costs as much as a quarter of a column group, so few groups per block waste
  // it); a list whose length is only known on the device is usually short and gets a block per group
  const size_t room = (scratch_bytes - fbytes) / ((size_t)count * 2 * S * sizeof(double));
  const int gx = (int)std::min<size_t>((size_t)ntiles, room);
  GC_CHECK(gx >= 1, GCAMPS_ECAPACITY, "density scoring scratch too small");
  const int groups = (count * S + kColsPerBlock - 1) / kColsPerBlock;
  const int gy = std::min(groups, std::max(1, (kDensityBlocks + gx - 1) / gx));
  const size_t side = left ? 0 : density_table_elems(d, set_count) / 2;
  if (ev0) GC_HIP(hipEventRecord(ev0, s));
#define GC_DENSITY(T, DD, TAB)                                                                                       \
  hipLaunchKernelGGL((k_density<T, DD>), dim3(gx, gy), dim3(256), 0, s, X, F, xd, left ? 1 : 0, npairs, list, nlimit, \
                     count, TAB + side, partial)
  if (d == 3 && fp32)
    GC_DENSITY(float, 3, tab32);
  else if (d == 3)
    GC_DENSITY(double, 3, tab);
  else if (fp32)
    GC_DENSITY(float, 2, tab32);
  else
    GC_DENSITY(double, 2, tab);
#undef GC_DENSITY
  GC_LAUNCH_CHECK();
  if (ev1) GC_HIP(hipEventRecord(ev1, s));
  hipLaunchKernelGGL(k_density_reduce, dim3(count), dim3(64), 0, s, d, gx, count, nlimit, partial, s2);
  GC_LAUNCH_CHECK();
}

}  // namespace gc
