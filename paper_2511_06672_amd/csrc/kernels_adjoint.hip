// Kernels of the reverse sweep (gradient of an observable with respect to phase-gate angles).
//
// Adjoint convention: for a real loss L and a complex array X, Xbar = dL/d conj(X), so that
// dL = 2 Re sum conj(Xbar) dX.  The dense products of the reverse sweep use the GEMM of
// kernels_linalg; the kernels here are the elementwise and reduction steps around them:
// * factorisation adjoint helpers (the sorted basis, gauge scalings, the renormalisation
//   projection, the kept/discarded mixing matrix);
// * the transpose of the MPO site map and the gradient of its coefficients;
// * Q^dagger applied to a two-site tensor.
#include "kernels.h"

namespace gc {

namespace {

inline unsigned nblocks(size_t n, int bs) { return (unsigned)((n + bs - 1) / bs); }

// Deterministic single-block sum of 1024 per-thread partials (fixed tree order).
__device__ double block_sum(double v, double* red) {
  const int t = threadIdx.x;
  red[t] = v;
  __syncthreads();
  for (int s = blockDim.x / 2; s > 0; s >>= 1) {
    if (t < s) red[t] += red[t + s];
    __syncthreads();
  }
  const double r = red[0];
  __syncthreads();
  return r;
}

// X = (base - X) / (sig[c]^2 rn^2) (by_cols; sig[r] otherwise) with rn = 1 / sqrt(sum_{j<k} sig_j^2), or 1
// when !renorm, also left in *rnp.  Every workgroup sums the k values itself: the sum, the copy of base and the scaling
// were a launch each, of 2.6, 1.7 and 1.7 us with the gaps between them.
__global__ __launch_bounds__(256) void k_gauge(z64* __restrict__ X, const z64* __restrict__ base, int rows, int cols,
                                               int by_cols, const double* __restrict__ sig, int k, int renorm,
                                               double* __restrict__ rnp) {
  __shared__ double red[256];
  const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
  const bool mine = idx < (size_t)rows * cols;
  z64 x = {0.0, 0.0};
  double s = 1.0;
  if (mine) {
    x = csub(base[idx], X[idx]);
    s = sig[by_cols ? idx % cols : idx / cols];
  }
  double v = 0.0;
  for (int j = threadIdx.x; j < k; j += 256) v += sig[j] * sig[j];
  const double tot = block_sum(v, red);
  const double rn = renorm ? 1.0 / sqrt(tot) : 1.0;
  if (idx == 0) rnp[0] = rn;
  if (mine) X[idx] = cscale(x, 1.0 / (s * s * rn * rn));
}

// out[0] = Re sum conj(a) b
__global__ __launch_bounds__(1024) void k_dot_re(const z64* __restrict__ a, const z64* __restrict__ b, size_t count,
                                                 double* __restrict__ out) {
  __shared__ double red[1024];
  double v = 0.0;
  for (size_t i = threadIdx.x; i < count; i += blockDim.x) v += a[i].re * b[i].re + a[i].im * b[i].im;
  const double tot = block_sum(v, red);
  if (threadIdx.x == 0) out[0] = tot;
}

// Xbar = rn (Nbar - N dot)
__global__ void k_renorm_bwd(const z64* __restrict__ Nbar, const z64* __restrict__ N, size_t count,
                             const double* __restrict__ rnp, const double* __restrict__ dotp, z64* __restrict__ Xbar) {
  size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= count) return;
  const double rn = rnp[0], dt = dotp[0];
  Xbar[idx] = cscale(csub(Nbar[idx], cscale(N[idx], dt)), rn);
}

// Both of the above in one workgroup, the entries in registers between them.
constexpr int kRenormPer = 8;
__global__ __launch_bounds__(1024) void k_renorm_bwd_small(const z64* __restrict__ Nbar, const z64* __restrict__ N,
                                                           int count, const double* __restrict__ rnp,
                                                           z64* __restrict__ Xbar) {
  __shared__ double red[1024];
  z64 a[kRenormPer], b[kRenormPer];
  double v = 0.0;
#pragma unroll
  for (int u = 0; u < kRenormPer; ++u) {
    const int i = threadIdx.x + u * 1024;
    a[u] = b[u] = z64{0.0, 0.0};
    if (i < count) {
      a[u] = N[i];
      b[u] = Nbar[i];
    }
    v += a[u].re * b[u].re + a[u].im * b[u].im;
  }
  const double dt = block_sum(v, red), rn = rnp[0];
#pragma unroll
  for (int u = 0; u < kRenormPer; ++u) {
    const int i = threadIdx.x + u * 1024;
    if (i < count) Xbar[i] = cscale(csub(b[u], cscale(a[u], dt)), rn);
  }
}

// A factorisation's basis as the reverse sweep wants it, in the sorted order: Us[r][a] = U[r][perm[a]] (m x m),
// Bs[a][c] = B[perm[a]][c] (m x kW) and the values sig.
__global__ void k_record(const z64* __restrict__ U, const z64* __restrict__ B, const double* __restrict__ sig,
                         const int* __restrict__ perm, int m, int kW, z64* __restrict__ Us, z64* __restrict__ Bs,
                         double* __restrict__ ss) {
  size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx < (size_t)m) ss[idx] = sig[idx];
  const size_t mm = (size_t)m * m;
  if (idx < mm) {
    Us[idx] = U[idx / m * m + perm[idx % m]];
  } else if (idx < mm + (size_t)m * kW) {
    idx -= mm;
    Bs[idx] = B[(size_t)perm[idx / kW] * kW + idx % kW];
  }
}

// Mixing of kept (index < k) and discarded rows in the sorted basis:
//   Zc[a][b] = (G1[a][b] + conj(G1[b][a])) / (s_kept^2 - s_discarded^2)  when exactly one of a, b < k,
// 0 otherwise (and 0 on an exact tie, where the derivative of the split does not exist).
// The rows >= k of Y (m x kW) are cleared on the way: what stays of it is the kept part.
__global__ void k_trunc_mix(const z64* __restrict__ G1, int m, int k, const double* __restrict__ sig,
                            z64* __restrict__ Zc, z64* __restrict__ Y, int kW) {
  size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx < (size_t)(m - k) * kW) Y[(size_t)k * kW + idx] = z64{0.0, 0.0};
  if (idx >= (size_t)m * m) return;
  const int a = (int)(idx / m), b = (int)(idx % m);
  z64 v = {0.0, 0.0};
  if ((a < k) != (b < k)) {
    const int kept = a < k ? a : b, disc = a < k ? b : a;
    const double delta = sig[kept] * sig[kept] - sig[disc] * sig[disc];
    if (delta > 0.0) v = cscale(cadd(G1[idx], cconj(G1[(size_t)b * m + a])), 1.0 / delta);
  }
  Zc[idx] = v;
}

// Transpose of the MPO site map k_mpo_site: in_bar[al, src, be] from out_bar.  Term b of the
// map sends in[al, src, be] to out[., (src + b dx) mod d, .] with weight K_b^{[kind 0,3]}
// omega^{(b dz) src}.
__global__ void k_mpo_site_bwd(int kind, int d, int chil, int chir, int dx, int dz, MpoCoeff co,
                               const z64* __restrict__ obar, z64* __restrict__ ibar) {
  size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  size_t total = (size_t)chil * d * chir;
  if (idx >= total) return;
  const int be = (int)(idx % chir);
  const int src = (int)((idx / chir) % d);
  const int al = (int)(idx / ((size_t)chir * d));
  const int orr = (kind == 0 || kind == 1) ? d * chir : chir;
  z64 acc = {0.0, 0.0};
  for (int b = 0; b < d; ++b) {
    const int a = (b * dx) % d, c = (b * dz) % d;
    const int s = (src + a) % d;
    z64 wgt = co.w[(c * src) % d];
    if (kind == 0 || kind == 3) wgt = cmul(co.k[b], wgt);
    size_t o;
    if (kind == 3)
      o = ((size_t)al * d + s) * orr + be;
    else if (kind == 0)
      o = ((size_t)al * d + s) * orr + (size_t)b * chir + be;
    else if (kind == 2)
      o = ((size_t)(b * chil + al) * d + s) * orr + be;
    else
      o = ((size_t)(b * chil + al) * d + s) * orr + (size_t)b * chir + be;
    acc = cadd(acc, cmulc(wgt, obar[o]));
  }
  ibar[idx] = acc;
}

// Gradient of the MPO coefficients at the first site (kind 0) or of a one-site MPO (kind 3):
//   Kbar_b = sum_e out_bar[e] conj(term_b[e]),  term_b = omega^{(b dz) src} in[al, src, be].
__global__ __launch_bounds__(1024) void k_mpo_coeff_bwd(int kind, int d, int chil, int chir, int dx, int dz,
                                                        MpoCoeff co, const z64* __restrict__ in,
                                                        const z64* __restrict__ obar, z64* __restrict__ kbar) {
  __shared__ double red[1024];
  double accr[kMaxD], acci[kMaxD];
  for (int b = 0; b < kMaxD; ++b) accr[b] = acci[b] = 0.0;
  const size_t total = (size_t)chil * d * chir;
  const int orr = (kind == 0) ? d * chir : chir;
  for (size_t idx = threadIdx.x; idx < total; idx += blockDim.x) {
    const int be = (int)(idx % chir);
    const int src = (int)((idx / chir) % d);
    const int al = (int)(idx / ((size_t)chir * d));
    const z64 v = in[idx];
    for (int b = 0; b < d; ++b) {
      const int a = (b * dx) % d, c = (b * dz) % d;
      const int s = (src + a) % d;
      const z64 term = cmul(co.w[(c * src) % d], v);
      const size_t o = (kind == 0) ? ((size_t)al * d + s) * orr + (size_t)b * chir + be
                                   : ((size_t)al * d + s) * orr + be;
      const z64 pr = cmulc(term, obar[o]);  // conj(term) * obar
      accr[b] += pr.re;
      acci[b] += pr.im;
    }
  }
  for (int b = 0; b < d; ++b) {
    const double r = block_sum(accr[b], red);
    const double i = block_sum(acci[b], red);
    if (threadIdx.x == 0) kbar[b] = z64{r, i};
  }
}

// A site operator |t> -> w_t |t + shift> on a site tensor, from the bra's side and back onto it.
__global__ void k_site_gather(int d, int chil, int chir, int shift, SitePhases w, const z64* __restrict__ in,
                              z64* __restrict__ out) {
  const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (size_t)chil * d * chir) return;
  const int b = (int)(idx % chir), t = (int)((idx / chir) % d);
  const size_t al = idx / ((size_t)chir * d);
  out[idx] = cmulc(w.w[t], in[(al * d + (t + shift) % d) * chir + b]);
}
__global__ void k_site_scatter(int d, int chil, int chir, int shift, SitePhases w, z64 cf, const z64* __restrict__ X,
                               z64* __restrict__ abar) {
  const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (size_t)chil * d * chir) return;
  const int b = (int)(idx % chir), t = (int)((idx / chir) % d);
  const size_t al = idx / ((size_t)chir * d), o = (al * d + (t + shift) % d) * chir + b;
  abar[o] = cadd(abar[o], cmul(cmul(cf, w.w[t]), X[idx]));
}

// theta <- Q_c^dagger theta on the physical pair of a (chil, d, d, chir) tensor.
__global__ void k_apply_qh(int d, int chil, int chir, int c, const z64* __restrict__ qm, z64* __restrict__ theta) {
  size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (size_t)chil * chir) return;
  const int a = (int)(idx / chir), b = (int)(idx % chir);
  const int D2 = d * d;
  const z64* q = qm + (size_t)c * D2 * D2;
  z64 v[kMaxD * kMaxD];
  for (int x = 0; x < D2; ++x) v[x] = theta[((size_t)a * D2 + x) * chir + b];
  for (int y = 0; y < D2; ++y) {
    z64 acc = {0.0, 0.0};
    for (int x = 0; x < D2; ++x) acc = cadd(acc, cmulc(q[x * D2 + y], v[x]));
    theta[((size_t)a * D2 + y) * chir + b] = acc;
  }
}

}  // namespace

void launch_gauge(hipStream_t s, z64* X, const z64* base, int rows, int cols, int by_cols, const double* sig, int k,
                  int renorm, double* rn) {
  hipLaunchKernelGGL(k_gauge, dim3(nblocks((size_t)rows * cols, 256)), dim3(256), 0, s, X, base, rows, cols, by_cols,
                     sig, k, renorm, rn);
  GC_LAUNCH_CHECK();
}
void launch_renorm_bwd(hipStream_t s, const z64* Nbar, const z64* N, size_t count, double* scal, z64* Xbar) {
  // one workgroup reads its 8192 entries in one go; more of them are left to the whole chip after the sum
  if (count <= (size_t)1024 * kRenormPer) {
    hipLaunchKernelGGL(k_renorm_bwd_small, dim3(1), dim3(1024), 0, s, Nbar, N, (int)count, scal, Xbar);
  } else {
    hipLaunchKernelGGL(k_dot_re, dim3(1), dim3(1024), 0, s, N, Nbar, count, scal + 1);
    hipLaunchKernelGGL(k_renorm_bwd, dim3(nblocks(count, 256)), dim3(256), 0, s, Nbar, N, count, scal, scal + 1, Xbar);
  }
  GC_LAUNCH_CHECK();
}
void launch_record(hipStream_t s, const z64* U, const z64* B, const double* sig, const int* perm, int m, int kW, z64* Us,
                   z64* Bs, double* ss) {
  hipLaunchKernelGGL(k_record, dim3(nblocks((size_t)m * (m + kW), 256)), dim3(256), 0, s, U, B, sig, perm, m, kW, Us, Bs,
                     ss);
  GC_LAUNCH_CHECK();
}
void launch_trunc_mix(hipStream_t s, const z64* G1, int m, int k, const double* sig, z64* Zc, z64* Y, int kW) {
  const size_t total = std::max((size_t)m * m, (size_t)(m - k) * kW);
  hipLaunchKernelGGL(k_trunc_mix, dim3(nblocks(total, 256)), dim3(256), 0, s, G1, m, k, sig, Zc, Y, kW);
  GC_LAUNCH_CHECK();
}
void launch_mpo_site_bwd(hipStream_t s, int kind, int d, int chil, int chir, int dx, int dz, const MpoCoeff& co,
                         const z64* obar, z64* ibar) {
  size_t total = (size_t)chil * d * chir;
  hipLaunchKernelGGL(k_mpo_site_bwd, dim3(nblocks(total, 256)), dim3(256), 0, s, kind, d, chil, chir, dx, dz, co,
                     obar, ibar);
  GC_LAUNCH_CHECK();
}
void launch_mpo_coeff_bwd(hipStream_t s, int kind, int d, int chil, int chir, int dx, int dz, const MpoCoeff& co,
                          const z64* in, const z64* obar, z64* kbar) {
  hipLaunchKernelGGL(k_mpo_coeff_bwd, dim3(1), dim3(1024), 0, s, kind, d, chil, chir, dx, dz, co, in, obar, kbar);
  GC_LAUNCH_CHECK();
}
void launch_site_gather(hipStream_t s, int d, int chil, int chir, int shift, const SitePhases& w, const z64* in, z64* out) {
  const size_t total = (size_t)chil * d * chir;
  hipLaunchKernelGGL(k_site_gather, dim3(nblocks(total, 256)), dim3(256), 0, s, d, chil, chir, shift, w, in, out);
  GC_LAUNCH_CHECK();
}
void launch_site_scatter(hipStream_t s, int d, int chil, int chir, int shift, const SitePhases& w, z64 cf, const z64* X,
                         z64* abar) {
  const size_t total = (size_t)chil * d * chir;
  hipLaunchKernelGGL(k_site_scatter, dim3(nblocks(total, 256)), dim3(256), 0, s, d, chil, chir, shift, w, cf, X, abar);
  GC_LAUNCH_CHECK();
}
void launch_apply_qh(hipStream_t s, int d, int chil, int chir, int c, const z64* qmats, z64* theta) {
  size_t total = (size_t)chil * chir;
  hipLaunchKernelGGL(k_apply_qh, dim3(nblocks(total, 128)), dim3(128), 0, s, d, chil, chir, c, qmats, theta);
  GC_LAUNCH_CHECK();
}

}  // namespace gc
