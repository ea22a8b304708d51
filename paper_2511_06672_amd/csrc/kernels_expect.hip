// Expectation <psi| W |psi> = <m| P |m> of a Weyl operator: the commutation of W through the tableau and the
// chain of transfer matrices E' = sum_t w_t A_{t + x}^H (E A_t), w_t = omega^{z t}, over the MPS m.
#include "jacobi.h"
#include "kernels.h"
#include "weyl.h"

namespace gc {

namespace {

constexpr int kThreads = 512;
constexpr int kPerThread = kExpectMaxSite / kThreads;

// The sites [first, last) in one workgroup, E and the site tensors in LDS; the next site's tensor is read
// into registers while the current one is contracted.  Bound by latency: three barriers and the shortest
// MFMA chain (d chi / 4 steps of 256 cycles) a site.  As 2 d products a site on the whole chip a chain of
// small tensors is bound by its launches instead: n = 10, d = 3, bonds up to 9: 64 launches and three copies,
// 295 us a call against 57 us.
// LDS: E transposed ([col][row], so that an operand row of E is read along its columns) | A | T.
__global__ __launch_bounds__(kThreads) void k_expect_chain(ExpectArgs a, int e_elems, int a_elems) {
  extern __shared__ z64 lds[];
  __shared__ DevWeyl P;
  __shared__ WeylScratch ws;
  z64* const E = lds;
  z64* const A = lds + e_elems;
  z64* const T = A + a_elems;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int col = lane & 15, quad = lane >> 4;
  const int d = a.d;
  z64 nx[kPerThread];
  auto fetch = [&](int site) {
    const int count = a.chi[site] * d * a.chi[site + 1];
    const z64* src = a.site[site];
#pragma unroll
    for (int i = 0; i < kPerThread; ++i)
      if (t + i * kThreads < count) nx[i] = src[t + i * kThreads];
  };
  if (a.first < a.last) fetch(a.first);
  if (a.extract) {
    weyl_commute(a.n, d, a.tx, a.tz, a.tp, a.target, P, ws);
    if (a.weyl) {
      for (int i = t; i < (int)(sizeof(DevWeyl) / sizeof(int)); i += kThreads)
        reinterpret_cast<int*>(a.weyl)[i] = reinterpret_cast<const int*>(&P)[i];
    }
  } else {
    for (int i = t; i < (int)(sizeof(DevWeyl) / sizeof(int)); i += kThreads)
      reinterpret_cast<int*>(&P)[i] = reinterpret_cast<const int*>(a.weyl)[i];
  }
  const int c0 = a.chi[a.first];
  for (int i = t; i < c0 * c0; i += kThreads) E[(i % c0) * c0 + i / c0] = a.e_in ? a.e_in[i] : z64{1.0, 0.0};
  for (int s = a.first; s < a.last; ++s) {
    const int cl = a.chi[s], cr = a.chi[s + 1], N = d * cr, K = cl * d;
#pragma unroll
    for (int i = 0; i < kPerThread; ++i)
      if (t + i * kThreads < cl * N) A[t + i * kThreads] = nx[i];
    __syncthreads();
    if (s + 1 < a.last) fetch(s + 1);
    // T[(al, tt), b] = w_tt sum_be E[al][be] A[(be, tt), b]
    const int tr = (cl + 15) >> 4, tn = (N + 15) >> 4;
    for (int tile = w; tile < tr * tn; tile += kThreads / 64) {
      const int r0 = (tile / tn) * 16, n0 = (tile % tn) * 16;
      d4 cr_ = {0, 0, 0, 0}, ci_ = {0, 0, 0, 0};
      for (int k0 = 0; k0 < cl; k0 += 4) {
        const int k = k0 + quad;
        z64 x = {0, 0}, y = {0, 0};
        if (k < cl && r0 + col < cl) x = E[k * cl + r0 + col];
        if (k < cl && n0 + col < N) y = A[k * N + n0 + col];
        mma4(x, y, cr_, ci_);
      }
      const int nn = n0 + col;
      if (nn < N) {
        const double ang = 2.0 * M_PI * ((P.z[s] * (nn / cr)) % d) / d;
        const z64 f = {cos(ang), sin(ang)};
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (r0 + 4 * q + quad < cl) T[(r0 + 4 * q + quad) * N + nn] = cmul(f, z64{cr_[q], ci_[q]});
      }
    }
    __syncthreads();
    // E'[b'][b] = sum_{al, tt} conj(A[(al, tt + x), b']) T[(al, tt), b]
    const int tc = (cr + 15) >> 4;
    for (int tile = w; tile < tc * tc; tile += kThreads / 64) {
      const int r0 = (tile / tc) * 16, n0 = (tile % tc) * 16;
      d4 cr_ = {0, 0, 0, 0}, ci_ = {0, 0, 0, 0};
      for (int k0 = 0; k0 < K; k0 += 4) {
        const int k = k0 + quad;
        z64 x = {0, 0}, y = {0, 0};
        if (k < K) {
          int sh = k % d + P.x[s];
          sh -= sh >= d ? d : 0;
          if (r0 + col < cr) x = A[(k - k % d + sh) * cr + r0 + col];
          if (n0 + col < cr) y = T[k * cr + n0 + col];
        }
        x.im = -x.im;
        mma4(x, y, cr_, ci_);
      }
      if (n0 + col < cr) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (r0 + 4 * q + quad < cr) E[(n0 + col) * cr + r0 + 4 * q + quad] = z64{cr_[q], ci_[q]};
      }
    }
    __syncthreads();
  }
  __syncthreads();
  if (a.e_out) {
    const int c1 = a.chi[a.last];
    for (int i = t; i < c1 * c1; i += kThreads) a.e_out[i] = E[(i % c1) * c1 + i / c1];
  }
  if (a.result && t == 0) {
    a.result->value = E[0];
    a.result->p = P.p;
    announce(&a.result->ticket, a.ticket);
  }
}

// out[(al, t), b] = conj(omega^{z t}) A[(al, t + x), b] with the exponents of site `site` of *P.
__global__ void k_weyl_site(int d, int chil, int chir, int site, const DevWeyl* __restrict__ P,
                            const z64* __restrict__ in, z64* __restrict__ out) {
  const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (size_t)chil * d * chir) return;
  const int b = (int)(idx % chir), s = (int)((idx / chir) % d);
  const size_t al = idx / ((size_t)chir * d);
  const double ang = -2.0 * M_PI * ((P->z[site] * s) % d) / d;
  out[idx] = cmul(z64{cos(ang), sin(ang)}, in[(al * d + (s + P->x[site]) % d) * chir + b]);
}

}  // namespace

void launch_expect_chain(hipStream_t s, const ExpectArgs& a) {
  int e = a.chi[a.first] * a.chi[a.first], m = 0;
  for (int i = a.first; i < a.last; ++i) {
    e = std::max(e, a.chi[i + 1] * a.chi[i + 1]);
    m = std::max(m, a.chi[i] * a.d * a.chi[i + 1]);
  }
  hipLaunchKernelGGL(k_expect_chain, dim3(1), dim3(kThreads), (size_t)(e + 2 * m) * sizeof(z64), s, a, e, m);
  GC_LAUNCH_CHECK();
}

void launch_weyl_site(hipStream_t s, int d, int chil, int chir, int site, const DevWeyl* P, const z64* in, z64* out) {
  const size_t total = (size_t)chil * d * chir;
  hipLaunchKernelGGL(k_weyl_site, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, d, chil, chir, site, P, in,
                     out);
  GC_LAUNCH_CHECK();
}

void expect_set_attributes() {
  (void)hipFuncSetAttribute(reinterpret_cast<const void*>(k_expect_chain), hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)((kExpectMaxBond2 + 2 * kExpectMaxSite) * sizeof(z64)));
  (void)hipGetLastError();
}

}  // namespace gc
