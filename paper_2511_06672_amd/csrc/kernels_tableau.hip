// Integer Z_d tableau kernels: Clifford layer update and commutation of a Weyl operator through C (§2.2, §2.3,
// §2.3.1, §3); the right multiplication by a disentangler is part of the bond's commit.
//
// Device layout: row r of the 2n-row tableau has exponents tx[r*n + i], tz[r*n + i] for site
// i and phase tp[r] (power of tau, mod 2d).  Rows 0..n-1 are S_k = C Z_k C^dagger, rows
// n..2n-1 are D_k = C X_k C^dagger.  All arithmetic is exact integer arithmetic.
#include "kernels.h"
#include "weyl.h"

namespace gc {

namespace {

__global__ void k_tableau_init(int n, int* tx, int* tz, int* tp) {
  int idx = blockIdx.x * blockDim.x + threadIdx.x;
  int total = 2 * n * n;
  if (idx < total) {
    int r = idx / n, i = idx % n;
    tx[idx] = (r >= n && r - n == i) ? 1 : 0;
    tz[idx] = (r < n && r == i) ? 1 : 0;
  }
  if (idx < 2 * n) tp[idx] = 0;
}

// One thread per tableau row; the words of a layer act on disjoint pairs and are applied
// in order.  lut entry: low 16 bits = image index, bits 16.. = tau-phase increment.
__global__ void k_tableau_layer(int n, int d, int count, const int* __restrict__ sites,
                                const uint32_t* __restrict__ luts, int* tx, int* tz, int* tp) {
  int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= 2 * n) return;
  const int D4 = d * d * d * d;
  int p = tp[r];
  for (int w = 0; w < count; ++w) {
    int a = sites[w], b = a + 1;
    int xa = tx[r * n + a], za = tz[r * n + a], xb = tx[r * n + b], zb = tz[r * n + b];
    int v = ((xa * d + za) * d + xb) * d + zb;
    uint32_t e = luts[(size_t)w * D4 + v];
    int img = (int)(e & 0xffffu);
    p = imod(p + (int)(e >> 16), 2 * d);
    tz[r * n + b] = img % d;
    tx[r * n + b] = (img / d) % d;
    tz[r * n + a] = (img / (d * d)) % d;
    tx[r * n + a] = img / (d * d * d);
  }
  tp[r] = p;
}

__global__ __launch_bounds__(kMaxN) void k_weyl_extract(int n, int d, const int* __restrict__ tx,
                                                        const int* __restrict__ tz, const int* __restrict__ tp,
                                                        WeylTarget target, DevWeyl* out, Ticket ticket) {
  __shared__ DevWeyl P;
  __shared__ WeylScratch ws;
  weyl_commute(n, d, tx, tz, tp, target, P, ws);
  const int t = threadIdx.x;
  if (t < n) {
    out->x[t] = P.x[t];
    out->z[t] = P.z[t];
  }
  if (t == 0) {
    out->p = P.p;
    out->l = P.l;
    out->r = P.r;
    out->bad = P.bad;
  }
  __threadfence_system();  // every thread's part before the ticket
  __syncthreads();
  if (t == 0) announce(&out->ticket, ticket);
}

}  // namespace

void launch_tableau_init(hipStream_t s, int n, int* tx, int* tz, int* tp) {
  int total = 2 * n * n;
  hipLaunchKernelGGL(k_tableau_init, dim3((total + 255) / 256), dim3(256), 0, s, n, tx, tz, tp);
  GC_LAUNCH_CHECK();
}

void launch_tableau_layer(hipStream_t s, int n, int d, int count, const int* sites, const uint32_t* luts,
                          int* tx, int* tz, int* tp) {
  hipLaunchKernelGGL(k_tableau_layer, dim3((2 * n + 127) / 128), dim3(128), 0, s, n, d, count, sites, luts,
                     tx, tz, tp);
  GC_LAUNCH_CHECK();
}

void launch_weyl_extract(hipStream_t s, int n, int d, const int* tx, const int* tz, const int* tp,
                         const WeylTarget& target, DevWeyl* out, Ticket ticket) {
  hipLaunchKernelGGL(k_weyl_extract, dim3(1), dim3(kMaxN), 0, s, n, d, tx, tz, tp, target, out, ticket);
  GC_LAUNCH_CHECK();
}

}  // namespace gc
