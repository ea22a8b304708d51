// Commutation of a Weyl operator through the tableau, P = C^dagger W C, by one workgroup: shared by the
// kernel that returns P to the host and by the expectation kernel, which uses it at once.
#pragma once

#include "internal.h"

namespace gc {

namespace {

__device__ __forceinline__ int imod(int v, int m) {
  v %= m;
  return v < 0 ? v + m : v;
}

struct WeylScratch {
  int sum, sd, bad, l, r;
};

// Exponents from the symplectic relations: delta_j = -lam(W, S_j), s_j = lam(W, D_j) with
// lam(u, v) = <z_u, x_v> - <x_u, z_v>.  The phase follows from multiplying the rows out:
// prod_j S_j^{s_j} D_j^{delta_j} = tau^q W(t), and P = W(delta, s, p_t - q + 2 <s, delta>).
//
// A product's phase p_a + p_b + 2 <z_a, x_b> is a sum over sites, so a thread carries one site through all
// 2n rows (its running z and its share of the phase) and the sites are summed once at the end: the row
// loads are independent and coalesced.  With one wave holding whole rows and reducing <z_a, x_b> at every
// row the same product was 2n dependent load-and-reduce steps (n = 8 to 10: 10 us a launch).  Sums stay far
// below 2^31 (n <= 128, d <= 7), so nothing is reduced modulo d on the way.  Blocks of at least n threads;
// out and ws in LDS.
__device__ __forceinline__ void weyl_commute(int n, int d, const int* __restrict__ tx, const int* __restrict__ tz,
                                             const int* __restrict__ tp, const WeylTarget& W, DevWeyl& out,
                                             WeylScratch& ws) {
  const int t = threadIdx.x;
  if (t == 0) ws = WeylScratch{0, 0, 0, n, -1};
  __syncthreads();
  if (t < n) {
    int ls = 0, ld = 0;
    for (int i = 0; i < n; ++i) {
      ls += W.z[i] * tx[t * n + i] - W.x[i] * tz[t * n + i];
      ld += W.z[i] * tx[(n + t) * n + i] - W.x[i] * tz[(n + t) * n + i];
    }
    const int dx = imod(-ls, d), sz = imod(ld, d);
    out.x[t] = dx;
    out.z[t] = sz;
    atomicAdd(&ws.sum, sz * tp[t] + dx * tp[n + t]);
    atomicAdd(&ws.sd, sz * dx);
    if (dx | sz) {
      atomicMin(&ws.l, t);
      atomicMax(&ws.r, t);
    }
  }
  __syncthreads();
  if (t < n) {
    int xa = 0, za = 0, ph = 0;
#pragma unroll 4
    for (int j = 0; j < n; ++j) {
      const int es = out.z[j], ed = out.x[j];
      const int sx = tx[j * n + t], sz = tz[j * n + t], dx = tx[(n + j) * n + t], dz = tz[(n + j) * n + t];
      ph += za * (es * sx) + sx * sz * (es * (es - 1) / 2);
      xa += es * sx;
      za += es * sz;
      ph += za * (ed * dx) + dx * dz * (ed * (ed - 1) / 2);
      xa += ed * dx;
      za += ed * dz;
    }
    atomicAdd(&ws.sum, 2 * (ph % d));
    if (xa % d != W.x[t] || za % d != W.z[t]) ws.bad = 1;
  }
  __syncthreads();
  if (t == 0) {
    out.p = imod(W.p - ws.sum + 2 * ws.sd, 2 * d);
    out.l = ws.r < 0 ? -1 : ws.l;
    out.r = ws.r;
    out.bad = ws.bad;
  }
  __syncthreads();
}

}  // namespace

}  // namespace gc
