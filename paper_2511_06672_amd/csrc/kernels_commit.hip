// The commit of a scored bond in one launch: the choice c* from the scores, Theta <- Q_c* Theta and the
// tableau update C <- C Q_c*^dagger.
#include <cfloat>
#include <climits>

#include "kernels.h"
#include "weyl.h"

namespace gc {

namespace {

constexpr int kThreads = 256;

__device__ __forceinline__ double block_min(double v, double* red) {
  for (int off = 32; off > 0; off >>= 1) v = fmin(v, __shfl_xor(v, off, 64));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  v = fmin(fmin(red[0], red[1]), fmin(red[2], red[3]));
  __syncthreads();
  return v;
}

__device__ __forceinline__ int block_min(int v, int* red) {
  for (int off = 32; off > 0; off >>= 1) v = min(v, __shfl_xor(v, off, 64));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  v = min(min(red[0], red[1]), min(red[2], red[3]));
  __syncthreads();
  return v;
}

// The lowest index within tol of the smallest score; with ranks, among the candidates of the smallest rank
// and 0 unless that rank is below the identity's.  Scores that compare with nothing leave the identity.
__device__ __forceinline__ int choose(const CommitRule& r, int count, double& smin) {
  __shared__ double red[4];
  __shared__ int redi[4];
  const int t = threadIdx.x;
  int rbest = 0;
  if (r.rank) {
    rbest = INT_MAX;
    for (int i = t; i < count; i += kThreads) rbest = min(rbest, r.rank[i]);
    rbest = block_min(rbest, redi);
  }
  smin = DBL_MAX;
  for (int i = t; i < count; i += kThreads)
    if (!r.rank || r.rank[i] == rbest) smin = fmin(smin, r.s2[i]);
  smin = block_min(smin, red);
  int best = INT_MAX;
  for (int i = t; i < count; i += kThreads)
    if ((!r.rank || r.rank[i] == rbest) && r.s2[i] <= smin + r.tol) best = min(best, r.list ? r.list[i] : i);
  best = block_min(best, redi);
  if (best == INT_MAX || (r.rank && rbest >= r.rank[0])) return 0;
  return best;
}

// New tableau row of image e (a word of Q^dagger P Q): D_a^xa S_a^za D_b^xb S_b^zb with the word's phase.
// A lane carries sites lane and lane + 64 through the four factors (the phase is a sum over sites), so one
// wave sum per row remains.
struct NewRow {
  int x[2], z[2], p;
};
__device__ __forceinline__ NewRow new_row(int n, int d, int site, uint32_t e, const int* __restrict__ tx,
                                          const int* __restrict__ tz, const int* __restrict__ tp, int lane) {
  const int img = (int)(e & 0xffffu);
  const int ex[4] = {img / (d * d * d), (img / (d * d)) % d, (img / d) % d, img % d};
  const int rows[4] = {n + site, site, n + site + 1, site + 1};
  NewRow o = {{0, 0}, {0, 0}, (int)(e >> 16)};
  int ph = 0;
#pragma unroll
  for (int f = 0; f < 4; ++f) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int i = lane + 64 * h;
      const int x = i < n ? tx[rows[f] * n + i] : 0, z = i < n ? tz[rows[f] * n + i] : 0;
      ph += o.z[h] * (ex[f] * x) + x * z * (ex[f] * (ex[f] - 1) / 2);
      o.x[h] += ex[f] * x;
      o.z[h] += ex[f] * z;
    }
    o.p += ex[f] * tp[rows[f]];
  }
  for (int off = 32; off > 0; off >>= 1) ph += __shfl_xor(ph, off, 64);
  o.p = (o.p + 2 * (ph % d)) % (2 * d);
  return o;
}

// Bound by latency: the scores are a few KB in L2 and Theta is read and written once.  Every workgroup makes
// the choice for itself (each reads all scores), which costs less than a launch for it: choice, rotation and
// tableau as three launches took 3.3 + 5.9 + 5.9 us with two gaps between them (d = 3, 512 candidates),
// this one 4.3 us.  A thread holds the d^2 entries of one (a, b) in registers; the last workgroup of a
// choosing launch updates the tableau, a wave per row, and writes the status.
template <int D>
__global__ __launch_bounds__(kThreads) void k_commit(CommitRule r, int chil, int chir, const z64* __restrict__ qm,
                                                     z64* __restrict__ theta, CommitTableau tb) {
  constexpr int D2 = D * D;
  const int64_t t0 = wall_clock64();
  __shared__ z64 q[D2 * D2];
  const int t = threadIdx.x;
  const bool last = r.fixed < 0 && blockIdx.x == gridDim.x - 1;
  const size_t idx = (size_t)blockIdx.x * kThreads + t;
  const bool mine = !last && idx < (size_t)chil * chir;
  z64* const col = theta + (idx / chir) * D2 * chir + idx % chir;
  z64 v[D2];
#pragma unroll
  for (int x = 0; x < D2; ++x) v[x] = mine ? col[(size_t)x * chir] : z64{0.0, 0.0};
  double smin = 0.0;
  const int count = r.fixed >= 0 ? 0 : r.list ? r.st->nwindow : r.count;
  const int c = r.fixed >= 0 ? r.fixed : choose(r, count, smin);
  if (last) {
    if (t == 0) {
      if (r.tick) *r.tick = t0;
      r.st->cstar = c;
      r.st->s2min = smin;
      r.host->cstar = c;
      announce(&r.host->ticket, r.ticket);
    }
    if (c == 0) return;
    // targets Z_a, Z_b, X_a, X_b (index ((xa d + za) d + xb) d + zb) of waves 0..3
    const int w = t >> 6, lane = t & 63, n = tb.n;
    const int tgt = w == 0 ? D * D : w == 1 ? 1 : w == 2 ? D * D * D : D;
    const int row = tb.site + (w & 1) + (w >> 1) * n;
    const NewRow o = new_row(n, D, tb.site, tb.inv_luts[(size_t)c * D2 * D2 + tgt], tb.tx, tb.tz, tb.tp, lane);
    __syncthreads();  // every old row has been read
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int i = lane + 64 * h;
      if (i < n) {
        tb.tx[row * n + i] = o.x[h] % D;
        tb.tz[row * n + i] = o.z[h] % D;
      }
    }
    if (lane == 0) tb.tp[row] = o.p;
    return;
  }
  if (c == 0) return;
  for (int i = t; i < D2 * D2; i += kThreads) q[i] = qm[(size_t)c * D2 * D2 + i];
  __syncthreads();
  if (!mine) return;
  for (int y = 0; y < D2; ++y) {
    z64 acc = {0.0, 0.0};
#pragma unroll
    for (int x = 0; x < D2; ++x) acc = cadd(acc, cmul(q[y * D2 + x], v[x]));
    col[(size_t)y * chir] = acc;
  }
}

}  // namespace

void launch_commit(hipStream_t s, int d, const CommitRule& r, int chil, int chir, const z64* qmats, z64* theta,
                   const CommitTableau& tb) {
  const unsigned blocks = (unsigned)(((size_t)chil * chir + kThreads - 1) / kThreads) + (r.fixed < 0 ? 1 : 0);
#define GC_COMMIT(D) \
  hipLaunchKernelGGL(k_commit<D>, dim3(blocks), dim3(kThreads), 0, s, r, chil, chir, qmats, theta, tb)
  if (d == 2)
    GC_COMMIT(2);
  else if (d == 3)
    GC_COMMIT(3);
  else if (d == 5)
    GC_COMMIT(5);
  else
    GC_COMMIT(7);
#undef GC_COMMIT
  GC_LAUNCH_CHECK();
}

}  // namespace gc
