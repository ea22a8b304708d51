// The dense state psi = C|MPS> of the validation calls (d^n <= 2^16), from the dense MPS vector m and the
// tableau: psi(y) = sum_x m(x) (C X^x C^dagger s0)(y) with s0 = C|0>.
//
// A basis index is held as packed digits, four bits each (n <= 16, d <= 7), site 0 in the highest used
// nibble, so that y - a over Z_d^n is a handful of 64-bit operations instead of n divisions.
#include "kernels.h"

namespace gc {

namespace {

constexpr uint64_t kHigh = 0x8888888888888888ull;
constexpr int kMaxNd = 40;        // powers of n tableau rows: n d <= 35 for d^n <= 2^16
constexpr int kPhases = 256;      // <b, s> of two digit strings: at most n (d - 1)^2 = 180

__device__ __forceinline__ z64 tau_pow(int p, int d) {
  double ang = M_PI * (double)p / (double)d;
  return z64{cos(ang), sin(ang)};
}

// Digitwise a - b mod d: every nibble of (a | 8) - b is 8 + a - b in 2..14 and has bit 3 where a >= b.
__device__ __forceinline__ uint64_t sub_digits(uint64_t a, uint64_t b, int d) {
  const uint64_t t = (a | kHigh) - b;
  return (t + ((~t & kHigh) >> 3) * (uint64_t)d) & ~kHigh;
}

__device__ __forceinline__ uint64_t pack_digits(long long y, int n, int d) {
  uint64_t w = 0;
  unsigned rem = (unsigned)y;
  for (int r = 0; r < n; ++r) {
    const unsigned q = rem / (unsigned)d;
    w |= (uint64_t)(rem - q * d) << (4 * r);
    rem = q;
  }
  return w;
}

// Index of the digits s and <b, s> (an integer, not reduced).
__device__ __forceinline__ void fold_digits(uint64_t s, uint64_t b, int n, int d, int& src, int& ph) {
  src = 0;
  ph = 0;
  for (int r = 4 * (n - 1); r >= 0; r -= 4) {
    const int si = (int)(s >> r) & 7;
    src = src * d + si;
    ph += ((int)(b >> r) & 7) * si;
  }
}

// Power e of tableau row `row` (tau^p X^x Z^z): digits x, z and the tau phase mod 2d.
__device__ void row_power(int n, int d, const int* __restrict__ tx, const int* __restrict__ tz,
                          const int* __restrict__ tp, int row, int e, uint64_t& x, uint64_t& z, int& p) {
  int xz = 0;
  x = z = 0;
  for (int i = 0; i < n; ++i) {
    const int a = tx[row * n + i], b = tz[row * n + i];
    xz += a * b;
    x |= (uint64_t)((e * a) % d) << (4 * (n - 1 - i));
    z |= (uint64_t)((e * b) % d) << (4 * (n - 1 - i));
  }
  p = (e * tp[row] + 2 * (xz % d) * (e * (e - 1) / 2)) % (2 * d);
}

// A fixed generic vector, whose projection on any stabilizer state does not vanish.
__global__ void k_dense_start(int D, z64* __restrict__ out) {
  const int y = blockIdx.x * blockDim.x + threadIdx.x;
  if (y < D) out[y] = z64{cos(0.731 * y + 0.2), sin(1.37 * y + 0.5) + 0.3};
}

// out = (1/d) sum_j S_k^j in: the projector on the +1 eigenspace of one stabilizer row, all powers in one
// pass (the sum over j reads d entries and writes one; it was one launch and one pass over out per power).
__global__ void k_stab_project(int n, int d, int D, int k, const int* __restrict__ tx, const int* __restrict__ tz,
                               const int* __restrict__ tp, const z64* __restrict__ in, z64* __restrict__ out) {
  __shared__ uint64_t px[kMaxD], pz[kMaxD];
  __shared__ int pp[kMaxD];
  __shared__ z64 om[kPhases];
  const int t = threadIdx.x;
  if (t < d) row_power(n, d, tx, tz, tp, k, t, px[t], pz[t], pp[t]);
  om[t] = tau_pow(2 * (t % d), d);
  __syncthreads();
  const int y = blockIdx.x * kPhases + t;
  if (y >= D) return;
  const uint64_t yd = pack_digits(y, n, d);
  z64 acc = {0.0, 0.0};
  for (int j = 0; j < d; ++j) {
    int src, ph;
    fold_digits(sub_digits(yd, px[j], d), pz[j], n, d, src, ph);
    acc = cadd(acc, cmul(tau_pow(pp[j], d), cmul(om[ph], in[src])));
  }
  out[y] = z64{acc.re / d, acc.im / d};
}

// C X^x C^dagger = prod_k D_k^{x_k} = tau^{p_x} X^{a_x} Z^{b_x}: ab[x] = the digits (a_x, b_x), and
// m[x] *= tau^{p_x}.  One thread per x; the n d row powers are in LDS.
__global__ void k_dense_table(int n, int d, int D, const int* __restrict__ tx, const int* __restrict__ tz,
                              const int* __restrict__ tp, ulonglong2* __restrict__ ab, z64* __restrict__ m) {
  __shared__ uint64_t px[kMaxNd], pz[kMaxNd];
  __shared__ int pp[kMaxNd];
  const int t = threadIdx.x;
  if (t < n * d) row_power(n, d, tx, tz, tp, n + t / d, t % d, px[t], pz[t], pp[t]);
  __syncthreads();
  const int x = blockIdx.x * blockDim.x + t;
  if (x >= D) return;
  const uint64_t xd = pack_digits(x, n, d);
  uint64_t a = 0, b = 0;
  int p = 0;
  for (int k = 0; k < n; ++k) {
    const int e = k * d + ((int)(xd >> (4 * (n - 1 - k))) & 7);
    int src, cross;
    fold_digits(px[e], b, n, d, src, cross);
    p += pp[e] + 2 * cross;
    a = sub_digits(a, sub_digits(0, px[e], d), d);
    b = sub_digits(b, sub_digits(0, pz[e], d), d);
  }
  ab[x] = ulonglong2{a, b};
  m[x] = cmul(tau_pow(p % (2 * d), d), m[x]);
}

// psi(y) = f sum_x m(x) omega^{<b_x, y - a_x>} s0(y - a_x), f = 1 / sqrt(*norm2).
// D^2 terms of about 60 integer operations and one gathered amplitude: bound by instruction issue.  A
// workgroup takes 64 indices y (one a lane) and its 16 waves split x, so that D / 64 x 16 waves are in
// flight (one thread per y left 104 waves for D = 6561, nine in ten SIMDs idle) and a_x, b_x, m(x) are
// uniform over a wave and come through the scalar cache; four x at a time keep as many gathers in flight.
// D = 6561: 5000 us in the one-thread form, 255 us in this one.
constexpr int kDenseWaves = 16;
constexpr int kDenseUnroll = 4;

__global__ __launch_bounds__(64 * kDenseWaves) void k_clifford_dense(
    int n, int d, int D, const ulonglong2* __restrict__ ab, const z64* __restrict__ m, const z64* __restrict__ s0,
    const double* __restrict__ norm2, z64* __restrict__ out) {
  __shared__ z64 om[kPhases];
  __shared__ z64 part[kDenseWaves][64];
  const int t = threadIdx.x, lane = t & 63;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  if (t < kPhases) om[t] = tau_pow(2 * (t % d), d);
  __syncthreads();
  const int y = blockIdx.x * 64 + lane;
  const uint64_t yd = pack_digits(y < D ? y : 0, n, d);
  z64 acc[kDenseUnroll];
  for (int u = 0; u < kDenseUnroll; ++u) acc[u] = z64{0.0, 0.0};
  const int step = kDenseWaves * kDenseUnroll;
  auto term = [&](int x, z64& sum) {
    const ulonglong2 e = ab[x];
    int src, ph;
    fold_digits(sub_digits(yd, e.x, d), e.y, n, d, src, ph);
    sum = cadd(sum, cmul(m[x], cmul(om[ph], s0[src])));
  };
  int x = w * kDenseUnroll;
  for (; x + kDenseUnroll <= D; x += step) {
#pragma unroll
    for (int u = 0; u < kDenseUnroll; ++u) term(x + u, acc[u]);
  }
  for (int u = 0; x + u < D && u < kDenseUnroll; ++u) term(x + u, acc[0]);
  part[w][lane] = cadd(cadd(acc[0], acc[1]), cadd(acc[2], acc[3]));
  __syncthreads();
  if (w != 0 || y >= D) return;
  z64 s = part[0][lane];
  for (int i = 1; i < kDenseWaves; ++i) s = cadd(s, part[i][lane]);
  const double f = 1.0 / sqrt(*norm2);
  out[y] = z64{f * s.re, f * s.im};
}

__global__ void k_norm2(const z64* __restrict__ v, int count, double* out) {
  __shared__ double red[1024];
  double s = 0.0;
  for (int i = threadIdx.x; i < count; i += 1024) s += cabs2(v[i]);
  red[threadIdx.x] = s;
  __syncthreads();
  for (int off = 512; off > 0; off >>= 1) {
    if ((int)threadIdx.x < off) red[threadIdx.x] += red[threadIdx.x + off];
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = red[0];
}

inline unsigned blocks_for(int n, int bs) { return (unsigned)((n + bs - 1) / bs); }

}  // namespace

void launch_stab_state(hipStream_t s, int n, int d, int D, const int* tx, const int* tz, const int* tp, z64*& v,
                       z64*& w, double* norm2) {
  hipLaunchKernelGGL(k_dense_start, dim3(blocks_for(D, 256)), dim3(256), 0, s, D, v);
  for (int k = 0; k < n; ++k) {
    hipLaunchKernelGGL(k_stab_project, dim3(blocks_for(D, kPhases)), dim3(kPhases), 0, s, n, d, D, k, tx, tz, tp, v,
                       w);
    std::swap(v, w);
  }
  hipLaunchKernelGGL(k_norm2, dim3(1), dim3(1024), 0, s, v, D, norm2);
  GC_LAUNCH_CHECK();
}

void launch_clifford_dense(hipStream_t s, int n, int d, int D, const int* tx, const int* tz, const int* tp, void* ab,
                           z64* m, const z64* s0, const double* norm2, z64* out) {
  ulonglong2* tab = reinterpret_cast<ulonglong2*>(ab);
  hipLaunchKernelGGL(k_dense_table, dim3(blocks_for(D, 256)), dim3(256), 0, s, n, d, D, tx, tz, tp, tab, m);
  hipLaunchKernelGGL(k_clifford_dense, dim3(blocks_for(D, 64)), dim3(64 * kDenseWaves), 0, s, n, d, D, tab, m, s0,
                     norm2, out);
  GC_LAUNCH_CHECK();
}

}  // namespace gc
