// Device code of the Hermitian Jacobi eigensolver shared by the single-workgroup kernels (a matrix of
// at most 32 rows in LDS) and the block-Jacobi rounds (32 x 32 sub-problems): the rotation, the
// parallel steps and the sweeps of a matrix in LDS.
#pragma once

#include "internal.h"

namespace gc {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef double d2 __attribute__((ext_vector_type(2)));

namespace {

// Round-robin (circle) pairing: step s of mp-1 steps pairs positions k and mp-1-k; position 0
// is fixed, position i >= 1 holds element ((i - 1 + s) mod (mp - 1)) + 1.  Every unordered pair
// of the mp indices meets exactly once per sweep.
__device__ __forceinline__ void rr_pair(int k, int s, int mp, int& p, int& q) {
  // k < mp / 2 and 0 <= s < mp - 1 keep both circle positions below 2 (mp - 1): one conditional
  // subtraction reduces them
  const int n1 = mp - 1, i0 = k, i1 = mp - 1 - k;
  const int x0 = i0 - 1 + s, x1 = i1 - 1 + s;
  int e0 = (i0 == 0) ? 0 : (x0 >= n1 ? x0 - n1 : x0) + 1;
  int e1 = (x1 >= n1 ? x1 - n1 : x1) + 1;
  p = e0 < e1 ? e0 : e1;
  q = e0 < e1 ? e1 : e0;
}

// Thresholds of the rotation test.  Absolute criterion: |g|^2 > t0 = thr^2.  Relative criterion:
// |g|^2 > t0 (the floor), |g|^2 > tol2 |a b| and max(|a|, |b|) > skip (pairs whose diagonal
// entries are both below skip are left alone).
struct JacobiThr {
  double t0, tol2, skip;
};
__device__ __forceinline__ JacobiThr jacobi_thr(double trace, double tol, double skip_rel, int rel, double floor_rel) {
  const double f = (rel ? floor_rel : tol) * trace;
  return JacobiThr{fmax(f * f, 1e-290), tol * tol, skip_rel * trace};
}

// Whether the pair with diagonal (a, b) and |off-diagonal|^2 = h2 is rotated.
template <bool REL>
__device__ __forceinline__ bool rot_needed(double a, double b, double h2, const JacobiThr& jt) {
  bool need = h2 > jt.t0;
  if (REL) {  // the three tests without branches
    const bool rel = h2 > jt.tol2 * fabs(a) * fabs(b), big = fmax(fabs(a), fabs(b)) > jt.skip;
    need = ((int)need & (int)rel & (int)big) != 0;
  }
  return need;
}

// Rotation J = [[c, -s], [conj(s), c]] (c real, |s|^2 = 1 - c^2) that diagonalises the Hermitian
// 2x2 [[a, g], [conj g, b]] as J H J^H, by the smaller angle: with
// den = |b - a| + sqrt((b - a)^2 + 4|g|^2),
// c = den / sqrt(den^2 + 4|g|^2) and s = sign(b - a) 2 g / sqrt(den^2 + 4|g|^2).
// den only sets the angle: it gets one Newton step on the hardware's 23-bit square root, and what
// a slightly wrong angle leaves off the diagonal stays in the matrix (the block is rotated as
// computed, nothing is set to zero).  The last factor is refined by
// one third-order step (the estimate's error cubed is below 2^-66), and c then takes up what its
// rounding leaves of c^2 + |s|^2 = 1 (with 1 - c / 2 for 1 / (2 c)): the thousands of small rotations
// a vector goes through would otherwise change its length by up to 2e-13.  Every lane
// computes the rotation and selects the identity where the pair is not rotated, so that a
// thread's two rotations interleave.
struct Rot {
  double c, sr, si;
};
template <bool REL>
__device__ __forceinline__ Rot make_rot(double a, double b, double gr, double gi, const JacobiThr& jt) {
  const double h2 = gr * gr + gi * gi;
  const bool need = rot_needed<REL>(a, b, h2, jt);
  const double dlt = b - a, h4 = 4.0 * h2;
  const double r2 = fma(dlt, dlt, h4);
  const double y0 = __builtin_amdgcn_rsq(r2);
  const double s0 = r2 * y0;
  const double den = fabs(dlt) + fma(fma(-s0, s0, r2), 0.5 * y0, s0);
  const double dd = fma(den, den, h4);
  const double y = __builtin_amdgcn_rsq(dd);
  const double e = fma(-(dd * y), y, 1.0);
  const double q = fma(y * e, fma(e, 0.375, 0.5), y);
  const double f = need ? copysign(2.0 * q, dlt) : 0.0;
  const double sr = f * gr, si = f * gi, c = den * q;
  const double miss = fma(-si, si, fma(-sr, sr, fma(-c, c, 1.0)));
  return Rot{need ? fma(miss, fma(-0.5, c, 1.0), c) : 1.0, sr, si};
}

// Rows of a 2x2 block (x above y): x' = c x - s y, y' = conj(s) x + c y.
__device__ __forceinline__ void rot_rows(z64& x, z64& y, const Rot& r) {
  const z64 u = {r.c * x.re - r.sr * y.re + r.si * y.im, r.c * x.im - r.sr * y.im - r.si * y.re};
  const z64 v = {r.c * y.re + r.sr * x.re + r.si * x.im, r.c * y.im + r.sr * x.im - r.si * x.re};
  x = u;
  y = v;
}
// Columns (x beside y): x' = c x - conj(s) y, y' = s x + c y.
__device__ __forceinline__ void rot_cols(z64& x, z64& y, const Rot& r) {
  const z64 u = {r.c * x.re - r.sr * y.re - r.si * y.im, r.c * x.im - r.sr * y.im + r.si * y.re};
  const z64 v = {r.c * y.re + r.sr * x.re - r.si * x.im, r.c * y.im + r.sr * x.im + r.si * x.re};
  x = u;
  y = v;
}

// x from lane (l + 1) mod 16 of the same 16-lane row (DPP row rotation by 15 to the right); every
// lane of the row must be active.
__device__ __forceinline__ double row_next(double x) {
  const long long v = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_mov_dpp((int)v, 0x12F, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_mov_dpp((int)(v >> 32), 0x12F, 0xF, 0xF, true);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// x of the first lane of the same 16-lane row (DPP row broadcast).
__device__ __forceinline__ double row_first(double x) {
  const long long v = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_mov_dpp((int)v, 0x150, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_mov_dpp((int)(v >> 32), 0x150, 0xF, 0xF, true);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// The step loops below work on 512 threads: of the first 256, H item (k1, k2) is the 2x2 block of pairs
// k1 and k2 and needs both rotations; of the others, V item (k1, k2) applies rotation k1 to two rows of the
// eigenvector accumulator.  A step is bound by its FP64 issue slots (two waves per SIMD), its LDS
// accesses and one dependent chain LDS read, rotation, update, LDS write, barrier.
// The items of a 16-lane row share k1 and start at k2 = k1: every lane computes rotation k2 and takes
// rotation k1 from the first lane.  The V items follow one step behind with the rotations that the first
// row leaves in LDS, off the H items' chain.  With both rotations computed by every H thread, rotation
// k1 by every V thread and all four elements through LDS, a 27 x 81 split took 206 us against 156 us and an
// inter-block round at m = 243 13.3 us against 12.0 us.
struct RotSlot {
  z64 s;
  double c, pad;
};

// The inter-block steps of a 32-index sub-problem on 512 threads: step s (0..15) pairs index
// k < 16 with q_k(s) = 16 + (k + s) mod 16, so the 16 steps visit every pair (i < 16 <= j) once and
// leave the matrix in h0 (32 x 32, row-major; h1 is scratch).  The eigenvector accumulator starts from vi (32 x 32,
// row-major; null: the identity) and ends in vo.
// H and V live in registers.  After a step pair k takes over index q_{k+1}: an element (p1, q2) comes
// from the next lane of its row, (q1, p2) and (q1, q2) from the next row through LDS, and the next step's
// diagonal and pair elements go to LDS beside them.  After 16 steps the indices are back.
template <bool REL>
__device__ __forceinline__ void jacobi_ib_steps(z64* __restrict__ h0, z64* __restrict__ h1, const z64* vi, z64* vo,
                                                const JacobiThr& jt) {
  const int t = threadIdx.x, e = t & 255, l = e & 15;
  if (__builtin_amdgcn_readfirstlane(t >> 8) == 0) {  // uniform over each wave
    const int k1 = e >> 4, k2 = (l + k1) & 15, down = ((k1 + 1) & 15) * 16;
    z64 a = h0[k1 * 32 + k2], b = h0[k1 * 32 + 16 + k2];
    z64 c = h0[(16 + k1) * 32 + k2], d = h0[(16 + k1) * 32 + 16 + k2];
    d2 ab = {h0[k2 * 33].re, h0[(16 + k2) * 33].re};
    z64 g = h0[k2 * 32 + 16 + k2];
    RotSlot* rot = reinterpret_cast<RotSlot*>(h1 + 544);
    // exchange buffers of even and odd steps: h0 is free once every thread has read its elements
#pragma unroll 2
    for (int step = 0; step < 16; ++step) {
      z64* x = (step & 1) ? h0 : h1;
      const Rot r2 = make_rot<REL>(ab.x, ab.y, g.re, g.im, jt);
      const Rot r1 = {row_first(r2.c), row_first(r2.sr), row_first(r2.si)};
      if (e < 16) rot[(step & 1) * 16 + l] = RotSlot{{r2.sr, r2.si}, r2.c, 0.0};
      rot_rows(a, c, r1);
      rot_rows(b, d, r1);
      rot_cols(a, b, r2);
      rot_cols(c, d, r2);
      if (step == 15) break;
      x[e] = c;
      x[256 + e] = d;
      double* px = reinterpret_cast<double*>(x + 512);
      if (l == 0) {
        px[2 * k1] = a.re;
        px[2 * ((k1 + 15) & 15) + 1] = d.re;
      } else if (l == 1) {
        x[528 + k1] = b;
      }
      b = z64{row_next(b.re), row_next(b.im)};
      __syncthreads();
      c = x[down + ((l + 15) & 15)];
      d = x[256 + down + l];
      ab = reinterpret_cast<const d2*>(x + 512)[k2];
      g = x[528 + k2];
    }
    const int q1 = 16 + ((k1 + 15) & 15), q2 = 16 + ((k2 + 15) & 15);
    h0[k1 * 32 + k2] = a;
    h0[k1 * 32 + q2] = b;
    h0[q1 * 32 + k2] = c;
    h0[q1 * 32 + q2] = d;
    __syncthreads();
  } else {
    // columns (p, q) = (l, q_l) of rows k2 (x*) and k2 + 16 (y*)
    const int k2 = e >> 4;
    z64 xp = {(l == k2) ? 1.0 : 0.0, 0.0}, xq = {0.0, 0.0}, yp = {0.0, 0.0}, yq = xp;
    if (vi) {
      xp = vi[k2 * 32 + l];
      xq = vi[k2 * 32 + 16 + l];
      yp = vi[(k2 + 16) * 32 + l];
      yq = vi[(k2 + 16) * 32 + 16 + l];
    }
    const RotSlot* rot = reinterpret_cast<const RotSlot*>(h1 + 544);
#pragma unroll 2
    for (int step = 0; step < 16; ++step) {
      __syncthreads();
      const RotSlot s = rot[(step & 1) * 16 + l];
      const Rot r = {s.c, s.s.re, s.s.im};
      rot_cols(xp, xq, r);
      rot_cols(yp, yq, r);
      xq = z64{row_next(xq.re), row_next(xq.im)};
      yq = z64{row_next(yq.re), row_next(yq.im)};
    }
    vo[k2 * 32 + l] = xp;
    vo[k2 * 32 + 16 + l] = xq;
    vo[(k2 + 16) * 32 + l] = yp;
    vo[(k2 + 16) * 32 + 16 + l] = yq;
  }
}

// The steps inside the two 16-blocks of a 32-index sub-problem on 512 threads: step s (1..15) pairs
// i with i xor s in each block, eight pairs per block, so the 15 steps visit every pair of a block
// once and leave the matrix in h1.  H is held in the two LDS buffers (one read, one written by a step):
// element (i, j) at i * 32 + j, so that a row of 16 consecutive elements and the 16 diagonal or pair elements of
// a step fall in distinct banks.  Pair k < 8 of the first block starts at the element whose
// lowest set bit of s is clear, pair k >= 8 of the second at one where it is set: the 16 first (and
// the 16 second) elements of a step then differ modulo 16.  v (32 x 32,
// LDS) is updated in place; FIRST: v is the identity before, so only its diagonal blocks change
// (one row per V thread, otherwise two).  Ends with a barrier.
__device__ __forceinline__ void intra_pair(int k, int s, int& p, int& q) {
  const int bit = s & -s, low = bit - 1, c = k & 7;
  p = (((c & ~low) << 1) | (c & low)) + (k >= 8 ? 16 + bit : 0);
  q = p ^ s;
}
template <bool REL, bool FIRST>
__device__ __forceinline__ void jacobi_intra_steps(z64* __restrict__ h0, z64* __restrict__ h1, z64* __restrict__ v,
                                                   const JacobiThr& jt) {
  __shared__ RotSlot rot[32];
  const int t = threadIdx.x, e = t & 255, l = e & 15;
  if (__builtin_amdgcn_readfirstlane(t >> 8) == 0) {  // uniform over each wave
    const int k1 = e >> 4, k2 = (l + k1) & 15;
    for (int s = 1; s < 16; ++s) {
      const z64* __restrict__ in = (s & 1) ? h0 : h1;
      z64* __restrict__ out = (s & 1) ? h1 : h0;
      int p1, q1, p2, q2;
      intra_pair(k1, s, p1, q1);
      intra_pair(k2, s, p2, q2);
      const double a2 = in[p2 * 33].re, b2 = in[q2 * 33].re;
      const z64 g2 = in[p2 * 32 + q2];
      z64 a = in[p1 * 32 + p2], b = in[p1 * 32 + q2], c = in[q1 * 32 + p2], d = in[q1 * 32 + q2];
      const Rot r2 = make_rot<REL>(a2, b2, g2.re, g2.im, jt);
      const Rot r1 = {row_first(r2.c), row_first(r2.sr), row_first(r2.si)};
      if (e < 16) rot[(s & 1) * 16 + l] = RotSlot{{r2.sr, r2.si}, r2.c, 0.0};
      rot_rows(a, c, r1);
      rot_rows(b, d, r1);
      rot_cols(a, b, r2);
      rot_cols(c, d, r2);
      out[p1 * 32 + p2] = a;
      out[p1 * 32 + q2] = b;
      out[q1 * 32 + p2] = c;
      out[q1 * 32 + q2] = d;
      __syncthreads();
    }
  } else {
    z64* x = v + ((e >> 4) + (FIRST && l >= 8 ? 16 : 0)) * 32;
    for (int s = 1; s < 16; ++s) {
      int p, q;
      intra_pair(l, s, p, q);
      z64 xp = x[p], xq = x[q], yp = {0.0, 0.0}, yq = yp;
      if (!FIRST) {
        yp = x[16 * 32 + p];
        yq = x[16 * 32 + q];
      }
      __syncthreads();
      const RotSlot o = rot[(s & 1) * 16 + l];
      const Rot r = {o.c, o.s.re, o.s.im};
      rot_cols(xp, xq, r);
      x[p] = xp;
      x[q] = xq;
      if (!FIRST) {
        rot_cols(yp, yq, r);
        x[16 * 32 + p] = yp;
        x[16 * 32 + q] = yq;
      }
    }
  }
  __syncthreads();
}

// A full round-robin sweep (mp - 1 steps of mp / 2 pairs, mp <= 2 HM even) over H and the
// eigenvector accumulator v (LDS, same layout, updated in place) on 2 HM^2 threads: the first
// HM^2 take the H items, the others the V items.  Returns the index (0/1) of the buffer that
// holds the result.
template <int HM, bool REL>
__device__ __forceinline__ int jacobi_rr_steps(z64* __restrict__ h0, z64* __restrict__ h1, z64* __restrict__ v, int mp,
                                               const JacobiThr& jt) {
  constexpr int LD = 2 * HM;
  const int t = threadIdx.x, half = mp / 2, n1 = mp - 1;
  const bool do_v = t >= HM * HM;
  const int e = do_v ? t - HM * HM : t;
  const int k1 = do_v ? e % HM : e / HM, k2 = do_v ? e / HM : e % HM;
  const bool act = k1 < half && k2 < half;
  // the circle elements of pairs k1 and k2: position i >= 1 holds ((i - 1 + s) mod n1) + 1
  int u1 = k1, w1 = mp - 1 - k1, u2 = k2, w2 = mp - 1 - k2;
  int cur = 0;
  for (int step = 0; step < n1; ++step) {
    const z64* __restrict__ in = cur ? h1 : h0;
    z64* __restrict__ out = cur ? h0 : h1;
    if (act) {
      const int p1 = min(u1, w1), q1 = max(u1, w1);
      const double a1 = in[p1 * (LD + 1)].re, b1 = in[q1 * (LD + 1)].re;
      const z64 g1 = in[p1 * LD + q1];
      if (!do_v) {
        const int p2 = min(u2, w2), q2 = max(u2, w2);
        const double a2 = in[p2 * (LD + 1)].re, b2 = in[q2 * (LD + 1)].re;
        const z64 g2 = in[p2 * LD + q2];
        z64 a = in[p1 * LD + p2], b = in[p1 * LD + q2], c = in[q1 * LD + p2], d = in[q1 * LD + q2];
        const Rot r1 = make_rot<REL>(a1, b1, g1.re, g1.im, jt), r2 = make_rot<REL>(a2, b2, g2.re, g2.im, jt);
        rot_rows(a, c, r1);
        rot_rows(b, d, r1);
        rot_cols(a, b, r2);
        rot_cols(c, d, r2);
        out[p1 * LD + p2] = a;
        out[p1 * LD + q2] = b;
        out[q1 * LD + p2] = c;
        out[q1 * LD + q2] = d;
      } else {
        const Rot r1 = make_rot<REL>(a1, b1, g1.re, g1.im, jt);
        z64* x = v + k2 * LD;
        z64* y = v + (k2 + half) * LD;
        z64 xp = x[p1], xq = x[q1], yp = y[p1], yq = y[q1];
        rot_cols(xp, xq, r1);
        rot_cols(yp, yq, r1);
        x[p1] = xp;
        x[q1] = xq;
        y[p1] = yp;
        y[q1] = yq;
      }
      u1 = (k1 == 0) ? 0 : (u1 == n1 ? 1 : u1 + 1);
      u2 = (k2 == 0) ? 0 : (u2 == n1 ? 1 : u2 + 1);
      w1 = (w1 == n1) ? 1 : w1 + 1;
      w2 = (w2 == n1) ? 1 : w2 + 1;
    }
    __syncthreads();
    cur ^= 1;
  }
  return cur;
}

// Sweeps over the Hermitian H (m x m, m <= 2 HM; hs: two LDS buffers of leading dimension 2 HM, the matrix
// in hs, zeros beyond m) until no pair passes the rotation test; v (LDS, same layout) accumulates the
// rotations.  At least 2 HM^2 threads.  Each sweep is preceded by the test over all pairs, so no
// sweep only confirms convergence.  pending: two LDS flags, cleared before.  Returns the buffer that
// holds the rotated matrix; *sweeps counts the sweeps, *conv tells convergence within max_sweeps.
template <int HM, bool REL>
__device__ z64* jacobi_sweeps(z64* hs, z64* v, int m, const JacobiThr& jt, int max_sweeps, int* pending, int* sweeps,
                              bool* conv) {
  constexpr int LD = 2 * HM;
  const int t = threadIdx.x, nt = blockDim.x, mp = m + (m & 1);
  int sw = 0, cur = 0;
  while (true) {
    // and the lower triangle made the mirror of the upper one again (the rotations keep them equal
    // only to rounding, which would add up over the sweeps)
    z64* h = hs + cur * LD * LD;
    bool hit = false;
    for (int idx = t; idx < LD * LD; idx += nt) {
      const int i = idx / LD, j = idx % LD;
      if (i < j && j < m) {
        const z64 g = h[idx];
        h[j * LD + i] = cconj(g);
        hit = hit || rot_needed<REL>(h[i * (LD + 1)].re, h[j * (LD + 1)].re, cabs2(g), jt);
      }
    }
    if (hit) pending[sw & 1] = 1;
    if (t == 0) pending[(sw + 1) & 1] = 0;  // last read a whole sweep ago
    __syncthreads();
    *conv = !pending[sw & 1];
    if (*conv || sw == max_sweeps) break;
    if constexpr (HM == 16) {  // 31 steps whatever m: 0.44 against 0.69 us per step in round-robin order
      jacobi_intra_steps<REL, false>(h, hs + (cur ^ 1) * LD * LD, v, jt);
      cur ^= 1;
      jacobi_ib_steps<REL>(hs + cur * LD * LD, hs + (cur ^ 1) * LD * LD, v, v, jt);
      __syncthreads();
    } else {
      cur ^= jacobi_rr_steps<HM, REL>(h, hs + (cur ^ 1) * LD * LD, v, mp, jt);
    }
    ++sw;
  }
  *sweeps = sw;
  return hs + cur * LD * LD;
}

// Trace of |diagonal| of the m x m matrix h (leading dimension LD) by wave 0 into *out (LDS); the caller's
// barrier makes it visible.
template <int LD>
__device__ __forceinline__ void jacobi_trace(const z64* h, int m, double* out) {
  const int t = threadIdx.x;
  if (t < 64) {
    double tr = t < m ? fabs(h[t * (LD + 1)].re) : 0.0;
    for (int off = 32; off > 0; off >>= 1) tr += __shfl_xor(tr, off, 64);
    if (t == 0) *out = tr;
  }
}

// Four MFMAs of one complex 16x16x4 product: acc += a b.
__device__ __forceinline__ void mma4(z64 a, z64 b, d4& accr, d4& acci) {
  accr = __builtin_amdgcn_mfma_f64_16x16x4f64(a.re, b.re, accr, 0, 0, 0);
  acci = __builtin_amdgcn_mfma_f64_16x16x4f64(a.re, b.im, acci, 0, 0, 0);
  accr = __builtin_amdgcn_mfma_f64_16x16x4f64(-a.im, b.im, accr, 0, 0, 0);
  acci = __builtin_amdgcn_mfma_f64_16x16x4f64(a.im, b.re, acci, 0, 0, 0);
}

}  // namespace
}  // namespace gc
