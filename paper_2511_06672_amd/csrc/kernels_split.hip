// The whole split of a small matrix in one launch (§2.4: truncation by SVD).
//
// A matrix M (p x q) whose smaller side m is at most 32 goes through the steps of the general
// factorisation in one workgroup: Gram G = W W^H of the wide orientation W (M or M^H, m x kW), Jacobi
// sweeps in LDS, B = U^H W with its row norms, descending sort and truncation rule, the
// relative-accuracy second pass on B B^H where a kept value calls for it, and the two factors.  As
// separate launches (Gram, eigensolver, B, norms, rule, factors, with a copied read-back before the
// last) such a split took 23 us from the Gram to the rule at m <= 8 (7 us now), 55 at m <= 16 (24) and
// 200 at 17 to 32 (130), averaged over circuits; most bonds of lightly entangled circuits are this
// small.  The larger side is limited because one workgroup then forms all of B: at 27 x 400 a call
// takes 0.27 ms, a tenth of it the products.
//
// What bounds it: the Jacobi sweeps (m = 27: 8 sweeps of 31 dependent steps), then latency.  The Gram
// and B products run on FP64 MFMA with operands read straight from global memory: the A operand of
// W W^H, conjugated, is its own B operand, so each element is loaded once per wave.
#include <algorithm>

#include "jacobi.h"
#include "kernels.h"

namespace gc {

namespace {

// Element (i, c) of W at p[i * ri + c * ci], its imaginary part times sg (M^H is read through its
// strides).
struct WView {
  const z64* p;
  size_t ri, ci;
  double sg;
  int m, kw;
  __device__ __forceinline__ z64 at(int i, int c) const {
    if (i >= m || c >= kw) return z64{0.0, 0.0};
    const z64 x = p[i * ri + c * ci];
    return z64{x.re, sg * x.im};
  }
};

// hs[0..LD^2) <- W W^H (upper triangle; real diagonal).  The pool hs..hs + 3 LD^2 (HM = 16) or 4 LD^2
// (HM = 8) holds the waves' partial sums: K is dealt to four groups of waves, a group's first wave
// taking the tiles of rows 0..15, its second the one of rows 16..31.
template <int HM>
__device__ __forceinline__ void small_gram(const WView& w, z64* hs) {
  constexpr int LD = 2 * HM;
  const int t = threadIdx.x, lane = t & 63, lo = lane & 15, hi = lane >> 4, wv = t >> 6;
  const int grp = HM == 16 ? wv >> 1 : wv, part = HM == 16 ? wv & 1 : 0;
  d4 r0 = {0, 0, 0, 0}, i0 = r0, r1 = r0, i1 = r0;
  const int steps = (w.kw + 3) / 4;
  for (int s = grp; s < steps; s += 4) {
    const int c = 4 * s + hi;
    const z64 hib = HM == 16 ? w.at(16 + lo, c) : z64{0.0, 0.0};
    if (part == 0) {
      const z64 lob = w.at(lo, c);
      mma4(lob, cconj(lob), r0, i0);
      if (HM == 16) mma4(lob, cconj(hib), r1, i1);
    } else {
      mma4(hib, cconj(hib), r0, i0);
    }
  }
  // partial tiles: group * 768 + {0: (0, 0), 256: (0, 1), 512: (1, 1)} (HM = 8: group * 256)
  z64* out = hs + grp * (HM == 16 ? 768 : 256) + (part ? 512 : 0);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int row = mfma_row_f64(lane, q);
    out[row * 16 + lo] = z64{r0[q], i0[q]};
    if (HM == 16 && part == 0) out[256 + row * 16 + lo] = z64{r1[q], i1[q]};
  }
  __syncthreads();
  constexpr int PER = (LD * LD + 2 * HM * HM - 1) / (2 * HM * HM);  // elements per thread, 2 HM^2 threads and more
  z64 x[PER];
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const int idx = t + u * blockDim.x, i = idx / LD, j = idx % LD;
    x[u] = z64{0.0, 0.0};
    if (idx < LD * LD && i <= j) {
      const int at = HM == 16 ? (j < 16 ? 0 : i < 16 ? 256 : 512) + (i & 15) * 16 + (j & 15) : i * 16 + j;
      constexpr int GS = HM == 16 ? 768 : 256;
      x[u] = cadd(cadd(hs[at], hs[GS + at]), cadd(hs[2 * GS + at], hs[3 * GS + at]));
      if (i == j) x[u].im = 0.0;
    }
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const int idx = t + u * blockDim.x;
    if (idx < LD * LD) hs[idx] = x[u];
  }
}

// B (m x kw, row-major) <- v^H W, and its squared row norms (the waves' parts summed in a fixed order)
// into norms[0..m).  B may be W's own storage: a wave reads the 16 columns it writes and no other.
template <int HM>
__device__ __forceinline__ void small_apply(const WView& w, const z64* v, z64* B, double (*part)[2 * HM],
                                            double* norms) {
  constexpr int LD = 2 * HM, RH = LD / 16, KS = LD / 4;
  const int t = threadIdx.x, lane = t & 63, lo = lane & 15, hi = lane >> 4, wv = t >> 6, nw = blockDim.x >> 6;
  double nrm[RH][4];
#pragma unroll
  for (int rh = 0; rh < RH; ++rh)
#pragma unroll
    for (int q = 0; q < 4; ++q) nrm[rh][q] = 0.0;
  for (int c0 = 16 * wv; c0 < w.kw; c0 += 16 * nw) {
    z64 b[KS];
#pragma unroll
    for (int j = 0; j < KS; ++j) b[j] = w.at(4 * j + hi, c0 + lo);
    d4 xr[RH], xi[RH];
#pragma unroll
    for (int rh = 0; rh < RH; ++rh) {
      xr[rh] = xi[rh] = d4{0, 0, 0, 0};
#pragma unroll
      for (int j = 0; j < KS; ++j) mma4(cconj(v[(4 * j + hi) * LD + 16 * rh + lo]), b[j], xr[rh], xi[rh]);
    }
#pragma unroll
    for (int rh = 0; rh < RH; ++rh)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int row = 16 * rh + mfma_row_f64(lane, q);
        nrm[rh][q] += xr[rh][q] * xr[rh][q] + xi[rh][q] * xi[rh][q];  // zero beyond kw and m
        if (row < w.m && c0 + lo < w.kw) B[(size_t)row * w.kw + c0 + lo] = z64{xr[rh][q], xi[rh][q]};
      }
  }
#pragma unroll
  for (int rh = 0; rh < RH; ++rh)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      double x = nrm[rh][q];
      for (int off = 8; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
      if (lo == 0) part[wv][16 * rh + mfma_row_f64(lane, q)] = x;
    }
  __syncthreads();
  if (t < w.m) {
    double x = 0.0;
    for (int k = 0; k < nw; ++k) x += part[k][t];
    norms[t] = x;
  }
}

struct Rule {
  int kept, flagged, need2;
  double eps, lam_max;
};

// The truncation rule on squared values key[0..m), m < 64, by wave 0 (see k_trunc for the rule): sorted
// order into perm, sorted sigma into sig (LDS), the decision into *out.
__device__ __forceinline__ void small_rule(const double* key_in, int m, const SplitRule& ru, int* perm, double* sig,
                                           Rule* out) {
  const int lane = threadIdx.x & 63;
  const double mine = lane < m ? fmax(key_in[lane], 0.0) : -1.0;
  int rank = 0;
  for (int j = 0; j < m; ++j) {
    const double o = __shfl(mine, j, 64);
    rank += (o > mine || (o == mine && j < lane)) ? 1 : 0;
  }
  if (lane < m) {
    perm[rank] = lane;
    sig[rank] = mine;
  }
  __builtin_amdgcn_wave_barrier();
  __threadfence_block();
  const double key = lane < m ? sig[lane] : 0.0;
  double tail = key;  // sum of the values from this one on, smallest first
  for (int off = 1; off < 64; off <<= 1) {
    const double o = __shfl_down(tail, off, 64);
    if (lane + off < 64) tail += o;
  }
  const double total = __shfl(tail, 0, 64), w = tail / total, s = sqrt(key);
  const double s0 = __shfl(s, 0, 64), prev = __shfl_up(s, 1, 64);
  const unsigned long long cut = __ballot(lane >= 1 && lane < m && w <= ru.cutoff);
  const unsigned long long above = __ballot(lane < m && s > 1e-13 * s0);
  const unsigned long long apart = __ballot(lane >= 1 && lane < m && !(s >= prev * (1.0 - 1e-10)));
  const int kcut = cut ? __ffsll(cut) - 1 : m, kfloor = __popcll(above);
  int k, flagged = 0;
  if (ru.mode == 1) {
    k = max(kfloor, 1);
  } else {
    k = max(min(min(kcut, kfloor), ru.chi_max), 1);
    if (k < m && k < kfloor && !((apart >> k) & 1)) {  // the cut splits a degenerate block: drop the whole block
      const unsigned long long below = apart & ((1ull << k) - 1);
      if (below)
        k = 63 - __clzll(below);
      else
        flagged = 1;
    }
  }
  if (ru.force_k > 0) {
    k = min(ru.force_k, m);
    flagged = 0;
  }
  const double eps = __shfl(w, k, 64), kk = __shfl(key, k - 1, 64);  // lane m (m < 64) holds an empty tail
  if (lane < m) sig[lane] = s;
  if (lane == 0) *out = Rule{k, flagged, kk < 1e-12 * key ? 1 : 0, eps, key};
}

template <int HM>
__global__ __launch_bounds__(2 * HM * HM < 256 ? 256 : 2 * HM * HM) void k_split_small(SplitArgs a, JacobiCrit c1,
                                                                                            JacobiCrit c2) {
  constexpr int LD = 2 * HM, NT = 2 * HM * HM < 256 ? 256 : 2 * HM * HM, NW = NT / 64;
  constexpr int POOL = HM == 16 ? 3 * LD * LD : 4 * LD * LD;
  __shared__ __align__(16) z64 pool[POOL];  // two matrix buffers and the accumulator; the Gram's partial sums
  __shared__ double part[NW][LD], norms[LD], sig[LD], trace;
  __shared__ int perm[LD], pending[2];
  __shared__ Rule rule;
  z64* v = pool + 2 * LD * LD;
  const int t = threadIdx.x;
  const bool wide = a.p <= a.q;
  const int m = wide ? a.p : a.q, kw = wide ? a.q : a.p;
  const long long t0 = wall_clock64();
  WView w = wide ? WView{a.M, (size_t)a.q, 1, 1.0, m, kw} : WView{a.M, 1, (size_t)a.q, -1.0, m, kw};
  int sweeps = 0;
  bool conv = false;
  int pass2 = 0;
  for (int pass = 0; pass < 2; ++pass) {
    const JacobiCrit& cr = pass ? c2 : c1;
    small_gram<HM>(w, pool);
    for (int idx = t; idx < LD * LD; idx += NT) v[idx] = z64{(idx / LD == idx % LD) ? 1.0 : 0.0, 0.0};
    if (t < 2) pending[t] = 0;
    __syncthreads();
    jacobi_trace<LD>(pool, m, &trace);
    __syncthreads();
    const JacobiThr jt = jacobi_thr(trace, cr.tol, cr.skip_rel, pass, cr.floor_rel);
    if (pass)
      jacobi_sweeps<HM, true>(pool, v, m, jt, cr.max_sweeps, pending, &sweeps, &conv);
    else
      jacobi_sweeps<HM, false>(pool, v, m, jt, cr.max_sweeps, pending, &sweeps, &conv);
    if (pass == 0) {
      for (int idx = t; idx < m * m; idx += NT) a.U[idx] = v[(idx / m) * LD + idx % m];
    } else {  // U <- U Z
      constexpr int PER = (LD * LD + NT - 1) / NT;
      z64 x[PER];
#pragma unroll
      for (int u = 0; u < PER; ++u) {
        const int idx = t + u * NT;
        x[u] = z64{0.0, 0.0};
        if (idx < m * m)
          for (int j = 0; j < m; ++j) x[u] = cadd(x[u], cmul(a.U[(idx / m) * m + j], v[j * LD + idx % m]));
      }
      __syncthreads();
#pragma unroll
      for (int u = 0; u < PER; ++u)
        if (t + u * NT < m * m) a.U[t + u * NT] = x[u];
    }
    small_apply<HM>(w, v, a.B, part, norms);
    __syncthreads();
    if (t < 64) small_rule(norms, m, a.rule, perm, sig, &rule);
    __syncthreads();  // also: U and B written
    if (pass == 1 || !(a.force_pass2 >= 0 ? a.force_pass2 : rule.need2) || !conv) break;
    w = WView{a.B, (size_t)kw, 1, 1.0, m, kw};
    pass2 = 1;
  }
  const long long t1 = wall_clock64();
  // the factors (see k_emit for the four cases)
  const int k = rule.kept;
  if (t < 64) {
    double s = t < k ? sig[t] * sig[t] : 0.0;
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
    if (t == 0) trace = a.renorm ? 1.0 / sqrt(s) : 1.0;
  }
  __syncthreads();
  const double rn = trace;
  for (int idx = t; idx < a.p * k; idx += NT) {
    const int i = idx / k, j = idx - i * k, pj = perm[j];
    a.L[idx] = wide ? cscale(a.U[i * m + pj], a.left ? 1.0 : sig[j] * rn)
                    : cscale(cconj(a.B[(size_t)pj * kw + i]), a.left ? 1.0 / sig[j] : rn);
  }
  for (int idx = t; idx < k * a.q; idx += NT) {
    const int j = idx / a.q, c = idx - j * a.q, pj = perm[j];
    a.R[idx] = wide ? cscale(a.B[(size_t)pj * kw + c], a.left ? rn : 1.0 / sig[j])
                    : cscale(cconj(a.U[c * m + pj]), a.left ? sig[j] * rn : 1.0);
  }
  if (t < m) {
    a.sig[t] = sig[t];
    a.perm[t] = perm[t];
  }
  if (t == 0) {
    DevStatus s = *a.st;  // keeps the selection's fields
    s.kept = k;
    s.eps = rule.eps;
    s.flagged = rule.flagged;
    s.need_pass2 = rule.need2;
    s.lam_max = rule.lam_max;
    s.converged = conv ? 1 : 0;
    s.sweeps = sweeps;
    s.pass2 = pass2;
    s.ticks = t1 - t0;
    *a.st = s;
    s.ticket = 0;
    *a.host_st = s;
    announce(&a.host_st->ticket, a.ticket);
  }
}

}  // namespace

void launch_split_small(hipStream_t s, const SplitArgs& a) {
  const int m = std::min(a.p, a.q);
  GC_CHECK(m >= 1 && m <= kSmallEig, GCAMPS_ECAPACITY, "small split: matrix side exceeds 32");
  const JacobiCrit c1 = jacobi_crit(m, 0), c2 = jacobi_crit(m, 1);
  if (m <= 16)
    hipLaunchKernelGGL((k_split_small<8>), dim3(1), dim3(256), 0, s, a, c1, c2);
  else
    hipLaunchKernelGGL((k_split_small<16>), dim3(1), dim3(512), 0, s, a, c1, c2);
  GC_LAUNCH_CHECK();
}

}  // namespace gc
