// Internal declarations shared by the HIP translation units of libgcamps.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <string>
#include <vector>

#include "../../include/gcamps.h"

namespace gc {

// ----------------------------------------------------------------- complex types
template <typename T>
struct cx {
  T re, im;
};
using z64 = cx<double>;
using c32 = cx<float>;

template <typename T>
__host__ __device__ __forceinline__ cx<T> cmul(cx<T> a, cx<T> b) {
  return {a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re};
}
template <typename T>
__host__ __device__ __forceinline__ cx<T> cmulc(cx<T> a, cx<T> b) {  // conj(a) * b
  return {a.re * b.re + a.im * b.im, a.re * b.im - a.im * b.re};
}
template <typename T>
__host__ __device__ __forceinline__ cx<T> cadd(cx<T> a, cx<T> b) {
  return {a.re + b.re, a.im + b.im};
}
template <typename T>
__host__ __device__ __forceinline__ cx<T> csub(cx<T> a, cx<T> b) {
  return {a.re - b.re, a.im - b.im};
}
template <typename T>
__host__ __device__ __forceinline__ cx<T> cscale(cx<T> a, T s) {
  return {a.re * s, a.im * s};
}
template <typename T>
__host__ __device__ __forceinline__ cx<T> cconj(cx<T> a) {
  return {a.re, -a.im};
}
template <typename T>
__host__ __device__ __forceinline__ T cabs2(cx<T> a) {
  return a.re * a.re + a.im * a.im;
}

// ----------------------------------------------------------------- MFMA 16x16x4 accumulators
// Row of accumulator item q in lane `lane` (column is lane % 16).  Measured on gfx950:
// v_mfma_f64_16x16x4f64 places row 4q + lane/16, v_mfma_f32_16x16x4f32 row 4(lane/16) + q.
__device__ __forceinline__ int mfma_row_f64(int lane, int q) { return 4 * q + (lane >> 4); }
__device__ __forceinline__ int mfma_row_f32(int lane, int q) { return 4 * (lane >> 4) + q; }
template <typename T>
__device__ __forceinline__ int mfma_row(int lane, int q);
template <>
__device__ __forceinline__ int mfma_row<double>(int lane, int q) { return mfma_row_f64(lane, q); }
template <>
__device__ __forceinline__ int mfma_row<float>(int lane, int q) { return mfma_row_f32(lane, q); }

// ----------------------------------------------------------------- errors
struct Error {
  int code;
  std::string msg;
};
void set_error(const std::string& msg);

#define GC_HIP(call)                                                              \
  do {                                                                            \
    hipError_t e_ = (call);                                                       \
    if (e_ != hipSuccess)                                                         \
      throw ::gc::Error{GCAMPS_EDEVICE, std::string(#call) + ": " + hipGetErrorString(e_)}; \
  } while (0)

#define GC_CHECK(cond, code, msg)                 \
  do {                                            \
    if (!(cond)) throw ::gc::Error{(code), (msg)}; \
  } while (0)

#define GC_LAUNCH_CHECK() GC_HIP(hipGetLastError())

// ----------------------------------------------------------------- limits
inline size_t align256(size_t v) { return (v + 255) & ~size_t(255); }

constexpr int kMaxD = 7;
constexpr int kMaxGateTerms = 81;  // Weyl terms of a general gate (two qutrits: 3^4)
constexpr int kMaxN = 128;
constexpr double kNearTieLowp = 1e-4;  // smallest re-score window with FP32 / split-BF16 scoring
constexpr size_t kDenseMax = size_t(1) << 16;  // largest d^n of the dense (validation) state
constexpr int kSmallEig = 32;   // largest m handled by the single-workgroup eigensolver
constexpr int kSplitSmallMaxK = 512;  // largest larger side of a one-launch split (kernels_split.hip)
// Truncating splits with kReduceMinM < m <= kReduceMaxM take the pivoted-Cholesky path; outside, it is
// untested against the plain path's accuracy.  The lower line is not where the times cross: on graded matrices
// (singular values over five decades) the plain path takes 0.80 ms at m = 48, 1.38 at 81, 2.67 at 144, 4.79 at 243 and
// 6.40 at 320, this path 0.60, 0.65, 1.24, 2.06 and 2.82 (rank about 0.78 m; 0.96 at 81 and 2.70 at 243 with full rank).
constexpr int kReduceMinM = 320;
constexpr int kReduceMaxM = 1024;
// m^2 k (m and k the smaller and larger side of the two-site matrix) from which a bond is scored through
// the two-site density matrix (kernels_density.hip): m = 32, k = 32 (d = 2) takes 40 us through it and 70
// directly, m = 27, k = 27 (d = 3) 69 and 52, m = 27, k = 243 57 and 158.
constexpr double kDensityMinWork = 25000;
constexpr int kDensityFew = 8;  // see gcamps_ctx::density_mode
constexpr double kDensityFewWork = 3e8;
constexpr int kBlk = 16;        // block size of the multi-workgroup block Jacobi

// ----------------------------------------------------------------- results in host memory
// A kernel that ends a host decision writes its result to pinned coherent host memory and then the ticket of its
// launch beside it (announce); the host waits for the ticket instead of for the stream.
using Ticket = uint32_t;
__device__ __forceinline__ void announce(Ticket* slot, Ticket ticket) {
  __threadfence_system();
  __hip_atomic_store(slot, ticket, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// ----------------------------------------------------------------- device status block
// Written by the selection / truncation kernels, read back once per bond.
struct DevStatus {
  int32_t cstar;       // selected candidate
  int32_t kept;        // kept rank after truncation
  int32_t flagged;     // degenerate cut flag
  int32_t nwindow;     // FP32 mode: number of candidates re-scored in FP64
  int32_t converged;   // eigensolver convergence flag (1 = ok)
  int32_t need_pass2;  // factorisation needs the accurate second pass
  int32_t sweeps;      // eigensolver sweeps used
  int32_t pass2;       // small split: the second pass ran
  double eps;          // discarded relative weight
  double smin_lp;      // minimum low-precision score
  double s2min;        // minimum FP64 score
  double norm2;        // |Theta|^2 of the scored tensor
  double lam_max;      // largest Gram eigenvalue
  int64_t ticks;       // small split: wall-clock ticks from the Gram to the truncation rule
  // wall clock around the fused scoring launches, each read by the first workgroup of the launch named: score,
  // what follows it (window, ranks or commit), re-score, commit
  int64_t score_tick[4];
  Ticket ticket;       // small split: the launch that left this block
};

// Weyl string to be commuted through the tableau (exponents in [0, d)), passed to kernels by value.
struct WeylTarget {
  uint8_t x[kMaxN];
  uint8_t z[kMaxN];
  int32_t p;
};

// Weyl string result of the commutation step (device layout).
struct DevWeyl {
  int32_t x[kMaxN];
  int32_t z[kMaxN];
  int32_t p;
  int32_t l, r;
  int32_t bad;  // nonzero: the rows did not multiply out to the target
  Ticket ticket;
};

// ----------------------------------------------------------------- compiled words
// A two-qudit Clifford word compiled to its action on Weyl strings of the pair:
// lut[v] for v = ((xa*d + za)*d + xb)*d + zb packs the image (x'a, z'a, x'b, z'b)
// in the same base-d index and the tau-phase increment in bits 16..23.
struct CompiledWord {
  std::vector<uint32_t> fwd;  // U W U^dagger
  std::vector<uint32_t> inv;  // U^dagger W U
  std::vector<z64> mat;       // d^2 x d^2 unitary, row-major (row = s_a*d + s_b)
};
CompiledWord compile_word(int d, const gcamps_word& w);
// Generator words (application order) of an exhaustive two-qudit Clifford set, identity first.
std::vector<std::vector<uint8_t>> clifford_word_set(int d, int kind);

}  // namespace gc

// ----------------------------------------------------------------- candidate set
struct gcamps_candset {
  int d;
  int count;
  std::vector<gc::CompiledWord> words;
  uint64_t uid;
};
