// Launch wrappers of the HIP kernels (one definition per .hip translation unit).
#pragma once

#include <chrono>

#include "internal.h"

namespace gc {

// Waits until the launch with ticket `want` has announced its results (slot: in pinned coherent memory).
// Polling returns 5 us earlier than a wait for the stream (an expectation of one launch: 53 against 58 us);
// after kPollMs the stream is waited for, which also reports a launch that failed.
constexpr int kPollMs = 2;
inline void await_ticket(hipStream_t s, const Ticket& slot, Ticket want) {
  const auto t0 = std::chrono::steady_clock::now();
  for (int i = 1; __atomic_load_n(&slot, __ATOMIC_ACQUIRE) != want; ++i) {
    __builtin_ia32_pause();
    if ((i & 63) == 0 && std::chrono::steady_clock::now() - t0 > std::chrono::milliseconds(kPollMs)) {
      GC_HIP(hipStreamSynchronize(s));
      GC_CHECK(__atomic_load_n(&slot, __ATOMIC_ACQUIRE) == want, GCAMPS_EDEVICE, "a launch left no result");
      return;
    }
  }
}

// ------------------------------------------------------------------ tableau (kernels_tableau.hip)
// Device tableau: tx[2n*n], tz[2n*n], tp[2n] (row r, site i at r*n + i); exponents in [0,d),
// phases in [0,2d).
void launch_tableau_init(hipStream_t s, int n, int* tx, int* tz, int* tp);
void launch_tableau_layer(hipStream_t s, int n, int d, int count, const int* sites,
                          const uint32_t* luts, int* tx, int* tz, int* tp);
// P = C^dagger W C for the target W; out may be host memory that the device addresses.
void launch_weyl_extract(hipStream_t s, int n, int d, const int* tx, const int* tz, const int* tp,
                         const WeylTarget& target, DevWeyl* out, Ticket ticket);

// ------------------------------------------------------------------ expectation (kernels_expect.hip)
// A run of sites whose tensors have at most kExpectMaxSite entries and whose bonds at most kExpectMaxBond2
// entries squared is contracted by one workgroup with E, A and E A in LDS (152 of 160 KB).  The line is what
// fits: at bond 32, d = 3 a site costs it 11 us of matrix instructions at the single CU's rate, against three
// launches of 6 us each for the form on the whole chip.
constexpr int kExpectMaxSite = 4096;
constexpr int kExpectMaxBond2 = 1600;
struct ExpectResult {
  z64 value;  // without the phase of P
  int32_t p;  // tau exponent of P's phase
  Ticket ticket;
};
struct ExpectArgs {
  int n, d, first, last;
  int extract;            // commute target through the tableau (else P is *weyl)
  const int *tx, *tz, *tp;
  DevWeyl* weyl;          // P, written when extract and not null
  const z64* e_in;        // left environment (chi x chi, row-major) at `first`; null: 1
  z64* e_out;             // environment at `last`, when not null
  Ticket ticket;
  ExpectResult* result;   // at the end of the chain, when not null (host memory that the device addresses)
  WeylTarget target;
  int chi[kMaxN + 1];
  const z64* site[kMaxN];
};
void launch_expect_chain(hipStream_t s, const ExpectArgs& a);
// out = the site tensor with the conjugate of P's factor at `site` applied from the bra's side:
// out[(al, t), b] = conj(omega^{z t}) in[(al, t + x), b].
void launch_weyl_site(hipStream_t s, int d, int chil, int chir, int site, const DevWeyl* P, const z64* in, z64* out);
void expect_set_attributes();

// ------------------------------------------------------------------ dense linear algebra
// C = alpha * op(A) op(B) (+ C if accumulate); row-major, complex128; op 0 = N, 1 = conj-transpose.
// herm != 0: C is Hermitian (M == N, op(B) = op(A)^H): only the upper triangle is computed and
// mirrored.
void launch_zgemm(hipStream_t s, int opa, int opb, int M, int N, int K, const z64* A, int lda,
                  const z64* B, int ldb, z64* C, int ldc, z64 alpha, int accumulate, int herm);
// Hermitian eigen-decomposition by two-sided Jacobi.  G (m x m, ld ldg) is destroyed (holds
// the rotated matrix, padded to mp x mp with ld mp in the block variant); U (ld ldu) receives
// eigenvectors, lam the eigenvalues (unsorted).  rel: relative-accuracy criterion.
// What a sweep's rounds tell the host: whether the sweep before rotated anything, and the ticket of their launch.
struct SweepReport {
  int32_t rotated;
  Ticket ticket;
};
struct EigWork {
  z64* G;      // three padded m_pad x m_pad planes: matrix, accumulator, second matrix buffer
  z64* V;      // block rotations (two rounds)
  z64* D;      // solved sub-problems (two rounds)
  int* flags;  // device flags
  int m_pad;
  double* host_rb;            // pinned host read-back slots (2 doubles)
  SweepReport *report, *report_dev;  // in pinned coherent host memory: what the host and the device address
  Ticket* ticket;             // the context's ticket counter
};
// Criteria of the sweeps.  Absolute criterion 3e-16 of the trace: what stays off the diagonal tilts a
// factor's columns by up to 3e-16 trace / lambda (1.1e-12 at 4e-15 on a Gaussian 300 x 97), and the kept space by
// that over the gap at a cut: over 24 gates of qutrit bonds up to 243 the fidelity estimate differed from the
// oracle's by up to 1.9e-10 of itself at 2e-15 and by 1.2e-11 at 2e-16.  The convergence is quadratic, so the
// tighter bound takes no further sweep (m = 48 to 243: equal times to 0.5%); rotations of degenerate
// pairs leave about 1e-16 of the trace.  A Rayleigh-Ritz step that is skipped keeps to this bound only between
// directions that the truncation may part (discardable, eig_hermitian).
struct JacobiCrit {
  double tol, skip_rel, floor_rel;
  int max_sweeps;
};
inline JacobiCrit jacobi_crit(int m, int rel) {
  // Relative pass: pairs whose diagonal entries are both below 1e-28 lambda_max (lambda_max >=
  // trace / m) are left alone.  They lie two decades below the rank floor (sigma^2 = 1e-26
  // sigma_0^2), so no decision depends on them, and exact null directions sit at the rounding
  // level (~1e-32 of the trace), where a relative criterion cannot be met.
  // An off-diagonal entry of at most 1e-29 trace / m (<= 1e-29 lambda_max) counts as converged
  // there.  On exactly rank-deficient matrices the rounding of the rotations keeps entries of that
  // size alive between directions at the rounding level, where a relative criterion is never met
  // (the pass then ran out of sweeps); an eigenvalue at or above the rank floor (1e-26 lambda_max)
  // moves by at most 1e-3 of itself because of such an entry.
  // Sweeps grow with m on these Grams: up to ~20 at m = 768, 19-26 at m = 3072, where one
  // decomposition needed more than 40 (every sub-problem still rotating for the first ~20
  // sweeps, then a steady decay).
  return JacobiCrit{rel ? 1e-14 : 3e-16, rel ? 1e-28 / (double)m : 0.0, rel ? 1e-29 / (double)m : 0.0,
                    m > 1024 ? 100 : 40};
}
// Offsets in a context's pinned read-back block: device status, pivoted and plain Cholesky
// states, eigensolver slots, conjugated Weyl string and its error flag.
constexpr size_t kRbStatus = 0, kRbPcState = 256, kRbChol = 384, kRbEig = 512, kRbWeyl = 1024, kRbExpect = 2560, kRbCommit = 2816, kRbSweep = 2880, kRbBytes = 4096;
// discardable >= 0 (for matrices expected to be diagonal already, as of a Rayleigh-Ritz step; absolute criterion,
// m > kSmallEig): every pair is tested first, and U = I, lam = diag(G) are returned without a sweep when no
// entry exceeds kPrecheckTol and none that exceeds the sweeps' own bound turns a direction of at most
// `discardable` of the trace, which the truncation rule may drop, by more than kPrecheckTilt (kernels_linalg.hip).
void eig_hermitian(hipStream_t s, const z64* G, int m, int ldg, z64* U, int ldu, double* lam,
                   int rel, EigWork& w, DevStatus* st, int* host_sweeps, double discardable = -1.0);
void launch_rownorm2(hipStream_t s, const z64* B, int m, int k, int ldb, double* out);
// Sort, truncation rule, pass-2 decision.  mode 0 = truncate (cutoff, chi_max), 1 = floor only;
// force_k > 0 keeps exactly that rank (frozen-decision replay).
// extra (nullable, device): weight of directions outside sig2 that are discarded whatever the
// rule (a rank reduction's remainder), added to every tail sum and to the total.
void launch_trunc(hipStream_t s, const double* sig2, int m, double cutoff, int chi_max, int mode,
                  int force_k, int* perm, double* sig_sorted, DevStatus* st, const double* extra = nullptr);
// Write the two factors (see kernels_linalg.hip for the case table).
void launch_emit(hipStream_t s, int wide, int left_ortho, int renorm, int p, int q, int kept,
                 const z64* U, int ldu, const z64* B, int ldb, const int* perm, const double* sig,
                 z64* L, z64* R);
// The whole split of a matrix M (p x q, smaller side m <= kSmallEig) in one launch: M -> L (p x kept),
// R (kept x q) as launch_emit writes them, by the rule of launch_trunc, with the relative-accuracy second
// pass where a kept value calls for it (force_pass2: -1, or the recorded decision).  U (m x m), B (m x the
// larger side), sig and perm are left as the general factorisation leaves them; *st and *host_st
// (pinned host memory as the device addresses it) get the decision, with the selection's fields of *st kept.
struct SplitRule {
  double cutoff;
  int chi_max, mode, force_k;
};
struct SplitArgs {
  const z64* M;
  int p, q, left, renorm, force_pass2;
  SplitRule rule;
  z64 *U, *B, *L, *R;
  double* sig;
  int* perm;
  DevStatus *st, *host_st;
  Ticket ticket;  // announced in *host_st
};
void launch_split_small(hipStream_t s, const SplitArgs& a);
void launch_copy(hipStream_t s, z64* dst, const z64* src, size_t count);
void launch_fill_identity(hipStream_t s, z64* U, int m, int ld);

// ------------------------------------------------------------------ rank reduction (kernels_reduce.hip)
// Pivoted Cholesky of the Hermitian PSD G (m x m, ld ldg; destroyed: it ends as the Schur
// complement): G = L L^H + S with L (m x r, ld ldl) and tr S <= tol_rel * tr G, or r = rmax
// columns without meeting the bound (then *host_state.done == 0).  dvec (m doubles) and pv
// (m ints) are scratch; stt is a device PcState.  Returns r; host_state receives the final state
// (tres = tr S).
struct PcState {
  int32_t r, done, pad0, pad1;
  double trace, tres;
};
int pchol_reduce(hipStream_t s, z64* G, int m, int ldg, z64* L, int ldl, double tol_rel, int rmax, double* dvec,
                 int* pv, PcState* stt, PcState* host_state);
// Columns of X (m x r, ld ldx) scaled to unit 2-norm.
void launch_normalize_cols(hipStream_t s, z64* X, int m, int r, int ldx);
// X (m x r, ld r) replaced by its polar factor by `iters` Newton-Schulz steps (X nearly
// orthonormal); Xn (m x r) and S (r x r) are scratch.
void orthonormalize_cols(hipStream_t s, z64* X, z64* Xn, z64* S, int m, int r, int iters);

// dst = f * src.
void launch_scaled_copy(hipStream_t s, z64* dst, const z64* src, size_t count, double f);

// ------------------------------------------------------------------ exact moves (kernels_chol.hip)
// Pivots of a Cholesky factorisation (largest diagonal entry of the matrix, smallest pivot) and the
// largest row sum of |S - I| seen by launch_identity_gap, which bounds the spectral norm of a Hermitian S - I.
struct CholState {
  double dmax, dmin, emax;
};
// Cholesky elimination of A's first m columns: rows 0..m hold the Hermitian G = K K^H (ld m; destroyed), rows
// m..rows a matrix X that ends as X K^-H.  st receives the pivots; a pivot that is not positive
// leaves dmin = 0 and finite garbage.
void launch_cholesky(hipStream_t s, z64* A, int m, int rows, CholState* st);
void launch_identity_gap(hipStream_t s, const z64* S, int m, CholState* st);
// dst (q x p) = src^H (src p x q).
void launch_conj_transpose(hipStream_t s, const z64* src, int p, int q, z64* dst);

// ------------------------------------------------------------------ MPS kernels (kernels_mps.hip)
struct MpoCoeff {
  z64 k[kMaxD];       // c_b tau^{phase of P^b}
  z64 w[kMaxD];       // omega^j, j = 0..d-1
};
// Block-MPO site update.  kind: 0 = left end (opens the b index), 1 = interior, 2 = right end,
// 3 = local operator (l == r).  (dx, dz): exponents of P on this site.
void launch_mpo_site(hipStream_t s, int kind, int d, int chil, int chir, int dx, int dz,
                     const MpoCoeff& coeff, const z64* in, z64* out);
// Site update of the MPO sum_j coef_j (x)_i X^{x_ji} Z^{z_ji} of bond J (one term per bond
// index): kind as above; xz[2j], xz[2j+1] are the exponents of term j on this site; coef is
// used by kinds 0 and 3 only.
struct MpoTerms {
  int x[kMaxGateTerms], z[kMaxGateTerms];
  z64 coef[kMaxGateTerms];
};
void launch_mpo_sum_site(hipStream_t s, int kind, int d, int J, int chil, int chir, const MpoTerms& terms,
                         const z64* in, z64* out);
// out = Q_c Theta for the candidate c given by the host (a copy for c == 0).
void launch_rotate_copy(hipStream_t s, int d, int chil, int chir, int c, const z64* qmats, const z64* theta,
                        z64* out);
// Candidate scores S2_c for the candidates cand_list[0..count) (or 0..count when cand_list is
// null), in the arithmetic of `prec` (GCAMPS_SCORE_*; REPLICA takes the full set only and
// needs replica_tables).  nlimit (nullable): device count that
// overrides `count` (the list length is then only known on the device).  partial: scratch of
// count * tiles doubles for the tiled path; nbuf: scratch for the rotated matrices of a chunk
// of candidates (the tiled path processes as many candidates per launch as fit).  evs: optional
// event pairs recorded around each Gram-purity launch (count returned in *evused).
void launch_score(hipStream_t s, int prec, int d, int chil, int chir, const z64* theta,
                  const z64* q64, const c32* q32, const int* cand_list, int count,
                  const int* nlimit, double* s2, double* partial, size_t partial_cap, void* nbuf,
                  size_t nbuf_bytes, hipEvent_t* evs = nullptr, int evcap = 0, int* evused = nullptr,
                  const z64* replica_tables = nullptr, int64_t* tick = nullptr);

// ------------------------------------------------------------------ commit of a bond (kernels_commit.hip)
// The choice: the lowest index with s2 <= min s2 + tol over the candidates 0..count, or over the
// st->nwindow entries of list (s2 per entry); with ranks, over the candidates of the smallest rank and only
// if that is below the identity's (else 0).  c* goes to st->cstar and *host, the minimum to st->s2min.
struct CommitResult {
  int32_t cstar;
  Ticket ticket;
};
struct CommitRule {
  int fixed;          // >= 0: this candidate, nothing is chosen and neither tableau nor status is written
  int count;
  const double* s2;
  const int* list;    // window, or null
  const int* rank;    // bond dimension per candidate, or null
  double tol;
  int64_t* tick;      // the wall clock at the start goes there, when not null
  DevStatus* st;
  CommitResult* host;  // host memory that the device addresses
  Ticket ticket;
};
struct CommitTableau {
  int n, site;
  const uint32_t* inv_luts;
  int *tx, *tz, *tp;
};
// Theta <- Q_{c*} Theta in place, Theta (chil, d, d, chir), and the tableau C <- C Q_{c*}^dagger.
void launch_commit(hipStream_t s, int d, const CommitRule& r, int chil, int chir, const z64* qmats, z64* theta,
                   const CommitTableau& tb);

// ------------------------------------------------------------------ bond-dimension criterion (kernels_rank.hip)
constexpr int kRankMaxM = 32;        // smaller side of the two-site matrix
constexpr int kRankMaxElems = 8192;  // entries of the two-site matrix (LDS of one workgroup)
// rank_out[c] = bond dimension left by candidate c (truncation rule of the split applied to the
// singular values of reshape(Q_c Theta), one-sided Jacobi SVD per candidate).
void launch_cand_rank(hipStream_t s, int d, int chil, int chir, const z64* theta, const z64* qmats, int count,
                      double cutoff, int chi_max, int* rank_out, int64_t* tick);
void rank_set_attributes();
void linalg_set_attributes();  // the block-Jacobi rounds' dynamic LDS limit

// ------------------------------------------------------------------ density scoring (kernels_density.hip)
// Scores through the two-site reduced density matrix F of Theta over its larger bond (d = 2, 3): one
// Gram of Theta, then a matrix product against the candidates' rows T_c for every pair of smaller-bond
// indices, |rho_c|^2 summed as it is formed.
size_t density_table_elems(int d, int count);  // rows T_c of both cuts; 0 for d > 3
void launch_density_tables(hipStream_t s, int d, int count, const z64* qmats, z64* tab, c32* tab32);
// Whether F and at least one block's partial sums of `count` candidates fit the scratch.
bool density_fits(int d, int chil, int chir, int count, size_t scratch_bytes);
// F of Theta at the start of the scratch (kept for the scores that follow).
void launch_density_gram(hipStream_t s, int d, int chil, int chir, const z64* theta, void* scratch);
// S2 of the candidates (list and nlimit as in launch_score) from F; set_count: candidates in the tables;
// events around the product's launch when given.
void launch_density_score(hipStream_t s, int d, bool fp32, int chil, int chir, const z64* tab, const c32* tab32,
                          int set_count, const int* list, int count, const int* nlimit, double* s2, void* scratch,
                          size_t scratch_bytes, hipEvent_t ev0, hipEvent_t ev1);

// ------------------------------------------------------------------ replica scoring (kernels_replica.hip)
// Full-set scores through the replica tensor of Theta (d = 2, 3): the Gram F of Theta over its
// larger bond, the pair sum A, and one D^4 dot product per candidate with its table.
constexpr int kReplicaMaxWg = 256;  // workgroups (partial sums) of the pair sum
constexpr int kScoreSmallM = 96;    // matrices up to this many rows are scored directly (fused kernel)
// complex128 elements of the tables of `count` candidates (left-cut and right-cut tables).
size_t replica_table_elems(int d, int count);
// Scratch bytes for bonds up to chi_max (F, the transposed Theta, partial sums, A).
size_t replica_scratch_bytes(int d, int chi_max);
// tables <- symmetrised V tables of the candidates qmats[0..count) (d^2 x d^2 unitaries).
void launch_replica_tables(hipStream_t s, int d, int count, const z64* qmats, z64* tables);
void launch_score_replica(hipStream_t s, int d, int chil, int chir, const z64* theta, const z64* tables,
                          int count, double* s2, void* scratch, size_t scratch_bytes);
// Low-precision window: list (ascending index) of candidates with s2lp <= min + window; the
// list length goes to st->nwindow.
void launch_window(hipStream_t s, int count, const double* s2lp, double window, int* list,
                   DevStatus* st, int64_t* tick);

// ------------------------------------------------------------------ dense state (kernels_dense.hip)
// v <- C|0> for the tableau's Clifford C, not normalised (norm2 = its squared norm): the stabilizer
// projectors applied to a fixed generic vector.  w is scratch; v and w trade places.
void launch_stab_state(hipStream_t s, int n, int d, int D, const int* tx, const int* tz, const int* tp, z64*& v,
                       z64*& w, double* norm2);
// out(y) = sum_x m(x) (C X^x C^dagger s0)(y) / sqrt(*norm2), D = d^n <= 2^16.  ab: 16 D bytes of scratch;
// m is overwritten.
void launch_clifford_dense(hipStream_t s, int n, int d, int D, const int* tx, const int* tz, const int* tp, void* ab,
                           z64* m, const z64* s0, const double* norm2, z64* out);

// ------------------------------------------------------------------ reverse sweep (kernels_adjoint.hip)
struct SitePhases {
  z64 w[kMaxD];
};
// Us, Bs, ss <- U (m x m), B (m x kW) and sig in the sorted order perm.
void launch_record(hipStream_t s, const z64* U, const z64* B, const double* sig, const int* perm, int m, int kW, z64* Us,
                   z64* Bs, double* ss);
// X (rows x cols) <- (base - X) / (sig_c^2 rn^2) per column (by_cols) or per row; *rn = 1/sqrt(sum_{j<k} sig_j^2)
// when renorm, else 1.
void launch_gauge(hipStream_t s, z64* X, const z64* base, int rows, int cols, int by_cols, const double* sig, int k,
                  int renorm, double* rn);
// Xbar = rn (Nbar - N Re<N, Nbar>), rn = scal[0]; scal[1] is scratch.
void launch_renorm_bwd(hipStream_t s, const z64* Nbar, const z64* N, size_t count, double* scal, z64* Xbar);
// Kept/discarded mixing matrix of the truncated-split adjoint (sorted basis, k kept); rows >= k of Y (m x kW)
// are cleared.
void launch_trunc_mix(hipStream_t s, const z64* G1, int m, int k, const double* sig, z64* Zc, z64* Y, int kW);
// abar[al, (t + shift) mod d, b] += cf w_t X[al, t, b] on site tensors (chil, d, chir).
void launch_site_scatter(hipStream_t s, int d, int chil, int chir, int shift, const SitePhases& w, z64 cf, const z64* X,
                         z64* abar);
// out[al, t, b] = conj(w_t) in[al, (t + shift) mod d, b].
void launch_site_gather(hipStream_t s, int d, int chil, int chir, int shift, const SitePhases& w, const z64* in, z64* out);
// Transpose of the MPO site map and the gradient of its coefficients (kinds 0 and 3).
void launch_mpo_site_bwd(hipStream_t s, int kind, int d, int chil, int chir, int dx, int dz, const MpoCoeff& co,
                         const z64* obar, z64* ibar);
void launch_mpo_coeff_bwd(hipStream_t s, int kind, int d, int chil, int chir, int dx, int dz, const MpoCoeff& co,
                          const z64* in, const z64* obar, z64* kbar);
// theta <- Q_c^dagger theta.
void launch_apply_qh(hipStream_t s, int d, int chil, int chir, int c, const z64* qmats, z64* theta);
}  // namespace gc
