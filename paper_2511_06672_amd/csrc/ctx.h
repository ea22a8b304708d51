// Host-side state of one GCAMPS simulation (gcamps_ctx): workspace carving, the bottom
// loop of the method (commute, MPO, compression, disentangling sweeps) and, for the
// gradient, recording and frozen replay of the same steps.
#pragma once

#include <algorithm>
#include <chrono>
#include <functional>
#include <cmath>
#include <complex>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>
#include <vector>

#include "kernels.h"

namespace gc {

struct Layout {
  size_t slot_elems, theta_elems, mcap, m_pad, ncand, ntp;
  int nslots;
  size_t off_slots, off_theta, off_G, off_U, off_Z, off_Utmp, off_B, off_B2, off_sig2, off_sig, off_lam,
      off_perm, off_eigG, off_eigV, off_eigD, off_flags, off_s2, off_s2w, off_wlist, off_partial, off_nbuf, nbuf_bytes, off_q64, off_q32,
      off_rtab, off_dtab, off_dtab32, off_qinv, off_tab, off_weyl, off_status, off_luts, off_sites, off_dense,
      dense_dim, off_pcst, off_chol, total;
};

Layout make_layout(const gcamps_config& c);

// ----------------------------------------------------------------- gradient support
// Bump allocator over a caller-provided device region (checkpoints, tape, adjoints).
struct Arena {
  char* base = nullptr;
  size_t cap = 0, used = 0, peak = 0;
  template <typename T>
  T* take(size_t count) {
    const size_t bytes = (count * sizeof(T) + 255) & ~size_t(255);
    GC_CHECK(used + bytes <= cap, GCAMPS_ECAPACITY,
             "gradient arena exhausted after " + std::to_string(used >> 20) + " MiB (pass a larger workspace)");
    T* p = reinterpret_cast<T*>(base + used);
    used += bytes;
    peak = std::max(peak, used);
    return p;
  }
};

// One factorisation as the reverse sweep needs it: W is the wide orientation of the split
// matrix M (W = M when p <= q, else M^H; m x kW), U (m x m) the eigenbasis of W W^H,
// B = U^H W, sig the singular values in descending order, perm their rows, k the kept rank.
struct FactRec {
  z64* U = nullptr;
  z64* B = nullptr;
  double* sig = nullptr;  // U's columns, B's rows and sig in descending order
  int m = 0, kW = 0, k = 0, p = 0, q = 0, wide = 0, left = 0, renorm = 0;
};

// Layout of a recorded factorisation decision (rank log entry).
constexpr int kPass2Bit = 30;
constexpr int32_t kRankMask = (1 << kPass2Bit) - 1;

enum TapeKind { TAPE_ABSORB_R = 0, TAPE_ABSORB_L = 1, TAPE_MPO = 2, TAPE_THETA = 3 };

// One step of the bottom loop, recorded for the reverse sweep.
//   ABSORB_R at i: (L, R) = split(A_i); A_i <- L; A_{i+1} <- R A_{i+1}    (x0 = old A_{i+1})
//   ABSORB_L at i: (L, R) = split(A_i); A_i <- R; A_{i-1} <- A_{i-1} L    (x0 = old A_{i-1})
//   MPO at i     : A_i <- MPO site tensor of kind mpo_kind            (x0 = old A_i, kinds 0, 3)
//   THETA at i   : (L, R) = split(Q_c A_i A_{i+1}); A_i <- L; A_{i+1} <- R (x0, x1 = old A_i, A_{i+1})
struct TapeOp {
  int kind = 0, site = 0;
  FactRec f;
  z64* x0 = nullptr;
  z64* x1 = nullptr;
  int d0[2] = {0, 0}, d1[2] = {0, 0};  // (rows, cols) of x0 and x1 as matrices
  int mpo_kind = 0, dx = 0, dz = 0, cstar = 0, chil = 0, chir = 0;
};

// Weyl string P = C^dagger W C of a gate or an observable (tau^p X^x Z^z per site) and its
// support [l, r].
struct GateRec {
  int l = 0, r = 0, p = 0, sd = 0;
  std::vector<int> x, z;
};

}  // namespace gc

using namespace gc;

struct gcamps_ctx {
  gcamps_config cfg{};
  Layout lay{};
  hipStream_t stream = nullptr;
  char* ws = nullptr;
  int d = 0, n = 0;
  bool poisoned = false;
  // device regions
  int *tx = nullptr, *tz = nullptr, *tp = nullptr, *dsites = nullptr;
  uint32_t* dluts = nullptr;
  DevWeyl* weyl = nullptr;
  DevStatus* st = nullptr;
  PcState* pcst = nullptr;  // rank-reduction state (device)
  CholState* chst = nullptr;  // pivots of an exact move (device)
  void* scratch_dev = nullptr;  // device address of the library's static scratch on this ctx's GPU
  z64 *theta = nullptr, *G = nullptr, *U = nullptr, *Z = nullptr, *Utmp = nullptr, *B = nullptr, *B2 = nullptr;
  double *sig2 = nullptr, *sig = nullptr, *lam = nullptr, *s2 = nullptr, *s2w = nullptr, *partial = nullptr;
  void* nbuf = nullptr;
  int *perm = nullptr, *wlist = nullptr;
  z64* q64 = nullptr;
  c32* q32 = nullptr;
  z64* rtab = nullptr;  // replica-scoring tables of the candidate set (replica mode only)
  z64* dtab = nullptr;    // density-scoring rows of the candidate set (d <= 3)
  c32* dtab32 = nullptr;  // the same in FP32 (FP32 and BF16 scoring)
  uint32_t* qinv = nullptr;
  EigWork eig{};
  // MPS
  std::vector<z64*> site;
  z64* Lbuf = nullptr;
  z64* Rbuf = nullptr;
  z64* spare = nullptr;
  std::vector<int> chi;  // chi[0..n], bond j between sites j-1 and j
  int centre = 0;
  // candidates
  int ncand = 0;
  uint64_t cand_uid = 0;
  // pinned staging
  char* pinned = nullptr;
  char* rb = nullptr;  // pinned read-back block (status, Cholesky state, eigensolver flags)
  Ticket ticket = 0;       // of the last launch that announces its results in rb
  char* rb_dev = nullptr;  // the same block as the device addresses it
  double tick_ms = 0.0;    // one tick of the device's wall clock in ms
  size_t pinned_bytes = 0;
  hipEvent_t stage_ev = nullptr;
  bool stage_pending = false;
  hipEvent_t ev0 = nullptr, ev1 = nullptr, ev2 = nullptr, ev3 = nullptr;
  hipEvent_t evf0 = nullptr, evf1 = nullptr;  // around one factorisation (Gram to truncation rule)
  hipEvent_t evm0 = nullptr, evm1 = nullptr;  // around one gate's MPO launches
  bool mpo_pending = false;                   // evm0/evm1 recorded and not yet accumulated
  std::vector<hipEvent_t> gram_ev;  // event pairs around the Gram-purity launches of one bond
  // host state
  double f_est = 1.0;
  std::vector<int32_t> choice_log;
  int64_t gates = 0;
  double stats[16] = {0};
  // [0] factorisations, [1] their SVD flops by the R-SVD count 4 (6 p q^2 + 20 q^3) (p >= q),
  // [2] their device ms (Gram to truncation rule, second pass included), [3] MPO site launches,
  // [4] MPO bytes (each site tensor read once and its product written once), [5] MPO device ms
  double kstats[8] = {0};
  // rank reduction of the rotated-tensor splits: [0] reduced factorisations, [1] their summed
  // basis sizes r, [2] their summed sides m, [3] attempts that fell back to the full basis
  double stats_red[4] = {0};
  int last_basis = 0;  // singular values resolved by the last factorisation (m, or r when reduced)
  bool trace_fact = std::getenv("GCAMPS_TRACE_FACT") != nullptr;
  // gradient: recording and frozen replay (all null in ordinary use)
  std::vector<int32_t>* rank_rec = nullptr;          // kept rank of every factorisation
  std::vector<GateRec>* gate_rec = nullptr;          // Weyl string of every non-Clifford gate
  const std::vector<int32_t>* rank_frz = nullptr;    // forced ranks, consumed from rank_pos
  size_t rank_pos = 0;
  const std::vector<int32_t>* choice_frz = nullptr;  // forced choices, consumed from choice_pos
  size_t choice_pos = 0;
  std::vector<TapeOp>* tape = nullptr;               // reverse-sweep record of the replayed steps
  Arena* arena = nullptr;                            // storage of the tape
  FactRec last_fact;

  ~gcamps_ctx() {
    if (pinned) (void)hipHostFree(pinned);
    if (rb) (void)hipHostFree(rb);
    if (stage_ev) (void)hipEventDestroy(stage_ev);
    if (ev0) (void)hipEventDestroy(ev0);
    if (ev1) (void)hipEventDestroy(ev1);
    if (ev2) (void)hipEventDestroy(ev2);
    if (ev3) (void)hipEventDestroy(ev3);
    for (hipEvent_t e : {evf0, evf1, evm0, evm1})
      if (e) (void)hipEventDestroy(e);
    for (auto e : gram_ev) (void)hipEventDestroy(e);
  }

  // ---------------------------------------------------------------- staging
  char* stage_begin() {
    if (stage_pending) {
      GC_HIP(hipEventSynchronize(stage_ev));
      stage_pending = false;
    }
    return pinned;
  }
  void stage_upload(void* dst, size_t bytes) {
    GC_HIP(hipMemcpyAsync(dst, pinned, bytes, hipMemcpyHostToDevice, stream));
    GC_HIP(hipEventRecord(stage_ev, stream));
    stage_pending = true;
  }
  static_assert(sizeof(DevStatus) <= kRbPcState && kRbPcState + sizeof(PcState) <= kRbChol &&
                    kRbChol + sizeof(CholState) <= kRbEig &&
                    kRbWeyl + sizeof(DevWeyl) <= kRbExpect && kRbExpect + sizeof(ExpectResult) <= kRbCommit &&
                    kRbCommit + sizeof(CommitResult) <= kRbSweep && kRbSweep + sizeof(SweepReport) <= kRbBytes,
                "read-back block layout");
  void await(const Ticket& slot, Ticket want) const { await_ticket(stream, slot, want); }
  void read_status(DevStatus& h) {  // through pinned memory: no staging copy
    GC_HIP(hipMemcpyAsync(rb + kRbStatus, st, sizeof(DevStatus), hipMemcpyDeviceToHost, stream));
    GC_HIP(hipStreamSynchronize(stream));
    std::memcpy(&h, rb + kRbStatus, sizeof(DevStatus));
  }

  int dim_l(int i) const { return chi[i]; }
  int dim_r(int i) const { return chi[i + 1]; }

  // ---------------------------------------------------------------- factorisation
  // Split M (p x q, row-major) into L (p x k) R (k x q).  mode 0: truncation rule with
  // renormalisation; mode 1: exact (rank floor only).  left_ortho: L has orthonormal columns
  // (else R has orthonormal rows).  Returns the status block of the final pass.
  // reduce: a truncating split of the bottom loop (mode 0 with a positive cutoff, outside
  // gradient recording and replay): the eigensolver runs on the r x r matrix of a pivoted
  // Cholesky factorisation of the Gram, which drops what the cutoff could never keep (rotated
  // two-site tensors often have rank far below m) and preconditions the Jacobi sweeps.
  DevStatus factorize(const z64* M, int p, int q, int mode, int left_ortho, z64* Lout, z64* Rout,
                      bool reduce = false, const std::function<void(int)>& ahead = {}) {
    const bool wide = p <= q;
    const int m = wide ? p : q, kW = wide ? q : p;
    GC_CHECK((size_t)m <= lay.mcap && (size_t)m * kW <= lay.slot_elems, GCAMPS_ECAPACITY,
             "factorisation exceeds workspace capacity");
    if (m <= kSmallEig && kW <= kSplitSmallMaxK) return split_small(M, p, q, mode, left_ortho, Lout, Rout, ahead);
    DevStatus mv{};
    if (mode == 1 && !tape && !rank_rec && !rank_frz && move_full_rank(M, p, q, left_ortho, Lout, Rout, mv)) return mv;
    const z64 one = {1.0, 0.0};
    GC_HIP(hipEventRecord(evf0, stream));
    auto gram = [&]() {
      if (wide)
        launch_zgemm(stream, 0, 1, m, m, q, M, q, M, q, G, m, one, 0, 1);
      else
        launch_zgemm(stream, 1, 0, m, m, p, M, q, M, q, G, m, one, 0, 1);
    };
    gram();
    // basis: nb columns of U (ld ldu); tail: weight outside the basis, always discarded
    int nb = m, ldu = m;
    int sw_h = 0, sw_main = 0, sw_p2 = 0;  // sweeps of the eigen-decompositions (trace only)
    const double* tail = nullptr;
    const bool try_reduce = reduce && mode == 0 && cfg.cutoff > 0.0 && m > kReduceMinM && m <= kReduceMaxM && !tape &&
                            !rank_rec && !rank_frz;
    bool reduced = false;
    if (try_reduce) {
      // stop once the Schur complement's trace is below min(1e-14, cutoff / 2m) of the trace: then
      // its directions hold less than the cutoff even all together, and no eigenvalue moves by
      // more than the Gram's own rounding
      const double tol_rel = std::min(1e-14, cfg.cutoff / (2.0 * m));
      PcState* hsp = reinterpret_cast<PcState*>(rb + kRbPcState);
      const int r = pchol_reduce(stream, G, m, m, Z, m, tol_rel, m, sig, perm, pcst, hsp);
      const PcState hs = *hsp;
      if (hs.done && r >= 1) {
        // H = L^H L = Y lam Y^H with relative accuracy, so that the columns of L Y are
        // orthogonal to ~1e-14 of their norms even where lam is tiny (an absolute criterion
        // leaves them off by ~tr H / lam times that)
        launch_zgemm(stream, 1, 0, r, r, m, Z, m, Z, m, Utmp, r, one, 0, 1);
        eig_hermitian(stream, Utmp, r, r, G, r, lam, 1, eig, st, &sw_h);
        launch_zgemm(stream, 0, 0, m, r, r, Z, m, G, r, U, r, one, 0, 0);     // L Y
        launch_normalize_cols(stream, U, m, r, r);
        orthonormalize_cols(stream, U, Z, Utmp, m, r, 2);
        nb = r;
        ldu = r;
        tail = &pcst->tres;
        reduced = true;
        stats_red[0] += 1;
        stats_red[1] += r;
        stats_red[2] += m;
      } else {
        gram();  // no useful reduction: the full eigen-decomposition of the (recomputed) Gram
        stats_red[3] += 1;
      }
    }
    if (!reduced) eig_hermitian(stream, G, m, m, U, m, lam, 0, eig, st, &sw_main);
    if (wide)
      launch_zgemm(stream, 1, 0, nb, q, m, U, ldu, M, q, B, q, one, 0, 0);
    else
      launch_zgemm(stream, 1, 1, nb, p, m, U, ldu, M, q, B, p, one, 0, 0);
    if (reduced) {
      // Rayleigh-Ritz on the reduced basis: B B^H = U^H G U with the full Gram, so its
      // eigenvalues err by the square of the basis error where L L^H's err by tr S
      launch_zgemm(stream, 0, 1, nb, nb, kW, B, kW, B, kW, G, nb, one, 0, 1);
      // nearly diagonal already: the pre-check usually finds nothing to rotate, and then the
      // eigenvectors are the identity and U and B stay as they are.  A direction dropped by the rank limit
      // is below chi_max others, one dropped by the cutoff holds at most the cutoff (and with a degenerate group
      // below the cut up to 1e-10 more of itself per member).
      const double discardable = std::max(1.0 / (cfg.chi_max + 1.0), cfg.cutoff) * (1.0 + 1e-6);
      eig_hermitian(stream, G, nb, nb, Z, nb, lam, 0, eig, st, &sw_main, discardable);
      if (sw_main != 0) {
        launch_zgemm(stream, 0, 0, m, nb, nb, U, ldu, Z, nb, Utmp, ldu, one, 0, 0);
        std::swap(U, Utmp);
        launch_zgemm(stream, 1, 0, nb, kW, nb, Z, nb, B, kW, B2, kW, one, 0, 0);
        std::swap(B, B2);
      }
    }
    int force_k, force_pass2;
    forced_decision(force_k, force_pass2);
    launch_rownorm2(stream, B, nb, kW, kW, sig2);
    launch_trunc(stream, sig2, nb, cfg.cutoff, cfg.chi_max, mode, force_k, perm, sig, st, tail);
    GC_HIP(hipEventRecord(evf1, stream));
    DevStatus h;
    read_status(h);
    GC_CHECK(nb > kSmallEig || h.converged, GCAMPS_ENUMERIC, "eigensolver did not converge");
    stats[5] += 8.0 * (double)m * m * kW * 2.0;
    const bool pass2 = force_pass2 >= 0 ? force_pass2 == 1 : h.need_pass2 != 0;
    if (pass2) {
      // accurate second pass on the nearly diagonal Gram of B (relative criterion)
      launch_zgemm(stream, 0, 1, nb, nb, kW, B, kW, B, kW, G, nb, one, 0, 1);
      eig_hermitian(stream, G, nb, nb, Z, nb, lam, 1, eig, st, &sw_p2);
      launch_zgemm(stream, 0, 0, m, nb, nb, U, ldu, Z, nb, Utmp, ldu, one, 0, 0);
      std::swap(U, Utmp);
      launch_zgemm(stream, 1, 0, nb, kW, nb, Z, nb, B, kW, B2, kW, one, 0, 0);
      std::swap(B, B2);
      launch_rownorm2(stream, B, nb, kW, kW, sig2);
      launch_trunc(stream, sig2, nb, cfg.cutoff, cfg.chi_max, mode, force_k, perm, sig, st, tail);
      GC_HIP(hipEventRecord(evf1, stream));
      read_status(h);
      GC_CHECK(nb > kSmallEig || h.converged, GCAMPS_ENUMERIC, "eigensolver did not converge (second pass)");
      stats[5] += 8.0 * (double)nb * nb * kW * 2.0;
    }
    GC_CHECK(std::isfinite(h.eps) && h.kept >= 1, GCAMPS_ENUMERIC, "factorisation produced non-finite values");
    {  // both events have completed: read_status synchronised the stream after evf1
      float fms = 0.0f;
      GC_HIP(hipEventElapsedTime(&fms, evf0, evf1));
      count_fact(p, q, fms);
      if (trace_fact)  // GCAMPS_TRACE_FACT: one line per factorisation on stderr
        std::fprintf(stderr, "gcamps-fact m=%d k=%d mode=%d reduce=%d basis=%d kept=%d pass2=%d ms=%.3f sweeps=%d/%d/%d\n",
                     m, kW, mode, reduced ? 1 : 0, nb, h.kept, pass2 ? 1 : 0, fms, sw_h, sw_main, sw_p2);
    }
    record_fact(h, pass2, mode, left_ortho, p, q);
    launch_emit(stream, wide ? 1 : 0, left_ortho, mode == 0 ? 1 : 0, p, q, h.kept, U, ldu, B, kW, perm, sig, Lout,
                Rout);
    last_basis = nb;
    return h;
  }

  // factorize() in mode 1 of a matrix of full rank: true when the pivots of the Gram's Cholesky
  // factorisation show full rank (see kernels_chol.hip).  A pivot of kMovePivot times the largest diagonal
  // entry leaves X K^-H orthonormal to about m 2^-53 / kMovePivot.  A Newton-Schulz step takes a defect of
  // norm e to 3/4 e^2 + 1/4 e^3, so two of them take kMoveGap, which a bound of the norm has to stay below, to 4.3e-17.
  // Gradient recordings and replays keep the eigenbasis their reverse sweep needs.
  bool move_full_rank(const z64* M, int p, int q, int left_ortho, z64* Lout, z64* Rout, DevStatus& h) {
    constexpr double kMovePivot = 1e-9, kMoveGap = 1e-4;
    const bool wide = p <= q;
    const int m = wide ? p : q, P = wide ? q : p;
    const bool trivial = wide == (left_ortho != 0);  // the orthonormal factor is the square one
    const z64 one = {1.0, 0.0};
    z64* A = reinterpret_cast<z64*>(ws + lay.off_B);  // B and B2 are adjacent: room for m + P rows
    if ((size_t)(m + P) * m > 2 * lay.slot_elems) return false;
    GC_HIP(hipEventRecord(evf0, stream));
    if (wide)
      launch_zgemm(stream, 0, 1, m, m, q, M, q, M, q, A, m, one, 0, 1);
    else
      launch_zgemm(stream, 1, 0, m, m, p, M, q, M, q, A, m, one, 0, 1);
    z64* X = A + (size_t)m * m;
    if (!trivial) {
      if (wide)
        launch_conj_transpose(stream, M, p, q, X);
      else
        launch_copy(stream, X, M, (size_t)P * m);
    }
    launch_cholesky(stream, A, m, trivial ? m : m + P, chst);
    if (trivial) {
      launch_fill_identity(stream, left_ortho ? Lout : Rout, m, m);
      launch_copy(stream, left_ortho ? Rout : Lout, M, (size_t)p * q);
    } else {
      z64* Xn = left_ortho ? Lout : Rout;  // P x m
      for (int it = 0; it < 2; ++it) {     // Newton-Schulz: X <- X (3 I - X^H X) / 2
        launch_zgemm(stream, 1, 0, m, m, P, X, m, X, m, G, m, one, 0, 1);
        if (it == 0) launch_identity_gap(stream, G, m, chst);
        launch_scaled_copy(stream, Xn, X, (size_t)P * m, 1.5);
        launch_zgemm(stream, 0, 0, P, m, m, X, m, G, m, Xn, m, z64{-0.5, 0.0}, 1, 0);
        std::swap(X, Xn);
      }
      if (left_ortho) {
        launch_copy(stream, Lout, X, (size_t)P * m);
        launch_zgemm(stream, 1, 0, m, q, p, X, m, M, q, Rout, q, one, 0, 0);
      } else {
        launch_zgemm(stream, 0, 0, p, m, q, M, q, X, m, Lout, m, one, 0, 0);
        launch_conj_transpose(stream, X, P, m, Rout);
      }
    }
    GC_HIP(hipEventRecord(evf1, stream));
    GC_HIP(hipMemcpyAsync(rb + kRbChol, chst, sizeof(CholState), hipMemcpyDeviceToHost, stream));
    GC_HIP(hipStreamSynchronize(stream));
    CholState cs;
    std::memcpy(&cs, rb + kRbChol, sizeof(CholState));
    if (!(cs.dmax > 0.0 && cs.dmin >= kMovePivot * cs.dmax && cs.emax <= kMoveGap)) return false;
    h = DevStatus{};
    h.kept = m;
    h.converged = 1;
    h.lam_max = cs.dmax;
    stats[5] += 8.0 * (double)m * m * P * 2.0;
    float fms = 0.0f;
    GC_HIP(hipEventElapsedTime(&fms, evf0, evf1));
    count_fact(p, q, fms);
    if (trace_fact)
      std::fprintf(stderr, "gcamps-fact m=%d k=%d mode=1 reduce=0 basis=%d kept=%d pass2=0 ms=%.3f sweeps=0/0/0\n", m, P, m,
                   m, fms);
    last_basis = m;
    return true;
  }

  // Recorded decision of the next factorisation in a frozen replay: kept rank in the low bits, bit 30 =
  // the accurate second pass ran.  force_k = 0 and force_pass2 = -1 outside replays.
  void forced_decision(int& force_k, int& force_pass2) {
    force_k = 0;
    force_pass2 = -1;
    if (!rank_frz) return;
    GC_CHECK(rank_pos < rank_frz->size(), GCAMPS_EINVAL, "frozen replay ran past the recorded ranks");
    const int32_t v = (*rank_frz)[rank_pos++];
    force_k = v & kRankMask;
    force_pass2 = (v >> kPass2Bit) & 1;
  }
  void count_fact(int p, int q, double ms) {
    const double pl = std::max(p, q), ql = std::min(p, q);
    kstats[0] += 1;
    kstats[1] += 4.0 * (6.0 * pl * ql * ql + 20.0 * ql * ql * ql);
    kstats[2] += ms;
  }
  // The decision into the rank log and the factorisation's basis (U, B, sig, perm) onto the tape.
  void record_fact(const DevStatus& h, bool pass2, int mode, int left_ortho, int p, int q) {
    if (rank_rec) rank_rec->push_back(h.kept | (pass2 ? (1 << kPass2Bit) : 0));
    if (!tape) return;
    const int m = std::min(p, q), kW = std::max(p, q);
    FactRec& f = last_fact;
    f.m = m;
    f.kW = kW;
    f.k = h.kept;
    f.p = p;
    f.q = q;
    f.wide = p <= q ? 1 : 0;
    f.left = left_ortho;
    f.renorm = mode == 0 ? 1 : 0;
    f.U = arena->take<z64>((size_t)m * m);
    f.B = arena->take<z64>((size_t)m * kW);
    f.sig = arena->take<double>(m);
    launch_record(stream, U, B, sig, perm, m, kW, f.U, f.B, f.sig);
  }
  // factorize() of a matrix whose smaller side fits one workgroup: one launch, which also leaves
  // the status in the pinned read-back block.  ahead: launches what follows for an assumed rank.
  DevStatus split_small(const z64* M, int p, int q, int mode, int left_ortho, z64* Lout, z64* Rout,
                        const std::function<void(int)>& ahead) {
    const int m = std::min(p, q), kW = std::max(p, q);
    int force_k, force_pass2;
    forced_decision(force_k, force_pass2);
    SplitArgs a{M, p, q, left_ortho, mode == 0 ? 1 : 0, force_pass2, {cfg.cutoff, cfg.chi_max, mode, force_k},
                U, B, Lout, Rout, sig, perm, st, reinterpret_cast<DevStatus*>(rb_dev + kRbStatus), ++ticket};
    launch_split_small(stream, a);
    if (ahead) ahead(force_k > 0 ? std::min(force_k, m) : m);
    await(reinterpret_cast<DevStatus*>(rb + kRbStatus)->ticket, a.ticket);
    DevStatus h;
    std::memcpy(&h, rb + kRbStatus, sizeof(DevStatus));
    GC_CHECK(h.converged, GCAMPS_ENUMERIC, "eigensolver did not converge");
    GC_CHECK(std::isfinite(h.eps) && h.kept >= 1, GCAMPS_ENUMERIC, "factorisation produced non-finite values");
    stats[5] += 8.0 * (double)m * m * kW * 2.0 * (h.pass2 ? 2 : 1);
    count_fact(p, q, h.ticks * tick_ms);
    if (trace_fact)
      std::fprintf(stderr, "gcamps-fact m=%d k=%d mode=%d reduce=0 basis=%d kept=%d pass2=%d ms=%.3f sweeps=0/%d/0\n", m, kW,
                   mode, m, h.kept, h.pass2, h.ticks * tick_ms, h.sweeps);
    record_fact(h, h.pass2 != 0, mode, left_ortho, p, q);
    last_basis = m;
    return h;
  }

  // Kept rank of the split's truncation rule on M (p x q): the first pass and, where the rank
  // floor matters, the relative-accuracy second pass of factorize(), without the factors, the
  // counters or any record (the bond-dimension criterion on bonds above the batched kernel's
  // size).
  int split_rank(const z64* M, int p, int q) {
    const bool wide = p <= q;
    const int m = wide ? p : q, kW = wide ? q : p;
    GC_CHECK((size_t)m <= lay.mcap && (size_t)m * kW <= lay.slot_elems, GCAMPS_ECAPACITY,
             "factorisation exceeds workspace capacity");
    const z64 one = {1.0, 0.0};
    if (wide)
      launch_zgemm(stream, 0, 1, m, m, q, M, q, M, q, G, m, one, 0, 1);
    else
      launch_zgemm(stream, 1, 0, m, m, p, M, q, M, q, G, m, one, 0, 1);
    eig_hermitian(stream, G, m, m, U, m, lam, 0, eig, st, nullptr);
    if (wide)
      launch_zgemm(stream, 1, 0, m, q, m, U, m, M, q, B, q, one, 0, 0);
    else
      launch_zgemm(stream, 1, 1, m, p, m, U, m, M, q, B, p, one, 0, 0);
    launch_rownorm2(stream, B, m, kW, kW, sig2);
    launch_trunc(stream, sig2, m, cfg.cutoff, cfg.chi_max, 0, 0, perm, sig, st);
    DevStatus h;
    read_status(h);
    GC_CHECK(m > kSmallEig || h.converged, GCAMPS_ENUMERIC, "eigensolver did not converge");
    if (h.need_pass2) {
      launch_zgemm(stream, 0, 1, m, m, kW, B, kW, B, kW, G, m, one, 0, 1);
      eig_hermitian(stream, G, m, m, Z, m, lam, 1, eig, st, nullptr);
      launch_zgemm(stream, 1, 0, m, kW, m, Z, m, B, kW, B2, kW, one, 0, 0);
      launch_rownorm2(stream, B2, m, kW, kW, sig2);
      launch_trunc(stream, sig2, m, cfg.cutoff, cfg.chi_max, 0, 0, perm, sig, st);
      read_status(h);
      GC_CHECK(m > kSmallEig || h.converged, GCAMPS_ENUMERIC, "eigensolver did not converge (second pass)");
    }
    GC_CHECK(std::isfinite(h.eps) && h.kept >= 1, GCAMPS_ENUMERIC, "factorisation produced non-finite values");
    return h.kept;
  }

  // ---------------------------------------------------------------- centre moves (exact)
  // copy of a site tensor into the tape arena (reverse sweep input)
  z64* keep_copy(const z64* src, size_t count) {
    z64* dst = arena->take<z64>(count);
    launch_copy(stream, dst, src, count);
    return dst;
  }
  void tape_absorb(int kind, int i, const z64* nb, int rows, int cols) {
    TapeOp op;
    op.kind = kind;
    op.site = i;
    op.f = last_fact;
    op.x0 = keep_copy(nb, (size_t)rows * cols);
    op.d0[0] = rows;
    op.d0[1] = cols;
    tape->push_back(op);
  }

  // A small split leaves its rank to the host, but an exact move nearly always keeps min(p, q): the product with the
  // neighbour is launched behind the split for that rank (or the recorded one) before the host knows, and
  // again only if the split kept another.  The queue then does not wait 6 us for the host.
  void move_right(int i) {  // centre i -> i+1
    const int p = chi[i] * d, q = chi[i + 1], ncols = d * chi[i + 2];
    int made = 0;
    auto absorb = [&](int k) {
      launch_zgemm(stream, 0, 0, k, ncols, q, Rbuf, q, site[i + 1], ncols, spare, ncols, z64{1.0, 0.0}, 0, 0);
      made = k;
    };
    DevStatus h = factorize(site[i], p, q, 1, 1, Lbuf, Rbuf, false, absorb);
    const int k = h.kept;
    if (tape) tape_absorb(TAPE_ABSORB_R, i, site[i + 1], q, ncols);
    if (made != k) absorb(k);
    std::swap(site[i], Lbuf);
    std::swap(site[i + 1], spare);
    chi[i + 1] = k;
    centre = i + 1;
  }
  void move_left(int i) {  // centre i -> i-1
    const int p = chi[i], q = d * chi[i + 1], nrows = chi[i - 1] * d;
    int made = 0;
    auto absorb = [&](int k) {
      launch_zgemm(stream, 0, 0, nrows, k, p, site[i - 1], p, Lbuf, k, spare, k, z64{1.0, 0.0}, 0, 0);
      made = k;
    };
    DevStatus h = factorize(site[i], p, q, 1, 0, Lbuf, Rbuf, false, absorb);
    const int k = h.kept;
    if (tape) tape_absorb(TAPE_ABSORB_L, i, site[i - 1], nrows, p);
    if (made != k) absorb(k);
    std::swap(site[i], Rbuf);
    std::swap(site[i - 1], spare);
    chi[i] = k;
    centre = i - 1;
  }
  void move_centre(int target) {
    while (centre < target) move_right(centre);
    while (centre > target) move_left(centre);
  }

  // ---------------------------------------------------------------- bottom loop
  // P = C^dagger W C for a Weyl target W = tau^p X^x Z^z (x, z, p given as 2n+1 ints).
  GateRec extract_string(const int* xzp) {
    WeylTarget W;
    for (int i = 0; i < n; ++i) {
      W.x[i] = (uint8_t)(((xzp[i] % d) + d) % d);
      W.z[i] = (uint8_t)(((xzp[n + i] % d) + d) % d);
    }
    W.p = xzp[2 * n];
    ++ticket;
    launch_weyl_extract(stream, n, d, tx, tz, tp, W, reinterpret_cast<DevWeyl*>(rb_dev + kRbWeyl), ticket);
    await(reinterpret_cast<DevWeyl*>(rb + kRbWeyl)->ticket, ticket);
    DevWeyl P;
    std::memcpy(&P, rb + kRbWeyl, sizeof(DevWeyl));
    GC_CHECK(P.bad == 0, GCAMPS_ENUMERIC, "tableau decomposition failed");
    GateRec g;
    g.l = P.l;
    g.r = P.r;
    g.p = P.p;
    g.x.assign(P.x, P.x + n);
    g.z.assign(P.z, P.z + n);
    int sd = 0;
    for (int i = 0; i < n; ++i) sd += P.x[i] * P.z[i];
    g.sd = sd % d;
    return g;
  }

  // MPO coefficients K_b = c_b tau^{ph_b} of sum_b c_b P^b for diag(e^{i phi_j}) = sum_b c_b Z^b,
  // c_b = (1/d) sum_j e^{i phi_j} omega^{-bj}; P^b = tau^{ph_b} X^{bx} Z^{bz} per site with
  // ph_b = b p + 2 <x, z> b(b-1)/2 (mod 2d).
  MpoCoeff mpo_coeff(const GateRec& P, const double* phi) const {
    MpoCoeff co;
    for (int b = 0; b < d; ++b) {
      std::complex<double> cb = 0.0;
      for (int j = 0; j < d; ++j) cb += std::polar(1.0, phi[j] - 2.0 * M_PI * b * j / d);
      cb /= (double)d;
      const int ph = (b * P.p + 2 * P.sd * (b * (b - 1) / 2)) % (2 * d);
      std::complex<double> kb = cb * std::polar(1.0, M_PI * ph / d);
      co.k[b] = z64{kb.real(), kb.imag()};
      co.w[b] = z64{std::cos(2.0 * M_PI * b / d), std::sin(2.0 * M_PI * b / d)};
    }
    return co;
  }

  void phase_rotation(int s, const double* phi) {
    std::vector<int> xzp(2 * n + 1, 0);
    xzp[n + s] = 1;  // target Z_s
    GateRec P = extract_string(xzp.data());
    GC_CHECK(P.l >= 0, GCAMPS_ENUMERIC, "tableau decomposition failed");
    if (gate_rec) gate_rec->push_back(P);
    phase_apply(P, phi);
  }

  // Timing of one gate's MPO launches: events recorded around them and read once they have
  // completed (the compression that follows synchronises the stream).
  void settle_mpo() {
    if (!mpo_pending) return;
    GC_HIP(hipEventSynchronize(evm1));
    float ms = 0.0f;
    GC_HIP(hipEventElapsedTime(&ms, evm0, evm1));
    kstats[5] += ms;
    mpo_pending = false;
  }
  void mpo_begin() {
    settle_mpo();
    GC_HIP(hipEventRecord(evm0, stream));
  }
  void mpo_end() {
    GC_HIP(hipEventRecord(evm1, stream));
    mpo_pending = true;
  }
  // Algorithmic bytes of one MPO site launch of bond J on [l, r]: the site tensor read once and
  // its product (bonds multiplied by J inside the support) written once, complex128.
  void mpo_count(int i, int l, int r, int J) {
    const double in = (double)chi[i] * d * chi[i + 1];
    const double out = (double)chi[i] * (i > l ? J : 1) * d * chi[i + 1] * (i < r ? J : 1);
    kstats[3] += 1;
    kstats[4] += 16.0 * (in + out);
  }

  // Apply sum_b c_b P^b (P from the tableau) to the MPS and compress.
  void phase_apply(const GateRec& P, const double* phi) {
    const int l = P.l, r = P.r;
    const MpoCoeff co = mpo_coeff(P, phi);
    move_centre(l);
    mpo_begin();
    for (int i = l; i <= r; ++i) {
      int kind = (l == r) ? 3 : (i == l ? 0 : (i == r ? 2 : 1));
      mpo_count(i, l, r, d);
      if (tape) {
        TapeOp op;
        op.kind = TAPE_MPO;
        op.site = i;
        op.mpo_kind = kind;
        op.dx = P.x[i];
        op.dz = P.z[i];
        op.chil = chi[i];
        op.chir = chi[i + 1];
        if (kind == 0 || kind == 3) {
          op.x0 = keep_copy(site[i], (size_t)chi[i] * d * chi[i + 1]);
          op.d0[0] = chi[i] * d;
          op.d0[1] = chi[i + 1];
        }
        tape->push_back(op);
      }
      launch_mpo_site(stream, kind, d, chi[i], chi[i + 1], P.x[i], P.z[i], co, site[i], spare);
      std::swap(site[i], spare);
    }
    mpo_end();
    for (int j = l + 1; j <= r; ++j) chi[j] *= d;
    compress(l, r);
    gates += 1;
    stats[0] += 1;
  }

  // After an MPO on [l, r] (centre at l): exact moves to r, then truncating splits back to l
  // (§2.4); F_est absorbs the discarded weights.
  void compress(int l, int r) {
    if (r > l) {
      for (int i = l; i < r; ++i) move_right(i);
      for (int i = r; i > l; --i) {
        const int p = chi[i], q = d * chi[i + 1];
        DevStatus h = factorize(site[i], p, q, 0, 0, Lbuf, Rbuf, true);
        const int k = h.kept;
        if (tape) tape_absorb(TAPE_ABSORB_L, i, site[i - 1], chi[i - 1] * d, p);
        std::swap(site[i], Rbuf);
        const int nrows = chi[i - 1] * d;
        launch_zgemm(stream, 0, 0, nrows, k, p, site[i - 1], p, Lbuf, k, spare, k, z64{1.0, 0.0}, 0, 0);
        std::swap(site[i - 1], spare);
        chi[i] = k;
        centre = i - 1;
        f_est *= (1.0 - h.eps);
        stats[3] += h.flagged;
      }
    }
  }

  // General gate U on sites s..s+k-1 (k = 1, 2): Weyl expansion, each term commuted through the
  // Clifford, the sum applied as an MPO of bond J = number of terms, then compressed.
  void general_gate(int s, int k, const std::vector<z64>& U) {
    GC_CHECK(tape == nullptr && rank_rec == nullptr && rank_frz == nullptr, GCAMPS_EUNSUPPORTED,
             "general gates are not recorded for gradients");
    int D = 1;
    for (int t = 0; t < k; ++t) D *= d;
    // c_xz = Tr(W_xz^dagger U) / D with W_xz |v> = omega^{z . v} |v + x> (digits of site s first)
    struct Term {
      std::vector<int> x, z;
      std::complex<double> c;
    };
    std::vector<Term> terms;
    double cmax = 0.0;
    const int nx = D;  // exponent vectors x (and z) enumerate like basis states
    auto digits = [&](int v, std::vector<int>& out) {
      out.assign(k, 0);
      for (int t = k - 1; t >= 0; --t) {
        out[t] = v % d;
        v /= d;
      }
    };
    std::vector<int> xv, zv, sv, tv;
    for (int xi = 0; xi < nx; ++xi)
      for (int zi = 0; zi < nx; ++zi) {
        digits(xi, xv);
        digits(zi, zv);
        std::complex<double> acc = 0.0;
        for (int v = 0; v < D; ++v) {
          digits(v, sv);
          int row = 0, dot = 0;
          for (int t = 0; t < k; ++t) {
            row = row * d + (sv[t] + xv[t]) % d;
            dot += zv[t] * sv[t];
          }
          const z64 uv = U[(size_t)row * D + v];  // <v + x| U |v>
          acc += std::polar(1.0, -2.0 * M_PI * (double)(dot % d) / d) * std::complex<double>(uv.re, uv.im);
        }
        acc /= (double)D;
        cmax = std::max(cmax, std::abs(acc));
        terms.push_back({xv, zv, acc});
      }
    std::vector<Term> kept;
    for (auto& t : terms)
      if (std::abs(t.c) > 1e-14 * cmax) kept.push_back(t);
    const int J = (int)kept.size();
    GC_CHECK(J <= std::max(d, cfg.max_gate_terms), GCAMPS_ECAPACITY,
             "gate has " + std::to_string(J) + " Weyl terms; raise max_gate_terms");
    // commute every term through C: P_j = C^dagger W_j C
    std::vector<GateRec> P(J);
    int l = n, r = -1;
    for (int j = 0; j < J; ++j) {
      bool ident = true;
      for (int t = 0; t < k; ++t) ident = ident && kept[j].x[t] == 0 && kept[j].z[t] == 0;
      if (ident) {  // C^dagger I C = I: no support, no phase
        P[j].x.assign(n, 0);
        P[j].z.assign(n, 0);
        P[j].p = 0;
        continue;
      }
      std::vector<int> xzp(2 * n + 1, 0);
      for (int t = 0; t < k; ++t) {
        xzp[s + t] = kept[j].x[t];
        xzp[n + s + t] = kept[j].z[t];
      }
      P[j] = extract_string(xzp.data());
      GC_CHECK(P[j].l >= 0, GCAMPS_ENUMERIC, "tableau decomposition failed");
      l = std::min(l, P[j].l);
      r = std::max(r, P[j].r);
    }
    if (r < l) l = r = s;  // U proportional to the identity
    MpoTerms tm;
    for (int j = 0; j < J; ++j) {
      const std::complex<double> cj = kept[j].c * std::polar(1.0, M_PI * P[j].p / d);
      tm.coef[j] = z64{cj.real(), cj.imag()};
    }
    move_centre(l);
    mpo_begin();
    for (int i = l; i <= r; ++i) {
      const int kind = (l == r) ? 3 : (i == l ? 0 : (i == r ? 2 : 1));
      for (int j = 0; j < J; ++j) {
        tm.x[j] = P[j].x[i];
        tm.z[j] = P[j].z[i];
      }
      mpo_count(i, l, r, J);
      launch_mpo_sum_site(stream, kind, d, J, chi[i], chi[i + 1], tm, site[i], spare);
      std::swap(site[i], spare);
    }
    mpo_end();
    for (int j = l + 1; j <= r; ++j) chi[j] *= J;
    compress(l, r);
    gates += 1;
    stats[0] += 1;
  }

  // ---------------------------------------------------------------- scoring
  // Whether a score of this mode goes through the density matrix: in FP64 always, in the low-precision modes (then
  // in FP32) where it is the faster form.  It pays its Gram product of Theta once, the rotated matrices pay theirs
  // per candidate.  Qutrits, FP32: always in a sweep, whose FP64 re-score reuses the Gram; for a score alone (score_bond)
  // of at most 8 candidates (one column group of the rotated form) the rotated matrices from m^2 k = 3e8 on: chi =
  // 192 takes 162 us through the matrix and 167 rotated, 243 254 and 215, 495 1343 and 1076; 9 candidates at 243 257 and
  // 361.  Qutrits, BF16: 64 candidates at chi = 81 take 78 against 74 us, 128 89
  // against 132, at chi = 243 16 take 291 against 213 and 128 426 against 990.  Qubits: density is the faster form for
  // 129 candidates at every size (chi = 64 40 us against 101 in FP32 and 72 in BF16, 512 593 against 4160 and 1947), and
  // would be for fewer; sets of up to 128 keep the rotated matrices because their launch parameters are tuned and saved by
  // shape (GCAMPS_TUNE_FILE) and sets of that size have saved ones.
  bool density_mode(int prec) const {
    if (prec == GCAMPS_SCORE_FP64) return true;
    if (prec == GCAMPS_SCORE_REPLICA || !dtab32) return false;
    return d == 2 ? ncand > 128 : prec == GCAMPS_SCORE_FP32 || ncand > 64;
  }
  // alone: no re-score of the same bond follows
  bool use_density(int prec, int cl, int cr, bool alone = false) const {
    const double work = (double)std::min(cl, cr) * std::min(cl, cr) * std::max(cl, cr) * d * d * d;
    const bool few = alone && prec == GCAMPS_SCORE_FP32 && ncand <= kDensityFew && work >= kDensityFewWork;
    return dtab && density_mode(prec) && work >= kDensityMinWork && !few && density_fits(d, cl, cr, ncand, lay.nbuf_bytes);
  }
  double density_flops(int cl, int cr) const {  // one candidate's product
    const double X = std::min(cl, cr);
    return 4.0 * X * (X + 1) * std::pow((double)d, 6);
  }
  // Scores of Theta (bonds cl, cr) in the arithmetic of prec: the full set, or (nlimit given) the window
  // list of an earlier pass.  f_ready: the scratch holds Theta's density matrix; it does after a pass
  // that used it.  evs, evcap and used as in launch_score; alone as in use_density.
  void score(int prec, int cl, int cr, const int* list, const int* nlimit, double* out, bool& f_ready,
             hipEvent_t* evs = nullptr, int evcap = 0, int* used = nullptr, int64_t* tick = nullptr, bool alone = false) {
    if (used) *used = 0;
    if (use_density(prec, cl, cr, alone)) {
      if (!f_ready) launch_density_gram(stream, d, cl, cr, theta, nbuf);
      f_ready = true;
      const bool ev = used && evcap >= 2;
      launch_density_score(stream, d, prec != GCAMPS_SCORE_FP64, cl, cr, dtab, dtab32, ncand, list, ncand, nlimit, out,
                           nbuf, lay.nbuf_bytes, ev ? evs[0] : nullptr, ev ? evs[1] : nullptr);
      if (ev) *used = 1;
      return;
    }
    f_ready = false;
    launch_score(stream, prec, d, cl, cr, theta, q64, q32, list, ncand, nlimit, out, partial, lay.ncand * lay.ntp * 2,
                 nbuf, lay.nbuf_bytes, evs, evcap, used, rtab, tick);
  }

  // Full-set scores of bond (i, i+1) in the configured mode, to host memory; commits nothing.
  void score_bond(int i, double* out) {
    move_centre(i);
    const int cl = chi[i], cm = chi[i + 1], cr = chi[i + 2];
    launch_zgemm(stream, 0, 0, cl * d, d * cr, cm, site[i], cm, site[i + 1], d * cr, theta, d * cr, z64{1.0, 0.0},
                 0, 0);
    bool f_ready = false;
    score(cfg.score_prec, cl, cr, nullptr, nullptr, s2, f_ready, nullptr, 0, nullptr, nullptr, true);
    GC_HIP(hipMemcpyAsync(out, s2, (size_t)ncand * sizeof(double), hipMemcpyDeviceToHost, stream));
    GC_HIP(hipStreamSynchronize(stream));
  }

  void disentangle(int* out_sweeps, int* out_changed) {
    GC_CHECK(ncand >= 1, GCAMPS_EINVAL, "no candidate set attached");
    int sweeps = 0, changed_total = 0;
    const int prec = cfg.score_prec;
    const bool frozen = choice_frz != nullptr;
    for (int sw = 0; sw < cfg.max_sweeps; ++sw) {
      ++sweeps;
      const bool ltr = (sw % 2 == 0);
      int changed = 0;
      for (int t = 0; t < n - 1; ++t) {
        const int i = ltr ? t : n - 2 - t;
        move_centre(ltr ? i : i + 1);
        const int cl = chi[i], cm = chi[i + 1], cr = chi[i + 2];
        const int mm = std::min(cl * d, d * cr), kk = std::max(cl * d, d * cr);
        int gram_used = 0;
        bool shortcut = false;
        // the fused scoring launches are timed by the launches themselves (an event costs 3 us of a 100 us bond)
        const bool batched_rank = mm <= kRankMaxM && (size_t)(mm + (mm & 1)) * kk <= kRankMaxElems;
        const bool ticks = mm <= kScoreSmallM && !use_density(prec, cl, cr) && !use_density(GCAMPS_SCORE_FP64, cl, cr) &&
                           (cfg.criterion != GCAMPS_CRITERION_BOND_DIM || (batched_rank && prec == GCAMPS_SCORE_FP64));
        auto tick = [&](int k) { return ticks ? st->score_tick + k : nullptr; };
        CommitRule rule{-1, ncand, s2, nullptr, nullptr, cfg.tie_tol, nullptr, st,
                        reinterpret_cast<CommitResult*>(rb_dev + kRbCommit), ++ticket};
        if (frozen) {
          // replay: the recorded choice replaces scoring and selection
          GC_CHECK(choice_pos < choice_frz->size(), GCAMPS_EINVAL, "frozen replay ran past the recorded choices");
          const int c = (*choice_frz)[choice_pos++];
          GC_CHECK(c >= 0 && c < ncand, GCAMPS_EINVAL, "recorded choice outside the candidate set");
          rule.fixed = c;
          shortcut = (c == 0 && mm > kSmallEig);
          if (!shortcut) {
            launch_zgemm(stream, 0, 0, cl * d, d * cr, cm, site[i], cm, site[i + 1], d * cr, theta, d * cr,
                         z64{1.0, 0.0}, 0, 0);
            if (c != 0) launch_commit(stream, d, rule, cl, cr, q64, theta, CommitTableau{});
          }
        } else {
          launch_zgemm(stream, 0, 0, cl * d, d * cr, cm, site[i], cm, site[i + 1], d * cr, theta, d * cr,
                       z64{1.0, 0.0}, 0, 0);
          const bool density = use_density(prec, cl, cr);
          const double pflops = density ? density_flops(cl, cr)
                                        : 4.0 * mm * mm * kk + 8.0 * std::pow((double)d, 4) * cl * cr;
          if (!ticks) GC_HIP(hipEventRecord(ev0, stream));
          bool f_ready = false;
          score(prec, cl, cr, nullptr, nullptr, s2, f_ready, gram_ev.data(), (int)gram_ev.size(), &gram_used, tick(0));
          if (!ticks) GC_HIP(hipEventRecord(ev1, stream));
          if (cfg.criterion == GCAMPS_CRITERION_BOND_DIM) {
            if (batched_rank) {
              launch_cand_rank(stream, d, cl, cr, theta, q64, ncand, cfg.cutoff, cfg.chi_max, wlist, st->score_tick + 1);
            } else {
              // larger bonds: every candidate's rotated tensor through the split's own
              // factorisation (Lbuf holds Q_c Theta; the split of the bond comes later)
              std::vector<int32_t> ranks(ncand);
              for (int c = 0; c < ncand; ++c) {
                launch_rotate_copy(stream, d, cl, cr, c, q64, theta, Lbuf);
                ranks[c] = split_rank(Lbuf, cl * d, d * cr);
              }
              int32_t* hr = reinterpret_cast<int32_t*>(stage_begin());
              std::memcpy(hr, ranks.data(), (size_t)ncand * sizeof(int32_t));
              stage_upload(wlist, (size_t)ncand * sizeof(int32_t));
            }
            rule.rank = wlist;
          } else if (prec != GCAMPS_SCORE_FP64) {
            launch_window(stream, ncand, s2, cfg.near_tie, wlist, st, tick(1));
            if (!ticks) GC_HIP(hipEventRecord(ev2, stream));
            score(GCAMPS_SCORE_FP64, cl, cr, wlist, &st->nwindow, s2w, f_ready, nullptr, 0, nullptr, tick(2));
            if (!ticks) GC_HIP(hipEventRecord(ev3, stream));
            rule.list = wlist;
            rule.s2 = s2w;
          }
          if (prec == GCAMPS_SCORE_REPLICA && mm > kScoreSmallM) {
            // Gram of Theta over the larger bond (Hermitian half), pair sum, one d^8 dot per candidate
            const double X = std::min(cl, cr), Y = std::max(cl, cr), XD = X * d * d, R2 = std::pow((double)d, 8);
            stats[4] += 4.0 * XD * XD * Y + 8.0 * X * (X + 1) / 2 * R2 + 2.0 * ncand * R2;
          } else {
            stats[4] += (double)ncand * pflops;
            if (density) stats[4] += 4.0 * std::pow((double)std::min(cl, cr) * d * d, 2) * std::max(cl, cr);
          }
          stats[10] += 1;
          rule.tick = tick(rule.list ? 3 : 1);
          if (rule.rank) rule.tick = nullptr;
          launch_commit(stream, d, rule, cl, cr, q64, theta, CommitTableau{n, i, qinv, tx, tz, tp});
          // When the identity is kept, Theta = A_i A_{i+1} with the neighbour of the centre
          // orthonormal (right-orthonormal A_{i+1} when sweeping left to right, left-orthonormal
          // A_i otherwise), so Theta's Schmidt values are those of the centre tensor alone and the
          // split only needs the factorisation of that (smaller) tensor.
          if (mm > kSmallEig) {
            CommitResult* made = reinterpret_cast<CommitResult*>(rb + kRbCommit);
            await(made->ticket, rule.ticket);
            shortcut = made->cstar == 0;
          }
        }
        DevStatus h;
        if (shortcut && ltr) {
          h = factorize(site[i], cl * d, cm, 0, 1, Lbuf, Rbuf, true);
          const int k = h.kept;
          if (tape) tape_absorb(TAPE_ABSORB_R, i, site[i + 1], cm, d * cr);
          launch_zgemm(stream, 0, 0, k, d * cr, cm, Rbuf, cm, site[i + 1], d * cr, spare, d * cr, z64{1.0, 0.0}, 0, 0);
          std::swap(site[i], Lbuf);
          std::swap(site[i + 1], spare);
        } else if (shortcut) {
          h = factorize(site[i + 1], cm, d * cr, 0, 0, Lbuf, Rbuf, true);
          const int k = h.kept;
          if (tape) tape_absorb(TAPE_ABSORB_L, i + 1, site[i], cl * d, cm);
          launch_zgemm(stream, 0, 0, cl * d, k, cm, site[i], cm, Lbuf, k, spare, k, z64{1.0, 0.0}, 0, 0);
          std::swap(site[i + 1], Rbuf);
          std::swap(site[i], spare);
        } else {
          TapeOp op;
          if (tape) {
            op.kind = TAPE_THETA;
            op.site = i;
            op.x0 = keep_copy(site[i], (size_t)cl * d * cm);
            op.d0[0] = cl * d;
            op.d0[1] = cm;
            op.x1 = keep_copy(site[i + 1], (size_t)cm * d * cr);
            op.d1[0] = cm;
            op.d1[1] = d * cr;
            op.chil = cl;
            op.chir = cr;
          }
          h = factorize(theta, cl * d, d * cr, 0, ltr ? 1 : 0, Lbuf, Rbuf, true);
          if (tape) {
            op.f = last_fact;
            op.cstar = frozen ? rule.fixed : h.cstar;
            tape->push_back(op);
          }
          std::swap(site[i], Lbuf);
          std::swap(site[i + 1], Rbuf);
        }
        if (frozen) h.cstar = rule.fixed;
        stats[14] += shortcut ? 1 : 0;
        if (!frozen) {
          float ms = 0.f;
          if (!ticks) {
            GC_HIP(hipEventSynchronize(prec != GCAMPS_SCORE_FP64 && !rule.rank ? ev3 : ev1));
            GC_HIP(hipEventElapsedTime(&ms, ev0, ev1));
          } else {
            ms = (float)((h.score_tick[1] - h.score_tick[0]) * tick_ms);
          }
          stats[6] += ms;
          if (gram_used > 0) {  // Gram-purity kernel alone: algorithmic 4 m^2 k flop per candidate
            for (int e = 0; e < gram_used; ++e) {
              float gm = 0.f;
              GC_HIP(hipEventElapsedTime(&gm, gram_ev[2 * e], gram_ev[2 * e + 1]));
              stats[12] += gm;
            }
            stats[11] += gram_used;
            if (use_density(prec, cl, cr)) {
              const double xd = (double)std::min(cl, cr) * d * d;
              stats[13] += (double)ncand * density_flops(cl, cr);
              stats[15] += 8.0 * xd * xd + (double)ncand * std::pow((double)d, 6) * (prec == GCAMPS_SCORE_FP64 ? 16.0 : 8.0);
            } else {
              stats[13] += (double)ncand * 4.0 * mm * mm * kk;
              stats[15] += (double)ncand * mm * kk * (prec == GCAMPS_SCORE_FP64 ? 16.0 : 8.0);
            }
          }
          stats[1] += 1;
          if (prec != GCAMPS_SCORE_FP64) {
            const double pflops = use_density(GCAMPS_SCORE_FP64, cl, cr)
                                      ? density_flops(cl, cr)
                                      : 4.0 * mm * mm * kk + 8.0 * std::pow((double)d, 4) * cl * cr;
            stats[2] += h.nwindow;
            stats[8] += (double)h.nwindow * pflops;
            if (!ticks)
              GC_HIP(hipEventElapsedTime(&ms, ev2, ev3));
            else
              ms = (float)((h.score_tick[3] - h.score_tick[2]) * tick_ms);
            stats[9] += ms;
          }
        }
        chi[i + 1] = h.kept;
        centre = ltr ? i + 1 : i;
        f_est *= (1.0 - h.eps);
        stats[3] += h.flagged;
        choice_log.push_back((int32_t)(gates - 1));
        choice_log.push_back(sw);
        choice_log.push_back(i);
        choice_log.push_back(h.cstar);
        if (h.cstar != 0) ++changed;
      }
      changed_total += changed;
      if (changed == 0) break;
    }
    if (out_sweeps) *out_sweeps = sweeps;
    if (out_changed) *out_changed = changed_total;
  }

  // ---------------------------------------------------------------- state save / restore
  // |0...0>: every site tensor (1, d, 1) = e_0, centre 0, fidelity estimate 1.
  void reset_mps() {
    chi.assign(n + 1, 1);
    centre = 0;
    f_est = 1.0;
    for (int i = 0; i < n; ++i) {
      GC_HIP(hipMemsetAsync(site[i], 0, d * sizeof(z64), stream));
      z64* one = reinterpret_cast<z64*>(stage_begin());
      *one = z64{1.0, 0.0};
      stage_upload(site[i], sizeof(z64));
    }
  }
  size_t mps_elems() const {
    size_t t = 0;
    for (int i = 0; i < n; ++i) t += (size_t)chi[i] * d * chi[i + 1];
    return t;
  }

};
