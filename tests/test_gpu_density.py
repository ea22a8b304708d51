"""Scoring through the two-site density matrix against the oracle's S2, bond by bond, in FP64 (d = 2, 3) and
FP32 (d = 3): every bond of a chain, so that both cuts, one pair of a 32-pair tile more or less, bonds
below and above the size where the form starts, and candidate counts whose rows fill a 128-row block,
miss it by a few or exceed it, all occur; and the FP64 re-score of a window list behind an FP32 pass.

Tolerance: an entry of rho sums Y + d^4 products (Y the larger bond), so it errs by at most (Y + d^4) u
times the two rows' norms, u = 2^-53 (FP64) or 2^-24 (FP32); the purity and the squared trace by twice
that relative to their size times the d^2 of the unitary's row sums, and S2 = -ln by the sum.
"""
import numpy as np
import pytest

from oracle.clifford import word_matrix
from oracle.gcamps import renyi2
from paper_2511_06672_amd.workload import brickwork_circuit, candidate_words

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def g():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_2511_06672_amd import gcamps
    gcamps.lib()
    return gcamps


def saturated(g, d, n, chi, prec, ncand):
    c = brickwork_circuit(d, n, n + 8, n + 8, seed=900 + d + chi)
    st = g.State(g.make_config(d, n, chi, 0.0, score_prec=prec, auto_disentangle=False, max_candidates=ncand))
    g.run_circuit(st, c)
    cands = candidate_words(d, ncand, 910 + d)
    st.set_candset(g.CandSet(d, cands))
    return st, [word_matrix(d, w.gens, w.weyl) for w in cands]


@pytest.mark.parametrize("prec_name,d,n,chi,ncand", [("fp64", 3, 7, 27, 14), ("fp64", 3, 7, 20, 15), ("fp64", 3, 8, 33, 29),
                                                     ("fp64", 2, 10, 31, 32), ("fp64", 2, 11, 32, 33),
                                                     ("fp64", 2, 12, 45, 65), ("fp32", 3, 7, 27, 15),
                                                     ("fp32", 3, 8, 41, 28)])
def test_density_scores_match_oracle(g, prec_name, d, n, chi, ncand):
    print(f"[gpu-case] density scores {prec_name} d={d} n={n} chi={chi} candidates={ncand}", flush=True)
    fp32 = prec_name == "fp32"
    st, mats = saturated(g, d, n, chi, g.SCORE_FP32 if fp32 else g.SCORE_FP64, ncand)
    u = 2.0 ** -24 if fp32 else 2.0 ** -53
    for i in range(n - 1):
        s = st.score_bond(i)
        dims = [1] + st.bond_dims() + [1]
        cl, cr = dims[i], dims[i + 2]
        theta = np.tensordot(st.site(i), st.site(i + 1), axes=([2], [0]))
        t = theta.reshape(cl, d * d, cr)
        ref = np.array([renyi2(np.matmul(q, t).reshape(theta.shape)) for q in mats])
        tol = 4 * d * d * (max(cl, cr) + d ** 4) * u
        assert np.max(np.abs(s - ref)) <= tol, (i, cl, cr, np.max(np.abs(s - ref)), tol)


@pytest.mark.parametrize("d,n,ncand", [(3, 8, 40), (2, 12, 90)])
def test_density_window_choices(g, d, n, ncand):
    """FP32 first pass with its FP64 window against plain FP64 scoring: the same choices and bonds."""
    print(f"[gpu-case] density window d={d} n={n}", flush=True)
    c = brickwork_circuit(d, n, n + 6, n + 6, seed=77 + d)
    out = []
    for prec in (g.SCORE_FP64, g.SCORE_FP32):
        st = g.State(g.make_config(d, n, 32, 1e-10, score_prec=prec, max_candidates=ncand))
        st.set_candset(g.CandSet(d, candidate_words(d, ncand, 88)))
        g.run_circuit(st, c)
        out.append((st.choice_log(), st.bond_dims(), st.fidelity()))
    assert np.array_equal(out[0][0], out[1][0]) and out[0][1] == out[1][1]
    assert out[0][2] == out[1][2]


@pytest.mark.parametrize("prec_name,d,n,chi,ncand", [("bf16", 3, 8, 41, 64), ("bf16", 3, 8, 41, 65), ("fp32", 2, 12, 64, 128),
                                                     ("fp32", 2, 12, 64, 129), ("bf16", 2, 12, 64, 128),
                                                     ("bf16", 2, 12, 49, 129), ("bf16", 2, 12, 64, 300)])
def test_low_precision_sets_on_both_sides_of_the_rule(g, prec_name, d, n, chi, ncand):
    """Set sizes where BF16 (and, for qubits, FP32) scoring goes from rotated matrices to the density matrix in
    FP32.  The rotated form is held to half of the smallest re-score window (1e-4), as the window assumes; the
    density form to the FP32 bound above."""
    print(f"[gpu-case] low-precision rule {prec_name} d={d} chi={chi} candidates={ncand}", flush=True)
    st, mats = saturated(g, d, n, chi, g.SCORE_FP32 if prec_name == "fp32" else g.SCORE_BF16, ncand)
    density = ncand > (128 if d == 2 else 64)
    for i in range(n // 2 - 2, n // 2 + 2):
        s = st.score_bond(i)
        dims = [1] + st.bond_dims() + [1]
        cl, cr = dims[i], dims[i + 2]
        theta = np.tensordot(st.site(i), st.site(i + 1), axes=([2], [0]))
        t = theta.reshape(cl, d * d, cr)
        ref = np.array([renyi2(np.matmul(q, t).reshape(theta.shape)) for q in mats])
        tol = 4 * d * d * (max(cl, cr) + d ** 4) * 2.0 ** -24 if density else 5e-5
        assert np.max(np.abs(s - ref)) <= tol, (i, cl, cr, np.max(np.abs(s - ref)), tol)
