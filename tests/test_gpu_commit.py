"""The commit of a bond (choice, rotation of Theta, tableau update) leaves the represented state as it was:
expectations of the Clifford frame's stabilizers and of their products with a phase before and after a sweep
that accepts candidates, for every local dimension, every rule of choice, fewer candidates than a workgroup,
one more and several times as many, and chains of more than 64 sites, where a lane carries two sites.

Tolerance: without truncation (cutoff 0, bonds below chi_max) each of the 2 (n - 1) splits and each
expectation errs by a few d chi u: 2 n splits give below 1e-12, one decade of margin for the smaller chains.
"""
import numpy as np
import pytest

from paper_2511_06672_amd.workload import brickwork_circuit, candidate_words

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def g():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_2511_06672_amd import gcamps
    gcamps.lib()
    return gcamps


@pytest.mark.parametrize("rule,d,n,ncand", [("fp64", 2, 8, 40), ("fp64", 3, 7, 257), ("fp64", 5, 5, 30),
                                            ("fp64", 7, 4, 12), ("fp64", 2, 70, 600), ("fp64", 3, 66, 20),
                                            ("window", 2, 9, 300), ("window", 3, 7, 64), ("rank", 2, 9, 255),
                                            ("rank", 3, 6, 33), ("rank", 5, 4, 9)])
def test_commit_keeps_the_state(g, rule, d, n, ncand):
    print(f"[gpu-case] commit rule={rule} d={d} n={n} candidates={ncand}", flush=True)
    c = brickwork_circuit(d, n, 4, 3, seed=90 + d + n, one_per_layer=False,
                          phases=[0.0] + [0.4 + 0.7 * k * k for k in range(1, d)])
    kw = {"score_prec": g.SCORE_FP32} if rule == "window" else {}
    if rule == "rank":
        kw["criterion"] = g.CRITERION_BOND_DIM
    st = g.State(g.make_config(d, n, 64, 0.0, auto_disentangle=False, max_candidates=ncand, **kw))
    g.run_circuit(st, c)
    rows = [[int(v) for v in r] for r in st.tableau()[:n]]
    pick = sorted({0, 1, n // 2, n - 2, n - 1})
    strings = [(rows[k][:n], rows[k][n:2 * n], rows[k][2 * n]) for k in pick]
    strings += [([(a + b) % d for a, b in zip(rows[k][:n], rows[k + 1][:n])],
                 [(a + b) % d for a, b in zip(rows[k][n:2 * n], rows[k + 1][n:2 * n])], 1) for k in pick[:-1]]
    before = np.array([st.expectation(*s) for s in strings])
    assert max(st.bond_dims()) > 1
    st.set_candset(g.CandSet(d, candidate_words(d, ncand, 95 + d)))
    sweeps, changed = st.disentangle()
    print(f"changed {changed}", flush=True)
    assert changed > 0
    after = np.array([st.expectation(*s) for s in strings])
    assert np.max(np.abs(after - before)) <= 1e-11, np.max(np.abs(after - before))
