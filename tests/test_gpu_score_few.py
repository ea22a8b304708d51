"""Scores of a few candidates at a large qutrit bond in FP32: which form they take, and their values against the FP64
mode's.  A form's score of a candidate does not depend on how many others are scored, and the two forms
round differently, so the scores of the first candidates of a larger set, which takes the density form, tell.

Tolerance: the low-precision modes' error in S2 is below half of the smallest allowed re-score window, 5e-5.
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


def entangled(g, t, prec):
    """2 t + 2 qutrits with every bond full up to 3^t."""
    n = 2 * t + 2
    for seed in range(40):
        c = brickwork_circuit(3, n, n + t, t, 11 + seed, one_per_layer=False)
        gates = [p for layer in c.layers for p in layer.phases]
        for layer in c.layers:
            layer.phases = []
        for k in range(t):
            c.layers[n + k].phases = [gates[k]]
        st = g.State(g.make_config(3, n, 3 ** t, 0.0, score_prec=prec, auto_disentangle=False, max_candidates=16))
        g.run_circuit(st, c)
        if st.bond_dims() == [3 ** min(j, n - j, t) for j in range(1, n)]:
            return st, n // 2 - 1
        st.close()
    raise AssertionError("no full state")


@pytest.mark.parametrize("t,cands,rotated", [(5, 1, True), (5, 8, True), (5, 9, False), (4, 8, False)])
def test_form_of_few_candidates(g, t, cands, rotated):
    print(f"[gpu-case] few candidates chi={3 ** t} {cands}", flush=True)
    words = candidate_words(3, 16, 21)
    st, bond = entangled(g, t, g.SCORE_FP32)
    st.set_candset(g.CandSet(3, words))
    many = st.score_bond(bond)
    st.set_candset(g.CandSet(3, words[:cands]))
    few = st.score_bond(bond)
    ref, bond = entangled(g, t, g.SCORE_FP64)
    ref.set_candset(g.CandSet(3, words))
    exact = ref.score_bond(bond)
    assert np.max(np.abs(many - exact)) <= 5e-5 and np.max(np.abs(few - exact[:cands])) <= 5e-5
    assert np.array_equal(few, many[:cands]) != rotated
