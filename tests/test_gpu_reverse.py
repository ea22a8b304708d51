"""The reverse sweep at sizes on both sides of its one-workgroup forms (8192 entries of a two-site matrix) and
for every local dimension, with and without disentangling, against the dense derivative.

Tolerance: as for the other exact gradients, the rounding of a few hundred FP64 steps whose splits divide by
gaps of at least 1e-5 of the largest value: 1e-8 of the largest component.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,n,layers,nphase,ncand", [(2, 5, 4, 10, 6), (3, 9, 4, 10, 5), (3, 9, 6, 14, 4),
                                                    (5, 4, 6, 12, 0), (5, 4, 6, 12, 6), (7, 3, 3, 5, 0), (7, 3, 3, 5, 5)])
def test_gradient_matches_dense_derivative(d, n, layers, nphase, ncand):
    from oracle.gradient import dense_gradient, dense_loss
    from paper_2511_06672_amd import gcamps as g
    from paper_2511_06672_amd.workload import brickwork_circuit, candidate_words
    print(f"[gpu-case] reverse sweep d={d} n={n} gates={nphase} candidates={ncand}", flush=True)
    c = brickwork_circuit(d, n, layers, nphase, seed=120 + d + n, one_per_layer=False, parametrised=True, ngens=4)
    items = sorted((ph.param, ph.phi[1:]) for L in c.layers for ph in L.phases if ph.param >= 0)
    th = np.array([x for _, phi in items for x in phi])
    dense = dense_gradient(c, th)
    assert np.max(np.abs(dense)) > 1e-3
    cands = g.CandSet(d, candidate_words(d, ncand, 905)) if ncand else None
    cfg = g.make_config(d, n, d ** (n // 2), 1e-12, auto_disentangle=bool(ncand), max_candidates=max(ncand, 1))
    gr = g.Gradient(cfg, c, cands, th)
    loss, grad = gr.gradient(th)
    assert abs(loss - dense_loss(c, th)) <= 1e-10
    err = np.max(np.abs(grad - dense)) / np.max(np.abs(dense))
    print(f"[gpu-case] error {err:.2e}", flush=True)
    assert err <= 1e-8
    gr.close()
