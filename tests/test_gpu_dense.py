"""The dense state C|MPS> against the dense product of the circuit's gates for every local dimension, at sizes
where the kernels' splits can go wrong: fewer indices than a wave, one wave less or more, remainders of the
four-index and 64-index steps, up to the largest size of each dimension, with both entry points.

Tolerance: a circuit of G gates without truncation errs by at most a few u per gate and split, far below 1e-11;
the sum over D terms adds sqrt(D) u.
"""
import numpy as np
import pytest

from oracle.statevector import simulate
from paper_2511_06672_amd.workload import brickwork_circuit, candidate_words

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def g():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_2511_06672_amd import gcamps
    gcamps.lib()
    return gcamps


@pytest.mark.parametrize("d,n", [(2, 2), (2, 6), (2, 7), (3, 2), (3, 4), (3, 7), (5, 2), (5, 4), (5, 6), (7, 2),
                                 (7, 3), (7, 5)])
def test_dense_state_matches_the_gates(g, d, n):
    print(f"[gpu-case] dense state d={d} n={n}", flush=True)
    c = brickwork_circuit(d, n, 6, 3, seed=60 + d + n, one_per_layer=False,
                          phases=[0.0] + [0.4 + 0.7 * k * k for k in range(1, d)])
    st = g.State(g.make_config(d, n, d ** (n // 2), 0.0, auto_disentangle=False))
    g.run_circuit(st, c)
    ref = simulate(c)
    got = st.statevector()
    assert abs(np.linalg.norm(got) - 1.0) <= 1e-11
    phase = np.vdot(got, ref)
    assert abs(abs(phase) - 1.0) <= 1e-11
    assert np.max(np.abs(got * phase - ref)) <= 1e-11
    assert np.array_equal(st.statevector_static(), got)
