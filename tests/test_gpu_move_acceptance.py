"""When a move of the orthogonality centre may take the Cholesky factorisation's orthonormal factor X K^-H.

Two Newton-Schulz steps take a defect S = X^H X of norm e = |S - I| to 3/4 (3/4 e^2)^2, so what the factorisation
reports as the defect must bound the spectral norm, not an entry: below 1e-4 the result is orthonormal to
4.3e-17.
"""
import ctypes as C
import re

import numpy as np
import pytest

from paper_2511_06672_amd.workload import brickwork_circuit, candidate_words

pytestmark = pytest.mark.gpu
IDENTITY_GAP = "_ZN2gc19launch_identity_gapEP12ihipStream_tPKNS_2cxIdEEiPNS_9CholStateE"


@pytest.fixture(scope="module")
def g():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_2511_06672_amd import gcamps
    gcamps.lib()
    return gcamps


def reported_gap(g, s):
    """The library's kernel on the matrix s: the gap in the state's third field."""
    import torch
    launch = getattr(C.CDLL(g.LIB_PATH), IDENTITY_GAP)
    launch.argtypes = [C.c_void_p, C.c_void_p, C.c_int, C.c_void_p]
    launch.restype = None
    dev = torch.from_numpy(np.ascontiguousarray(s)).cuda()
    st = torch.zeros(3, dtype=torch.float64, device="cuda")
    launch(torch.cuda.current_stream().cuda_stream, dev.data_ptr(), s.shape[0], st.data_ptr())
    return float(st.cpu()[2])


@pytest.mark.parametrize("m", [1, 33, 64, 243, 300])
@pytest.mark.parametrize("kind", ["coherent", "random", "one"])
def test_gap_bounds_the_norm(g, m, kind):
    print(f"[gpu-case] identity gap m={m} {kind}", flush=True)
    rng = np.random.default_rng(m)
    if kind == "coherent":
        e = np.full((m, m), 9e-6, dtype=complex)
    elif kind == "random":
        e = 1e-6 * (rng.standard_normal((m, m)) + 1j * rng.standard_normal((m, m)))
        e = e + e.conj().T
    else:
        e = np.zeros((m, m), dtype=complex)
        e[m - 1, 0] = e[0, m - 1] = 1e-3
    got = reported_gap(g, np.eye(m) + e)
    norm, rows = np.linalg.norm(e, 2), np.abs(e).sum(axis=1).max()
    # 1 + e rounds e by 2^-53 an entry; |re| + |im| is at most sqrt(2) |e|
    slack = m * 2.0 ** -52
    assert norm - slack <= got <= np.sqrt(2.0) * rows + slack


def test_gap_of_a_matrix_with_nan_refuses(g):
    s = np.eye(70, dtype=complex)
    s[3, 60] = np.nan
    assert reported_gap(g, s) >= 1e30


@pytest.mark.parametrize("phi,side", [(0.5, "cholesky"), (0.2, None), (0.15, None), (0.12, None), (0.1, None), (0.06, None),
                                      (0.04, None), (0.02, None), (0.01, "eigen")])
def test_moves_on_both_sides_of_the_acceptance_line(g, phi, side, monkeypatch, capfd):
    """Four weak gates on a chain of qutrits: bonds of 81 whose Schmidt weights are products of factors
    phi^2 / 3, the smallest about (phi^2 / 3)^4 of the largest, from 5e-5 to 1e-18 of it (the line is a pivot of
    1e-9).  Whichever way a move takes, the site it leaves is orthonormal and the state is the same.  Tolerances: the
    products of a move sum up to 3 chi = 243 terms, 243 2^-53 = 2.7e-14; an eigen-decomposition's factor tilts by
    up to 3e-16 / lambda with lambda down to 1e-12, where its relative pass takes over."""
    print(f"[gpu-case] moves phi={phi}", flush=True)
    monkeypatch.setenv("GCAMPS_TRACE_FACT", "1")
    d, n, t = 3, 10, 4
    c = brickwork_circuit(d, n, n + t, t, 5, phases=(0.0, phi, -phi), one_per_layer=False)
    gates = [p for layer in c.layers for p in layer.phases]
    for layer in c.layers:
        layer.phases = []
    for k in range(t):
        c.layers[n + k].phases = [gates[k]]
    st = g.State(g.make_config(d, n, 81, 0.0, auto_disentangle=False, max_candidates=1))
    st.set_candset(g.CandSet(d, candidate_words(d, 1, 5)))
    g.run_circuit(st, c)
    before = st.statevector()
    st.score_bond(0)
    seen = set()
    for bond in (n - 2, 0, n - 2):
        capfd.readouterr()
        st.score_bond(bond)
        moves = re.findall(r"gcamps-fact m=(\d+) .*? sweeps=(\S+)", capfd.readouterr().err)
        assert len(moves) == n - 2
        for j, (m, sweeps) in enumerate(moves):
            i = j if bond else n - 2 - j
            a = np.asarray(st.site(i))
            if bond:
                a = a.reshape(-1, a.shape[2])
                defect = a.conj().T @ a
            else:
                a = a.reshape(a.shape[0], -1)
                defect = a @ a.conj().T
            way = "small" if int(m) <= 32 else "cholesky" if sweeps == "0/0/0" else "eigen"
            seen.add((int(m), way))
            tol = 1e-13 if way == "cholesky" else 1e-13 + 3e-16 / 1e-12
            assert np.max(np.abs(defect - np.eye(len(defect)))) <= tol, (bond, i, way)
    after = st.statevector()
    assert np.max(np.abs(after - before)) <= 1e-12 * np.max(np.abs(before)) * np.sqrt(len(before))
    print(f"  bonds {st.bond_dims()} moves {sorted(seen)}", flush=True)
    assert max(m for m, _ in seen) > 32
    if side:
        assert (81, side) in seen
