"""Weyl-string expectations against the dense state: chains whose sites all fit one workgroup, chains with a run
of larger sites in the middle (bonds of one tile, a remainder, up to 81) between two runs of small ones, and
every local dimension; identity, single-site, stabilizer and full-length strings with a phase.

Tolerance: E at each of n sites sums at most chi d products of entries below 1 after a normalised state: the
error is below n chi d u, 1e-12 with a margin of ten.
"""
import numpy as np
import pytest

from paper_2511_06672_amd.workload import SplitMix64, brickwork_circuit

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def g():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_2511_06672_amd import gcamps
    gcamps.lib()
    return gcamps


def dense_expectation(psi, d, n, x, z, p):
    """<psi| tau^p X^x Z^z |psi>, site 0 most significant."""
    v = psi.reshape((d,) * n)
    w = v
    for i in range(n):
        ph = np.exp(2j * np.pi * ((z[i] * np.arange(d)) % d) / d)
        w = np.roll(w * ph.reshape([-1 if k == i else 1 for k in range(n)]), x[i], axis=i)
    return np.exp(1j * np.pi * p / d) * np.vdot(v, w)


@pytest.mark.parametrize("d,n,chi,tdepth", [(2, 2, 2, 1), (2, 9, 16, 9), (2, 14, 128, 24), (3, 6, 27, 6), (3, 8, 36, 12),
                                            (3, 8, 37, 12), (3, 9, 81, 14), (5, 5, 25, 8), (7, 4, 49, 6)])
def test_expectations_match_dense_state(g, d, n, chi, tdepth):
    print(f"[gpu-case] expectations d={d} n={n} chi={chi}", flush=True)
    c = brickwork_circuit(d, n, n + 4, tdepth, seed=70 + d + n, one_per_layer=False,
                          phases=[0.0] + [0.4 + 0.7 * k * k for k in range(1, d)])
    st = g.State(g.make_config(d, n, chi, 0.0, auto_disentangle=False))
    g.run_circuit(st, c)
    print(f"bonds {st.bond_dims()}", flush=True)
    psi = st.statevector()
    psi = psi / np.linalg.norm(psi)
    rng = SplitMix64(17 * d + n)
    strings = [([0] * n, [0] * n, 0), ([0] * n, [1] + [0] * (n - 1), 1), ([0] * (n - 1) + [1], [0] * n, 2 * d - 1)]
    strings += [(list(map(int, r[:n])), list(map(int, r[n:2 * n])), int(r[2 * n])) for r in st.tableau()[:2]]
    strings += [([int(rng.below(d)) for _ in range(n)], [int(rng.below(d)) for _ in range(n)], k) for k in range(4)]
    norm = st.expectation(*strings[0])
    for x, z, p in strings:
        got = st.expectation(x, z, p) / norm.real
        ref = dense_expectation(psi, d, n, x, z, p)
        assert abs(got - ref) <= 1e-12, (x, z, p, got, ref)


@pytest.mark.parametrize("d,n", [(2, 1 + 63), (2, 65), (3, 100), (2, 128)])
def test_stabilizers_of_long_chains(g, d, n):
    """A Clifford state of up to the largest chain: every sampled row of its tableau has expectation 1."""
    print(f"[gpu-case] stabilizers d={d} n={n}", flush=True)
    c = brickwork_circuit(d, n, 5, 0, seed=80 + n, one_per_layer=False)
    st = g.State(g.make_config(d, n, 4, 0.0, auto_disentangle=False))
    g.run_circuit(st, c)
    tab = st.tableau()
    for k in (0, 1, n // 2, n - 1):
        r = [int(v) for v in tab[k]]
        assert abs(st.expectation(r[:n], r[n:2 * n], r[2 * n]) - 1.0) <= 1e-12
        assert abs(st.expectation(r[:n], r[n:2 * n], r[2 * n] + 1) - np.exp(1j * np.pi / d)) <= 1e-12
