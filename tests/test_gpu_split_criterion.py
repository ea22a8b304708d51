"""What the splits' convergence criterion leaves of a rotation between kept and discarded directions, and exactly
degenerate spectra, where rotations never end if the criterion lies below their rounding.

The sweeps stop at off-diagonal entries of 3e-16 of the trace.  An entry g between a kept and a discarded
direction of Gram eigenvalues a > b tilts the kept space by g / (a - b); the products before and after the sweeps
(four of them, entries of at most the trace) add 2^-53 of the trace each.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
CRITERION = 3e-16
ROUNDING = 4 * 2.0 ** -53


@pytest.fixture(scope="module")
def g():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_2511_06672_amd import gcamps
    gcamps.lib()
    return gcamps


def unitary_columns(rng, m, k):
    return np.linalg.qr(rng.standard_normal((m, k)) + 1j * rng.standard_normal((m, k)))[0]


def pivots(gram, count):
    s, out = gram.copy(), []
    for _ in range(count):
        diag = s.diagonal().real.copy()
        diag[out] = -1.0
        p = int(np.argmax(diag))
        col = s[:, p] / np.sqrt(diag[p])
        s = s - np.outer(col, col.conj())
        out.append(p)
    return out


def nearly_tied(seed, m=384, r=40, weight=1.5e-15, gap=1e-7):
    """r directions u (more than the 32 of the single-workgroup eigensolver), eight of them with nearly all of the
    weight, of which numbers 5 and 6 have nearly the same, and one more whose weight is below the bound at which the
    pivoted factorisation stops, orthogonal to all of u but with the sum of the two at
    the pivots' rows: the factorisation's basis mixes the two by weight / (their gap), and the exact
    invariant spaces are those of u."""
    rng = np.random.default_rng(seed)
    u, v = unitary_columns(rng, m, r), unitary_columns(rng, m, r + 1)
    lam = np.append(1.0 + 0.3 * np.arange(8)[::-1], 1e-2 * (1.0 - 0.01 * np.arange(r - 8)))
    lam[5] = lam[4] * (1.0 - gap)
    lam /= lam.sum()
    top = u * np.sqrt(lam)
    piv = pivots(top @ top.conj().T, r)
    rest = np.setdiff1d(np.arange(m), piv)
    a = np.zeros(m, dtype=complex)
    a[piv] = u[piv][:, [4, 5]].sum(axis=1)
    a[rest] = -u[rest] @ np.linalg.solve(u[rest].conj().T @ u[rest], u[piv].conj().T @ a[piv])
    return u, lam, top @ v[:, :r].conj().T + np.sqrt(weight) * np.outer(a, v[:, r].conj())


@pytest.mark.parametrize("seed", [0, 1, 2])
def test_reduced_split_does_not_mix_kept_and_discarded(g, seed):
    print(f"[gpu-case] reduced split, nearly tied cut, seed {seed}", flush=True)
    u, lam, x = nearly_tied(seed)
    st = g.State(g.make_config(3, 2, 5, 1e-10, auto_disentangle=False, max_candidates=1, max_gate_terms=81))
    sig, k, eps, left, _ = st.factorize(x, factors=True, reduce=True)
    assert k == 5 and np.count_nonzero(sig) == 40       # the reduced path, cut between the two
    tilt = np.abs(u[:, 5:].conj().T @ left)
    assert np.max(tilt) <= (CRITERION + ROUNDING) / (lam[4] - lam[5])


@pytest.mark.parametrize("m", [12, 24, 33, 48, 97, 243])
def test_sweeps_stop_at_their_criterion(g, m):
    """A Gram that is diagonal but for one entry of 1.2e-15 of the trace, above the criterion and below the looser one
    that sweeps had before (2e-15), between the last kept direction and the first dropped one."""
    print(f"[gpu-case] plain split, one entry off the diagonal, m={m}", flush=True)
    lam = np.append(1.0 + 0.3 * np.arange(8)[::-1], 1e-2 * (1.0 - 0.003 * np.arange(m - 8)))
    lam[5] = lam[4] * (1.0 - 1e-7)
    lam /= lam.sum()
    x = np.diag(np.sqrt(lam)).astype(complex)
    x[5, 4] = 1.2e-15j / x[4, 4].real                   # G[5, 4] = 1.2e-15 i
    theta = 0.5 * np.arctan2(2 * 1.2e-15, lam[4] - lam[5])
    dropped = np.zeros(m, dtype=complex)
    dropped[4], dropped[5] = 1j * np.sin(theta), np.cos(theta)
    st = g.State(g.make_config(3, 2, 5, 1e-10, auto_disentangle=False, max_candidates=1, max_gate_terms=81))
    sig, k, eps, left, _ = st.factorize(x, factors=True)
    assert k == 5
    assert np.max(np.abs(dropped.conj() @ left)) <= (CRITERION + ROUNDING) / (lam[4] - lam[5])


@pytest.mark.parametrize("m,equal,reduce", [(20, 2, False), (32, 8, False), (33, 2, False), (48, 3, False), (81, 2, False),
                                            (81, 8, False), (97, 5, False), (243, 2, False), (243, 4, False),
                                            (333, 2, True), (333, 8, True)])
def test_exactly_degenerate_spectra(g, m, equal, reduce):
    """`equal` values of 1 and the rest zero, in the diagonal basis times random unitaries: the whole trace in a
    few values is where the criterion, relative to the trace, is closest to the rounding of a rotation."""
    print(f"[gpu-case] degenerate m={m} equal={equal} reduce={reduce}", flush=True)
    chi = -(-m // 3)
    st = g.State(g.make_config(3, 2, chi, 1e-10, auto_disentangle=False, max_candidates=1))
    for seed in range(4):
        rng = np.random.default_rng(100 * m + 10 * equal + seed)
        u, v = unitary_columns(rng, m, equal), unitary_columns(rng, m, equal)
        x = u @ v.conj().T
        sig, k, eps, left, right = st.factorize(x, factors=True, reduce=reduce)
        assert k == equal
        # sums of m products of entries below 1 and about 20 m rotations a vector
        tol = 20 * m * 2.0 ** -53
        assert np.max(np.abs(sig[:k] - 1.0)) <= tol
        assert np.max(np.abs(left.conj().T @ left - np.eye(k))) <= tol
        assert np.max(np.abs(left @ right * np.sqrt(equal) - x)) <= tol
