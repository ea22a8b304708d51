"""One-launch split of small matrices (smaller side at most 32, larger at most 512) against LAPACK and the
oracle's truncation rule: both orientations, single rows and columns, sides around the 16 and 32 index
kernels, larger sides that are no multiple of a 16-column chunk, the last size of the launch and the
first beyond it, exact rank deficiency and a graded spectrum that needs the second pass.

Tolerances: sigma_i^2 errs by the rounding of the Gram and of the sweeps, below (kw + 64) 2^-52 of the
trace, plus 2e-15 of it left off the diagonal; the factors' columns by that over lambda_kept plus the
rounding of the rotations.  With the second pass a kept sigma is accurate to the rounding of the input,
2^-52 sqrt(kw) sigma_0; the second pass counts an off-diagonal entry of at most 1e-29 trace / m as
converged, which tilts the columns B^H / sigma of a tall matrix by up to that over lambda_kept.
"""
import numpy as np
import pytest

from oracle.mps import rtrunc

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def g():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_2511_06672_amd import gcamps
    gcamps.lib()
    return gcamps


def gauss(rng, p, q):
    return rng.standard_normal((p, q)) + 1j * rng.standard_normal((p, q))


def state(g, cutoff, chi=300):
    return g.State(g.make_config(2, 2, chi, cutoff, auto_disentangle=False, max_candidates=1))


@pytest.mark.parametrize("p,q", [(1, 1), (1, 512), (512, 1), (2, 3), (8, 8), (9, 17), (17, 9), (16, 512), (16, 513),
                                 (17, 511), (513, 31), (512, 32), (32, 33), (5, 31)])
def test_small_split_shapes(g, p, q):
    print(f"[gpu-case] small split {p} x {q}", flush=True)
    rng = np.random.default_rng(p * 1000 + q)
    x = gauss(rng, p, q)
    sig, k, eps, L, R = state(g, 1e-10).factorize(x, factors=True)
    ref = np.linalg.svd(x, compute_uv=False)
    kr, er, _ = rtrunc(ref, 1e-10, 300)
    tr = np.sum(ref ** 2)
    tol = (max(p, q) + 64) * 2.0 ** -52 + 2e-15
    assert k == kr and abs(eps - er) <= tol
    assert np.all(np.diff(sig) <= 0) and np.max(np.abs(sig ** 2 - ref ** 2)) <= tol * tr
    tilt = tol * tr / ref[k - 1] ** 2 + 640 * 2.0 ** -53
    assert np.max(np.abs(L.conj().T @ L - np.eye(k))) <= tilt
    assert np.max(np.abs(R - L.conj().T @ x / np.linalg.norm(ref[:k]))) <= tilt


@pytest.mark.parametrize("p,q,r", [(9, 27, 4), (27, 9, 4), (30, 64, 11), (32, 32, 1)])
def test_small_split_rank_floor(g, p, q, r):
    print(f"[gpu-case] small split, exact rank {r} in {p} x {q}, cutoff 0", flush=True)
    rng = np.random.default_rng(p + q + r)
    x = gauss(rng, p, r) @ gauss(rng, r, q)
    sig, k, eps, L, R = state(g, 0.0).factorize(x, factors=True)
    ref = np.linalg.svd(x, compute_uv=False)
    assert k == r and eps <= 1e-26
    assert np.max(np.abs(sig[:k] - ref[:k])) <= 2.0 ** -52 * np.sqrt(max(p, q)) * 8 * ref[0]
    assert np.max(np.abs(L @ R * np.linalg.norm(ref) - x)) <= 1e-13 * ref[0]


@pytest.mark.parametrize("m,kw", [(14, 20), (32, 48)])
def test_small_split_graded_second_pass(g, m, kw):
    print(f"[gpu-case] small split, graded spectrum {m} x {kw}", flush=True)
    rng = np.random.default_rng(m)
    u, _ = np.linalg.qr(gauss(rng, m, m))
    v, _ = np.linalg.qr(gauss(rng, kw, m))
    true = 10.0 ** (-1.1 * np.arange(m))
    for x in ((u * true) @ v.conj().T, (v * true) @ u.conj().T):
        sig, k, _, L, R = state(g, 0.0).factorize(x, factors=True)
        assert k == 12                 # 10^-12.1 > 1e-13 > 10^-13.2
        assert np.max(np.abs(sig[:k] - true[:k])) <= 2.0 ** -52 * np.sqrt(kw) * 8
        tilt = 1e-12 if x.shape[0] <= x.shape[1] else 1e-29 * np.sum(true ** 2) / (m * true[k - 1] ** 2)
        assert np.max(np.abs(L.conj().T @ L - np.eye(k))) <= tilt
