"""Block-Jacobi eigensolver at the sizes where its tiling changes: the largest matrix of one workgroup
and the first of the block form, one pair of blocks more or less than full, an odd and an even number
of tiles, the last size with two sweeps per read-back, and both sides of the sizes whose rounds
hold a CU per block.  Every size goes through the absolute criterion, and through the relative one by
the rank-reduced path (sides above 320).

Tolerances: the criterion leaves off-diagonal entries of at most 2e-15 of the trace, so a kept
sigma_i^2 errs by less than that and the rounding of the Gram (m eps trace); both are below
m 2^-52 + 4e-15 of the trace, and columns tilt by at most 2e-15 trace / lambda_kept plus the rounding
of the rotations (2^-53 per rotation step, about 20 m steps).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def g():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_2511_06672_amd import gcamps
    gcamps.lib()
    return gcamps


def graded(m, decades, seed):
    rng = np.random.default_rng(seed)
    a = rng.standard_normal((m, m)) + 1j * rng.standard_normal((m, m))
    b = rng.standard_normal((m, m)) + 1j * rng.standard_normal((m, m))
    x = (a * 10.0 ** (-decades * np.arange(m) / m)) @ b
    return x / np.linalg.norm(x)


@pytest.mark.parametrize("m,reduce", [(15, False), (16, False), (17, False), (31, False), (32, False), (33, False),
                                      (64, False), (65, False), (95, False), (97, False), (256, False), (257, False),
                                      (321, True), (353, True), (640, True), (897, False)])
def test_decomposition_at_tile_edges(g, m, reduce):
    print(f"[gpu-case] jacobi m={m} reduce={reduce}", flush=True)
    x = graded(m, 2.0, 40 + m)
    chi = -(-m // 3)
    st = g.State(g.make_config(3, 2, chi, 1e-10, auto_disentangle=False, max_candidates=1))
    sig, k, eps, L, R = st.factorize(x, factors=True, reduce=reduce)
    ref = np.linalg.svd(x, compute_uv=False)
    tr = np.sum(ref ** 2)
    assert k == min(chi, m)
    assert np.max(np.abs(sig[:k] ** 2 - ref[:k] ** 2)) <= (m * 2.0 ** -52 + 4e-15) * tr
    tilt = 2e-15 * tr / ref[k - 1] ** 2 + 20 * m * 2.0 ** -53
    assert np.max(np.abs(L.conj().T @ L - np.eye(k))) <= tilt
    assert np.max(np.abs(L @ R - (L @ (L.conj().T @ x)) / np.linalg.norm(ref[:k]))) <= tilt
