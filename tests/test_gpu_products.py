"""Products at the edges of the tile forms, through the entry points that use them: splits whose Gram, rotation
and reconstruction products have one element more or less than a 16-row tile, K ranges of less than one group of
eight values, of one wave's share and of several, and sizes on both sides of the line between the two forms.

Tolerance: singular values, reconstruction and orthonormality of a split as elsewhere, a few m u with m the
smaller side; 1e-12 covers the largest (1100) with a decade to spare.
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


@pytest.mark.parametrize("p,q", [(33, 34), (47, 33), (48, 49), (33, 900), (900, 34), (63, 65), (64, 128), (65, 64),
                                 (255, 257), (1023, 64), (40, 1100), (1030, 1030)])
def test_split_products(g, p, q):
    print(f"[gpu-case] split products {p} x {q}", flush=True)
    chi = max(4, -(-min(p, q) // 3))
    while 27 * chi * chi < p * q or 3 * chi < min(p, q):
        chi += 1
    st = g.State(g.make_config(3, 2, chi, 0.0, auto_disentangle=False, max_candidates=1))
    rng = np.random.default_rng(p + q)
    m = rng.normal(size=(p, q)) + 1j * rng.normal(size=(p, q))
    m /= np.linalg.norm(m)
    sig, k, eps, left, right = st.factorize(m, factors=True)
    ref = np.linalg.svd(m, compute_uv=False)
    assert np.max(np.abs(sig[:k] - ref[:k])) <= 1e-12 * ref[0]
    kept = np.sqrt((ref[:k] ** 2).sum())
    assert np.linalg.norm(left @ right * kept - m) <= 1e-12 + np.sqrt((ref[k:] ** 2).sum()) * (1 + 1e-12)
    assert np.max(np.abs(left.conj().T @ left - np.eye(k))) <= 1e-12
