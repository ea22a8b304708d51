"""Discarded weights of the truncation rule for more than 1024 values, where a thread of the rule's workgroup
holds two or four consecutive ones, with a spectral gap between the values of one thread: an odd number of
large values, then a tail 22 decades below them.

The matrices are diagonal, so that every product before the rule is exact and the rule sees sigma^2 to one
rounding.  Tolerance: the tail is a sum of at most 4096 positive numbers, each of which passes through fewer
additions than that, so its relative error is below 4096 2^-53 = 4.6e-13; 1e-12 with the roundings of
sigma^2, the total and the quotient.
"""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
HEAD = 257  # the first value of a wave's first thread, at two and at four values a thread


@pytest.fixture(scope="module")
def g():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_2511_06672_amd import gcamps
    gcamps.lib()
    return gcamps


def spectrum(m):
    """sigma: HEAD ones, then values from 1e-11 down (above the rank floor, no two degenerate)."""
    tail = 1e-11 * (1.0 - 1e-6 * np.arange(m - HEAD))
    return np.append(np.ones(HEAD), tail)


def tails(sig):
    w = [float(s) * float(s) for s in sig]
    total = math.fsum(w)
    return np.array([math.fsum(w[k:]) / total for k in range(HEAD, HEAD + 200)])


@pytest.mark.parametrize("m", [1025, 1536, 2187, 3072])
@pytest.mark.parametrize("part", [None, 0.95])
def test_tail_beside_a_gap(g, m, part):
    print(f"[gpu-case] truncation tail m={m} part={part}", flush=True)
    sig = spectrum(m)
    ref = tails(sig)
    # part: the cutoff as a share of the whole tail, so that a tail summed too small would be dropped whole
    cutoff = 1e-12 if part is None else part * ref[0]
    want = HEAD + int(np.argmax(ref <= cutoff))
    chi = -(-m // 3)
    assert HEAD <= want < chi
    st = g.State(g.make_config(3, 2, chi, cutoff, auto_disentangle=False, max_candidates=1))
    order = np.random.default_rng(m).permutation(m)
    got, k, eps, _, _ = st.factorize(np.diag(sig[order].astype(np.complex128)))
    assert np.max(np.abs(got / sig - 1.0)) <= 1e-15
    assert k == want
    assert abs(eps / ref[want - HEAD] - 1.0) <= 1e-12
