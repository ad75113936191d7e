"""Block medians by selection: one histogram, then the keys of one bucket ranked by counting.

The keys are given directly (a spectrum of real amplitudes), so the powers are
single roundings and the medians must equal numpy's exactly.  The blocks hold
what can go wrong: a bucket of more keys than the list takes, equal keys, a
middle pair split over two buckets, zeros, and windows from the smallest to the
largest.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _blocks(W, nblk, rng):
    """Amplitudes of nblk blocks of W bins, one kind of block after the other."""
    kinds = [
        lambda: np.sqrt(rng.exponential(1.0, W)),                            # noise
        lambda: np.full(W, 1.7),                                             # all equal: one bucket, one key
        lambda: 1.0 + np.arange(W) * 2.0**-18,                               # one bucket, all different
        lambda: np.where(np.arange(W) < W // 2, 0.5, 3.0),                   # the middle pair in two buckets
        lambda: np.where(np.arange(W) < W // 2 - 1, 0.5, 3.0),               # both of it in the upper one
        lambda: np.where(np.arange(W) < W // 2 + 1, 0.5, 3.0),               # both in the lower one
        lambda: np.where(rng.random(W) < 0.6, 0.0, rng.random(W)),           # mostly zeros
        lambda: 10.0 ** rng.uniform(-15, 15, W),                             # every exponent
        lambda: 1.0 + rng.integers(0, 3, W) * 2.0**-23,                      # neighbouring keys, many ties
    ]
    out = [rng.permutation(kinds[i % len(kinds)]()) for i in range(nblk)]
    return np.concatenate(out).astype(np.float32)


@pytest.mark.parametrize("W", [32, 64, 256, 512, 1024, 2048, 8192])
def test_medians_equal_sorted_ones(gpu_lib, W):
    import torch
    n = 1 << (19 if W > 2048 else 16)
    nb = n // 2
    amp = _blocks(W, nb // W, np.random.default_rng(W))
    bank = gpu_lib.make_templates(4.0, 2.0)
    plan = gpu_lib.Plan(bank, n, 256, nharm_max=1, sigma=20.0, median_window=W)
    plan.search(torch.from_numpy(amp.astype(np.complex64)).cuda(), kind=1, cap=1000, allow_overflow=True)
    medg = torch.empty(nb // W, dtype=torch.float64, device="cuda")
    plan.fetch_spectrum(None, medg)
    want = np.median((amp * amp).reshape(-1, W).astype(np.float64), axis=1)
    np.testing.assert_array_equal(medg.cpu().numpy(), want)
    plan.close()
    bank.close()
