"""Lists around and beyond 4096 records, into every kind of destination: the
records are those of a timed search, which enqueues every kernel at once."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SMALL = 4096  # records of one tile of the one-kernel form


def _tones(nb, ntones, k_min, seed, noise=0.0):
    rng = np.random.default_rng(seed)
    X = (noise * (rng.standard_normal(nb) + 1j * rng.standard_normal(nb))).astype(np.complex64)
    k = k_min + 8 * rng.permutation((nb - k_min) // 8 - 1)[:ntones]
    X[k] = (10.0 + 30.0 * rng.random(ntones)) * np.exp(2j * np.pi * rng.random(ntones))
    return X


@pytest.mark.parametrize("zmax,dz,nharm,ntones,k_min,noise,long_list", [
    (0.0, 1.0, 16, 600, 1 << 14, 0.0, True),   # five records for the two cells of a tone
    (10.0, 1.0, 1, 1000, 8, 0.3, False),       # many cells, few of them maxima
    (10.0, 1.0, 4, 3000, 8, 0.3, True),
])
def test_list_destinations(gpu_lib, zmax, dz, nharm, ntones, k_min, noise, long_list):
    import torch
    nb = 1 << 15
    bank = gpu_lib.make_templates(zmax, dz)
    plan = gpu_lib.Plan(bank, 2 * nb, 256, nharm_max=nharm, sigma=6.0, cand_capacity=1 << 18)
    X = torch.from_numpy(_tones(nb, ntones, k_min, ntones, noise)).cuda()
    kind = gpu_lib.IN_SPECTRUM_NORMALISED
    plan.enable_timing(True)
    want, found = plan.search(X, kind=kind)
    plan.enable_timing(False)
    assert found == len(want) and (found > SMALL) == long_list
    key = (np.log2(want["nharm"]).astype(np.int64) * nb + want["k"]) * bank.nz + want["iz"]
    assert np.all(np.diff(key) > 0)
    for _ in range(3):
        pageable, n = plan.search(X, kind=kind)
        assert n == found and np.array_equal(pageable, want)
        pinned, n = plan.search(X, kind=kind, out=gpu_lib.pinned_candidates(found))
        assert n == found and np.array_equal(pinned, want)
        for cap in (0, 100, SMALL + 1, found - 1):
            short, n = plan.search(X, kind=kind, cap=cap, allow_overflow=True)
            assert n == found and np.array_equal(short, want[:cap])
    plan.close()
    bank.close()


@pytest.mark.parametrize("order", ["lsslllslss", "sl", "lll", "l"])
def test_batch_of_long_and_short_lists(gpu_lib, order):
    import torch
    n = 1 << 16
    bank = gpu_lib.make_templates(10.0, 1.0)
    plan = gpu_lib.Plan(bank, n, 256, nharm_max=4, sigma=6.0, median_window=256, cand_capacity=1 << 17)
    rng = np.random.default_rng(len(order))
    xs = []
    for c in order:
        spec = np.fft.rfft(rng.standard_normal(n))
        if c == "l":
            spec[8 * (1 + rng.permutation(n // 16 - 2)[:1500])] += 40.0 * np.sqrt(n)
        xs.append(torch.from_numpy(np.fft.irfft(spec, n).astype(np.float32)).cuda())
    want = [plan.search(x)[0] for x in xs]
    assert [len(w) > SMALL for w in want] == [c == "l" for c in order]
    caps = [len(w) + 1 for w in want]
    pinned = gpu_lib.pinned_candidates(sum(caps))
    for _ in range(2):
        for got in (plan.search_batch(xs, caps=caps), plan.search_batch(xs, caps=caps, out=pinned)):
            assert all(np.array_equal(g, w) for g, w in zip(got, want))
    plan.close()
    bank.close()


@pytest.mark.parametrize("n", [4096, 4097, 8191, 8192, 8193, 12289, 32767, 32768, 32769, 40000])
def test_lengths_where_the_form_changes(gpu_lib, n):
    """8192 records: one kernel below, a sort above; 32768: the last that reach
    ordinary memory through the plan's page-locked records."""
    import torch
    nb = 1 << 19
    bank = gpu_lib.make_templates(0.0, 1.0)
    plan = gpu_lib.Plan(bank, 2 * nb, 256, nharm_max=1, sigma=6.0, cand_capacity=1 << 16)
    X = _tones(nb, n, 8, n)
    k = np.flatnonzero(X)
    X, kind = torch.from_numpy(X).cuda(), gpu_lib.IN_SPECTRUM_NORMALISED
    plan.enable_timing(True)
    want, found = plan.search(X, kind=kind)
    plan.enable_timing(False)
    assert found == n and np.array_equal(want["k"], k)
    pageable, found = plan.search(X, kind=kind)
    assert found == n and np.array_equal(pageable, want)
    pinned, found = plan.search(X, kind=kind, out=gpu_lib.pinned_candidates(n))
    assert found == n and np.array_equal(pinned, want)
    for cap in (1, n // 2, n - 1):
        short, found = plan.search(X, kind=kind, cap=cap, allow_overflow=True)
        assert found == n and np.array_equal(short, want[:cap])
        short, found = plan.search(X, kind=kind, out=gpu_lib.pinned_candidates(cap), allow_overflow=True)
        assert found == n and np.array_equal(short, want[:cap])
    plan.close()
    bank.close()
