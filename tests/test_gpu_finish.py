"""Candidate finishing at the lengths where it changes form (one kernel,
its keys in tiles of 4096, up to 8192 records, a radix sort above) and for every kind of destination, and the
FP64 significance over its range."""
import numpy as np
import pytest

import paper_1511_07343_amd as fdas

pytestmark = pytest.mark.gpu

SMALL = 4096  # records of one tile of keys


def _search(lib, n_want, **opts):
    """A search whose list has exactly n_want records: a spectrum of isolated
    tones, one candidate each, on one template (powers only)."""
    import torch
    nb = 1 << 15
    rng = np.random.default_rng(n_want)
    X = np.zeros(nb, dtype=np.complex64)
    k = 4 + 4 * rng.permutation(nb // 4 - 2)[:n_want]
    X[k] = (10.0 + 30.0 * rng.random(n_want)) * np.exp(2j * np.pi * rng.random(n_want))
    bank = lib.make_templates(0.0, 1.0)
    plan = lib.Plan(bank, 2 * nb, 256, nharm_max=1, sigma=6.0, cand_capacity=1 << 14, **opts)
    return plan, bank, torch.from_numpy(X).cuda(), np.sort(k)


@pytest.mark.parametrize("n", [1, 63, 64, 65, 1000, SMALL - 1, SMALL, SMALL + 1, 7000])
def test_list_lengths_and_destinations(gpu_lib, n):
    plan, bank, X, k = _search(gpu_lib, n)
    pinned = gpu_lib.pinned_candidates(n)
    got, found = plan.search(X, kind=gpu_lib.IN_SPECTRUM_NORMALISED, out=pinned)
    assert found == n and np.array_equal(got["k"], k) and np.all(got["iz"] == 0)
    pageable, _ = plan.search(X, kind=gpu_lib.IN_SPECTRUM_NORMALISED)
    assert np.array_equal(got, pageable)
    # a capacity below the count: its first records, and the true count
    short, found = plan.search(X, kind=gpu_lib.IN_SPECTRUM_NORMALISED, cap=n // 2, allow_overflow=True)
    assert found == n and np.array_equal(short, pageable[: n // 2])
    out = gpu_lib.pinned_candidates(max(1, n // 2))
    short, found = plan.search(X, kind=gpu_lib.IN_SPECTRUM_NORMALISED, out=out, allow_overflow=True)
    assert found == n and np.array_equal(short, pageable[: len(out)])
    assert plan.search_counts()[0] == n
    # with the stages timed every kernel is enqueued at once
    plan.enable_timing(True)
    timed, _ = plan.search(X, kind=gpu_lib.IN_SPECTRUM_NORMALISED)
    assert np.array_equal(timed, pageable) and plan.stage_times()[1] == 1
    timed, _ = plan.search(X, kind=gpu_lib.IN_SPECTRUM_NORMALISED, out=pinned)
    assert np.array_equal(timed, pageable)
    plan.close()
    # refinement follows the finished list
    plan, bank2, X, k = _search(gpu_lib, n, refine_levels=1)
    refined, found = plan.search(X, kind=gpu_lib.IN_SPECTRUM_NORMALISED)
    assert found == n and np.array_equal(refined["k"], k)
    plan.close()
    bank.close()
    bank2.close()


@pytest.mark.parametrize("n", [200, SMALL + 500])
def test_batch_and_server_lists(gpu_lib, n):
    import torch
    bank = gpu_lib.make_templates(0.0, 1.0)
    opts = dict(nharm_max=1, sigma=6.0, cand_capacity=1 << 14)
    nsamp = 1 << 16
    x = np.zeros(nsamp)
    rng = np.random.default_rng(n)
    spec = np.zeros(nsamp // 2 + 1, dtype=complex)
    spec[4 + 4 * rng.permutation(nsamp // 8 - 2)[:n]] = 60.0
    spec[1:] += (rng.standard_normal(nsamp // 2) + 1j * rng.standard_normal(nsamp // 2))
    x = np.fft.irfft(spec * np.sqrt(nsamp), nsamp).astype(np.float32)
    plan = gpu_lib.Plan(bank, nsamp, 256, **opts)
    xd = torch.from_numpy(x).cuda()
    alone, found = plan.search(xd)
    assert (found > SMALL) == (n > SMALL) and found >= n
    for r in plan.search_batch([xd, xd, xd], caps=[1 << 14] * 3):
        assert np.array_equal(r, alone)
    server = gpu_lib.Server(bank, 256, nsamp, **opts)
    for i in range(3):
        server.submit(x, i)
    for _ in range(3):
        assert np.array_equal(server.poll()[1], alone)
    server.close()
    plan.close()
    bank.close()


@pytest.mark.parametrize("nharm", [1, 2, 4, 8, 16])
def test_significance_over_its_range(gpu_lib, nharm):
    """Records of known powers: refinement evaluates the significance of
    S(r, z) at the record's own point.  A spectrum that is constant has a
    power that is known from the host's FP64 function within float32."""
    import torch
    nb = 1 << 14
    bank = gpu_lib.make_templates(0.0, 1.0)
    plan = gpu_lib.Plan(bank, 2 * nb, 256, nharm_max=1, sigma=50.0)
    rng = np.random.default_rng(nharm)
    X = (10.0 ** rng.uniform(-1.5, 8.0, nb) * np.exp(2j * np.pi * rng.random(nb))).astype(np.complex64)
    plan.search(torch.from_numpy(X).cuda(), kind=gpu_lib.IN_SPECTRUM_NORMALISED, cap=0, allow_overflow=True)
    rec = np.zeros(400, dtype=gpu_lib.CAND_DTYPE)
    rec["nharm"], rec["iz"] = nharm, 0
    rec["k"] = nharm * rng.integers(20, nb // nharm - 40, len(rec))
    got = plan.refine(rec, 1)
    for c in got:
        want = gpu_lib.significance(float(c["power"]), nharm)
        # float32 result of an FP64 value
        assert abs(float(c["sigma"]) - want) <= 2.0 ** -23 * abs(want) + 1e-9, (c, want)
    plan.close()
    bank.close()
