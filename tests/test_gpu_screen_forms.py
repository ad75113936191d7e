"""The screen's remaining forms against a direct evaluation of the search's own
plane, as in test_gpu_screen: one and two harmonics, the half-bin plane (a code
for each pair k, k + 1/2) and the own-row form of the time-domain search."""
import numpy as np
import pytest

import synth
import test_gpu_screen as direct

pytestmark = pytest.mark.gpu


def _check(lib, plan, x, rows, columns, nharm, sigma, izc, unfold=None):
    import torch
    plane = torch.empty((rows, columns), device="cuda")
    cands, found = plan.search(torch.from_numpy(x.astype(np.float32)).cuda(), plane=plane, cap=1 << 21)
    torch.cuda.synchronize()
    P = plane.cpu().numpy()
    P = unfold(P) if unfold else P
    thr = {1 << l: np.float32(lib.threshold(sigma, 1 << l)) for l in range(5)}
    want = direct._candidates(P, izc, nharm, thr)
    got = {(int(c["nharm"]), int(c["k"]), int(c["iz"])): c["power"] for c in cands}
    assert found == len(cands) == len(got) > 0
    assert got.keys() == want.keys()
    assert all(got[key] == want[key] for key in got)


def _series(log2n, zmax):
    return synth.make_series(1 << log2n, seed=log2n, pulsars=[synth.Pulsar(r=(1 << log2n) / 37.0, z=0.4 * zmax, amp=0.15)]).x


@pytest.mark.parametrize("log2n,nz,nharm,sigma", [(10, 3, 1, 1.0), (15, 41, 1, 3.0), (18, 21, 1, 4.0), (10, 5, 2, 1.0),
                                                  (15, 21, 2, 3.0), (20, 161, 2, 5.5)])
def test_one_and_two_harmonics(gpu_lib, log2n, nz, nharm, sigma):
    zmax = 0.25 * (nz - 1)
    bank = gpu_lib.make_templates(zmax, 0.5)
    plan = gpu_lib.Plan(bank, 1 << log2n, 512 if nz > 41 else 256, nharm_max=nharm, sigma=sigma, median_window=256)
    _check(gpu_lib, plan, _series(log2n, zmax), nz, 1 << (log2n - 1), nharm, sigma, (nz - 1) // 2)
    plan.close()
    bank.close()


@pytest.mark.parametrize("log2n,nz,nharm,sigma", [(10, 3, 1, 1.0), (11, 5, 2, 1.5), (14, 21, 4, 3.0), (15, 21, 8, 3.0),
                                                  (18, 41, 16, 5.0)])
def test_half_bin_plane(gpu_lib, log2n, nz, nharm, sigma):
    zmax, nb = 0.25 * (nz - 1), 1 << (log2n - 1)

    def unfold(P):  # bins, then half-bin points, to columns of half bins
        out = np.empty_like(P)
        out[:, 0::2], out[:, 1::2] = P[:, :nb], P[:, nb:]
        return out
    bank = gpu_lib.make_templates(zmax, 0.5)
    plan = gpu_lib.Plan(bank, 1 << log2n, 256, nharm_max=nharm, sigma=sigma, median_window=256, interbin=True)
    _check(gpu_lib, plan, _series(log2n, zmax), nz, 2 * nb, nharm, sigma, (nz - 1) // 2, unfold)
    plan.close()
    bank.close()


@pytest.mark.parametrize("log2n,nalpha,nharm,sigma", [(10, 1, 1, 1.0), (11, 3, 2, 1.5), (14, 9, 4, 3.0), (15, 17, 8, 3.0),
                                                      (18, 21, 16, 4.0)])
def test_time_domain_rows(gpu_lib, monkeypatch, log2n, nalpha, nharm, sigma):
    # every term of a row's sums comes from the row itself
    monkeypatch.setattr(direct, "_fraction", lambda P, izc, j: P[:, (np.arange(P.shape[1], dtype=np.int64) * j + 8) >> 4])
    plan = gpu_lib.TdPlan(1 << log2n, 0.01, nalpha, nharm_max=nharm, sigma=sigma, median_window=256)
    _check(gpu_lib, plan, _series(log2n, 0.0), nalpha, 1 << (log2n - 1), nharm, sigma, 0)
    plan.close()
