"""The harmonic-sum screen, four harmonics and more on the plain plane.

The candidates of a search are compared with those of a direct evaluation on
the search's own plane: FP32 sums of every cell in the library's order, every
threshold and every neighbour.  The sums are the same single-precision numbers,
so the lists must be equal: a bin that the screen passed over shows as a
missing candidate.
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def _fraction(P, izc, j):
    """Term j of every cell: row and column rounded half away from zero."""
    nz, nb = P.shape
    d = np.arange(nz) - izc
    rows = izc + np.sign(d) * ((np.abs(d) * j + 8) >> 4)
    cols = (np.arange(nb, dtype=np.int64) * j + 8) >> 4
    return P[np.ix_(rows, cols)]


def _candidates(P, izc, nharm, thr):
    """{(nh, k, iz): power} of the cells that reach their level's threshold and
    exceed the four neighbours before them (in row order) and are not exceeded
    by the four after them."""
    v = {j: _fraction(P, izc, j) for j in range(1, 17) if j % (16 // nharm) == 0}
    s = v[16]
    sums = {1: s}
    if nharm >= 2:
        sums[2] = s = s + v[8]
    if nharm >= 4:
        sums[4] = s = s + (v[4] + v[12])
    if nharm >= 8:
        sums[8] = s = s + ((v[2] + v[6]) + (v[10] + v[14]))
    if nharm >= 16:
        sums[16] = s + (((v[1] + v[3]) + (v[5] + v[7])) + ((v[9] + v[11]) + (v[13] + v[15])))
    out = {}
    nz, nb = P.shape
    for nh, S in sums.items():
        pad = np.full((nz + 2, nb + 2), -np.inf, dtype=np.float32)
        pad[1:-1, 1:-1] = S
        keep = S >= thr[nh]
        for dz in (-1, 0, 1):
            for dk in (-1, 0, 1):
                if (dz, dk) == (0, 0):
                    continue
                other = pad[1 + dz:1 + dz + nz, 1 + dk:1 + dk + nb]
                keep &= S > other if (dz, dk) < (0, 0) else S >= other
        for iz, k in zip(*np.nonzero(keep)):
            out[(nh, int(k), int(iz))] = S[iz, k]
    return out


# lengths of fewer groups than a wave takes at a time, of one wave and of many
# tiles; rows of one and of several tiles; sparse and dense lists
@pytest.mark.parametrize("log2n,nz,nharm,sigma", [
    (10, 5, 4, 1.0), (11, 3, 8, 1.0), (10, 3, 16, 1.0), (12, 21, 16, 2.0), (15, 21, 4, 3.0), (15, 41, 8, 3.0),
    (15, 41, 16, 3.5), (18, 41, 16, 5.0), (20, 161, 16, 5.5), (20, 161, 4, 5.5),
])
def test_screen_misses_nothing(gpu_lib, log2n, nz, nharm, sigma):
    import torch
    n, zmax = 1 << log2n, 0.25 * (nz - 1)
    x = synth.make_series(n, seed=log2n + nz, pulsars=[synth.Pulsar(r=n / 37.0, z=0.4 * zmax, amp=0.15)]).x
    bank = gpu_lib.make_templates(zmax, 0.5)
    assert bank.nz == nz
    plan = gpu_lib.Plan(bank, n, 512 if nz > 41 else 256, nharm_max=nharm, sigma=sigma, median_window=256)
    plane = torch.empty((nz, n // 2), device="cuda")
    cands, found = plan.search(torch.from_numpy(x.astype(np.float32)).cuda(), plane=plane, cap=1 << 21)
    torch.cuda.synchronize()
    thr = {1 << l: np.float32(gpu_lib.threshold(sigma, 1 << l)) for l in range(5)}
    want = _candidates(plane.cpu().numpy(), (nz - 1) // 2, nharm, thr)
    got = {(int(c["nharm"]), int(c["k"]), int(c["iz"])): c["power"] for c in cands}
    assert found == len(cands) == len(got)
    assert len(got) > 0
    assert got.keys() == want.keys()
    assert all(got[key] == want[key] for key in got)
    plan.close()
    bank.close()
