"""The matrix-core correlators take templates in pairs +-z, whose taps are
conjugates of each other: that property of the banks, and the correlators at
the edges of their tiles (16 pairs per slice, 16 taps per step, 512 bins per
block) within the rounding bound derived in test_gpu_matrix."""
import numpy as np
import pytest

import oracle as O
import paper_1511_07343_amd as fdas
import synth
from test_gpu_matrix import _bound


@pytest.mark.parametrize("zmax,nz", [(0.0, 1), (1.0, 4), (7.5, 31), (20.0, 21), (64.0, 160), (200.0, 201), (510.0, 86)])
def test_taps_of_opposite_drifts_are_conjugate(zmax, nz):
    bank = fdas.make_templates(zmax, 2 * zmax / (nz - 1) if nz > 1 else 1.0)
    assert bank.nz == nz
    for iz in range((nz + 1) // 2):
        # each tap is formed in FP64 from Fresnel integrals of arguments up to ~30
        assert np.abs(bank.taps(iz) - bank.taps(nz - 1 - iz).conj()).max() < 1e-11
    bank.close()


@pytest.mark.gpu
@pytest.mark.parametrize("corr", ["bf16", "f16"])
@pytest.mark.parametrize("zmax,nz,log2n,seg,window", [
    (0.0, 1, 10, 256, 128),      # one template, its own pair; one block of 512 bins
    (1.0, 2, 11, 256, 256),      # one pair, no template at zero drift
    (8.0, 31, 12, 256, 256),     # 16 pairs, the last the zero-drift template
    (8.0, 32, 13, 256, 512),     # 16 pairs, all of two
    (16.0, 33, 13, 256, 512),    # a second slice of the zero-drift template alone
    (33.0, 66, 13, 512, 512),    # a third slice of one pair
    (510.0, 35, 13, 2048, 512),  # the widest templates (h = 271, 34 steps)
])
def test_matrix_pairs_within_rounding_bound(gpu_lib, corr, zmax, nz, log2n, seg, window):
    import torch
    n = 1 << log2n
    dz = 2 * zmax / (nz - 1) if nz > 1 else 1.0
    t = synth.make_series(n, seed=900 + nz, pulsars=[synth.Pulsar(r=n / 9.7, z=0.6 * zmax, amp=0.2)])
    bank = gpu_lib.make_templates(zmax, dz)
    plan = gpu_lib.Plan(bank, n, seg, correlator=corr, median_window=window, nharm_max=1)
    plane = torch.full((nz, n // 2), -1.0, dtype=torch.float32, device="cuda")
    plan.search(torch.from_numpy(t.x).cuda(), plane=plane)
    torch.cuda.synchronize()
    orc = O.search(t.x, zmax=zmax, dz=dz, sigma=6.0, nharm_max=1, W=window)
    E = _bound(t.x, zmax, dz, window, corr)
    assert np.all(np.abs(plane.cpu().numpy().astype(np.float64) - orc.plane) <= 2.0 * np.sqrt(orc.plane) * E + E * E)
    plan.close()
    bank.close()
