"""The drift of a record is its template's, z(iz) / nharm to the last bit, by
whichever kernel its list was finished."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ntones,long_list", [(4, False), (40, True)])
@pytest.mark.parametrize("interbin", [False, True])
def test_drift_is_the_templates(gpu_lib, ntones, long_list, interbin):
    import torch
    nb = 1 << 15
    bank = gpu_lib.make_templates(8.0, 16.0 / 159.0)  # a step that is no short fraction
    plan = gpu_lib.Plan(bank, 2 * nb, 256, nharm_max=16, sigma=6.0, interbin=interbin, cand_capacity=1 << 20)
    rng = np.random.default_rng(ntones)
    X = (0.3 * (rng.standard_normal(nb) + 1j * rng.standard_normal(nb))).astype(np.complex64)
    X[8 + 8 * rng.permutation(nb // 8 - 2)[:ntones]] = 30.0
    X = torch.from_numpy(X).cuda()
    zs = np.array([bank.z(i) for i in range(bank.nz)])
    kind = gpu_lib.IN_SPECTRUM_NORMALISED
    for out in (None, gpu_lib.pinned_candidates(1 << 20)):
        c, found = plan.search(X, kind=kind, out=out) if out is not None else plan.search(X, kind=kind, cap=1 << 20)
        assert found == len(c) > 0 and (found > 8192) == long_list
        assert np.array_equal(c["z"], zs[c["iz"]] / c["nharm"])
        assert np.array_equal(c["r"], c["k"] / (c["nharm"] * (2.0 if interbin else 1.0)))
    plan.close()
    bank.close()
