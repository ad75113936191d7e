"""Splits of the work that are chosen by the launch's size do not change a
result: templates per correlation workgroup, and the trials of a time-domain
search whose spectra are formed together."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def _dev(x):
    import torch
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


@pytest.mark.parametrize("log2n,zmax,nz,seg,interbin", [
    (12, 8.0, 5, 256, False),      # a workgroup per template
    (15, 20.0, 21, 512, False),
    (17, 100.0, 101, 2048, False),
    (17, 100.0, 34, 8192, True),   # a few templates each
    (18, 8.0, 33, 256, False),     # many workgroups
])
def test_templates_per_workgroup(gpu_lib, log2n, zmax, nz, seg, interbin):
    import torch
    x = _dev(synth.make_series(1 << log2n, seed=nz).x)
    bank = gpu_lib.make_templates(zmax, 2 * zmax / (nz - 1))
    planes = []
    for tpb in (0, 1, 4, 13):
        plan = gpu_lib.Plan(bank, 1 << log2n, seg, nharm_max=1, median_window=512, interbin=interbin,
                            templates_per_block=tpb)
        plane = torch.full((nz, plan.plane_columns), -1.0, device="cuda")
        plan.search(x, plane=plane)
        torch.cuda.synchronize()
        planes.append(plane.cpu().numpy())
        plan.close()
    assert planes[0].min() >= 0.0
    for p in planes[1:]:
        assert np.array_equal(planes[0], p)
    bank.close()


@pytest.mark.parametrize("log2n,nalpha", [(12, 16), (12, 33), (20, 17), (22, 6), (24, 3)])
def test_time_domain_trials_together(gpu_lib, log2n, nalpha):
    # the middle trial and the first and last ones, alone (alpha 0 as a plan of
    # one trial, the others as a plan of three) and among the others
    import torch
    n, amax = 1 << log2n, 0.02
    x = _dev(np.random.default_rng(nalpha).standard_normal(n).astype(np.float32))

    def rows(count):
        plan = gpu_lib.TdPlan(n, amax if count > 1 else 0.0, count, nharm_max=1, sigma=7.0)
        plane = torch.empty((count, n // 2), device="cuda")
        plan.search(x, plane=plane)
        torch.cuda.synchronize()
        plan.close()
        return plane

    many, three = rows(nalpha), rows(3)
    assert torch.equal(many[0], three[0]) and torch.equal(many[-1], three[2])
    if nalpha % 2:
        assert torch.equal(many[nalpha // 2], rows(1)[0])
