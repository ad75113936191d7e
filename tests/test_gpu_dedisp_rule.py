"""De-dispersion on both sides of the line between the staged and the direct
forms (spans of 1280 samples times trials), bit-exact against the sums."""
import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ndm,spans", [(16, 128), (16, 127), (10, 205), (10, 204), (33, 63), (33, 62), (8, 400), (8, 399),
                                       (17, 189), (17, 188), (7, 1000), (7, 999), (6, 1200)])
@pytest.mark.parametrize("short", [0, 1279])
def test_dedisperse_on_both_sides(gpu_lib, ndm, spans, short):
    import torch
    nchan, f_top, foff, tsamp = 18, 1450.0, 300.0 / 18, 2.56e-4
    nout = 1280 * spans - short
    dms = np.linspace(3.0, 3.0 + 2.0 * ndm, ndm)
    d = O.dm_delays(nchan, f_top, foff, tsamp, dms)
    g = torch.Generator(device="cuda").manual_seed(ndm + spans)
    fil = torch.randint(0, 256, (nchan, nout + int(d.max())), dtype=torch.uint8, device="cuda", generator=g)
    got = gpu_lib.dedisperse(fil, f_top, foff, tsamp, dms, nout)
    for i in range(ndm):
        want = torch.zeros(nout, dtype=torch.int32, device="cuda")
        for c in range(nchan):
            want += fil[c, int(d[i, c]):int(d[i, c]) + nout]
        assert torch.equal(got[i], want.float()), i
