"""De-dispersion at the edges of its kernels' tiles (spans of 256, 1024
and 1280 samples, groups of 4 and blocks of 64 channels, 4 DM trials per workgroup
directly and 16 staged), bit-exact against the oracle: integer sums, so there is no tolerance."""
import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nchan,ndm,nout", [
    (1, 1, 1), (3, 2, 255), (4, 1, 256), (5, 3, 257), (17, 1, 1023), (64, 4, 1024), (65, 5, 1025), (257, 2, 3001),
    (15, 7, 40000),                   # one trial per workgroup, its channels split over the waves
    (6, 5, (1 << 20) + 5),            # one trial per wave, ragged last span, last workgroup with idle waves
    (67, 4, (1 << 20) + 1023),
])
def test_dedisperse_tile_edges(gpu_lib, nchan, ndm, nout):
    import torch
    f_top, foff, tsamp = 1450.0, 300.0 / nchan, 2.56e-4
    dms = np.linspace(0.0, 150.0, ndm)[::-1].copy()
    d = O.dm_delays(nchan, f_top, foff, tsamp, dms)
    rng = np.random.default_rng(nchan + nout)
    # every byte value, the ends of the range most often; one sample more than needed
    # would be read if a span ran past its end, so the filterbank ends exactly at the last one
    fil = rng.choice(np.array([0, 127, 128, 255] * 16 + list(range(256)), dtype=np.uint8), (nchan, nout + int(d.max())))
    got = gpu_lib.dedisperse(torch.from_numpy(fil).cuda(), f_top, foff, tsamp, dms, nout).cpu().numpy()
    want = np.zeros((ndm, nout))
    for i in range(ndm):
        for c in range(nchan):
            want[i] += fil[c, d[i, c]:d[i, c] + nout]
    assert np.array_equal(got.astype(np.float64), want)


@pytest.mark.parametrize("nchan,ndm,nout,dm_max", [
    (1, 16, 1 << 19, 0.0),            # one channel, no spread
    (19, 17, (1 << 19) + 77, 30.0),   # a stage of 16 channels and 3; 16 trials and 1
    (33, 40, 200000, 300.0),          # rows near their largest
    (16, 300, 30011, 900.0),          # two launches of trials, the second of 44
    (22, 16, 205 * 1280, 234.0),      # whole spans, the longest rows
    (14, 16, 205 * 1280 - 1279, 20.0),
])
def test_dedisperse_staged_rows(gpu_lib, nchan, ndm, nout, dm_max):
    import torch
    f_top, foff, tsamp = 1450.0, 300.0 / nchan, 2.56e-4
    dms = np.linspace(0.0, dm_max, ndm)
    dms[2:9] = dms[2:9][::-1].copy()  # in no order within a group
    d = O.dm_delays(nchan, f_top, foff, tsamp, dms)
    rng = np.random.default_rng(nchan + nout)
    fil = rng.integers(0, 256, (nchan, nout + int(d.max())), dtype=np.uint8)  # ends at the last sample needed
    got = gpu_lib.dedisperse(torch.from_numpy(fil).cuda(), f_top, foff, tsamp, dms, nout).cpu().numpy()
    for i in range(ndm):
        want = np.zeros(nout, dtype=np.int64)
        for c in range(nchan):
            want += fil[c, d[i, c]:d[i, c] + nout]
        assert np.array_equal(got[i].astype(np.int64), want), i
