"""De-dispersion of more work items than one launch takes (2^32 threads)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_dedisperse_beyond_one_launch(gpu_lib):
    import torch
    nchan, ndm, f_top, foff, tsamp = 64, 15, 1450.0, 300.0 / 64, 2.56e-4
    nout = (1 << 32) // ndm + 300001  # spans of 256 samples a trial, 256 threads each
    assert nout * ndm > 1 << 32
    if torch.cuda.mem_get_info()[0] < 48 << 30:
        pytest.skip("needs 48 GB of free GPU memory")
    dms = np.linspace(0.0, 900.0, ndm)  # too far apart for the staged form
    f = f_top - foff * np.arange(nchan)
    d = np.floor(4.148808e3 * dms[:, None] * (f ** -2.0 - f_top ** -2.0) / tsamp + 0.5).astype(np.int64)
    g = torch.Generator(device="cuda").manual_seed(5)
    fil = torch.randint(0, 256, (nchan, nout + int(d.max())), dtype=torch.uint8, device="cuda", generator=g)
    got = gpu_lib.dedisperse(fil, f_top, foff, tsamp, dms, nout)
    for i in (0, 7, 14):
        for t in (0, nout // 3, nout // 2, nout - 70000, nout - 5000):
            n = min(5000, nout - t)
            want = torch.zeros(n, dtype=torch.int64, device="cuda")
            for c in range(nchan):
                want += fil[c, t + int(d[i, c]):t + int(d[i, c]) + n]
            assert torch.equal(got[i, t:t + n].long(), want), (i, t)
    del fil, got
    torch.cuda.empty_cache()
