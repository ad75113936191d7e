"""De-dispersion of wide bands and at the ends of the accepted range, in every
form of the kernel, bit-exact against the rounded delays."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _delays(nchan, f_top, foff, tsamp, dms):
    f = f_top - foff * np.arange(nchan)
    with np.errstate(over="ignore"):
        raw = 4.148808e3 * np.asarray(dms)[:, None] * (1.0 / (f * f) - 1.0 / (f_top * f_top))[None, :] / tsamp
    return np.floor(raw + 0.5).astype(np.int64)


@pytest.mark.parametrize("f_top,foff,tsamp,nchan,dms,nout", [
    (1500.0, 1490.0 / 64, 1e-3, 65, np.linspace(0.0, 2.0, 5), 3001),        # a band of 150 to 1, split channels
    (1500.0, 1490.0 / 32, 1e-3, 33, np.linspace(0.0, 0.04, 32), 1 << 17),    # staged
    (1500.0, 1490.0 / 32, 1e-3, 33, np.linspace(0.0, 0.2, 5), (1 << 20) + 7),  # a wave per trial
    (1500.0, 1490.0 / 16, 1e-3, 17, np.linspace(0.0, 0.2, 5), 200),         # short
    (1500.0, 0.0, 1e-310, 9, np.array([0.0, 10.0, 3e5]), 3001),             # 1 / tsamp overflows, every delay is 0
    (1500.0, 0.0, 1e-310, 9, np.linspace(0.0, 1e5, 32), 1 << 17),
    (1e160, 1e157, 1e-3, 9, np.array([0.0, 10.0]), 3001),                   # f^2 overflows
    (9.9e153, 0.0, 1e-300, 9, np.array([1e3]), 3001),                       # 1 / f^2 is subnormal
])
def test_dedisperse_delay_range(gpu_lib, f_top, foff, tsamp, nchan, dms, nout):
    import torch
    d = _delays(nchan, f_top, foff, tsamp, dms)
    assert d.min() == 0
    rng = np.random.default_rng(nchan + nout)
    fil = rng.integers(0, 256, (nchan, nout + int(d.max())), dtype=np.uint8)  # ends at the last sample needed
    got = gpu_lib.dedisperse(torch.from_numpy(fil).cuda(), f_top, foff, tsamp, dms, nout).cpu().numpy()
    for i in range(len(dms)):
        want = np.zeros(nout, dtype=np.int64)
        for c in range(nchan):
            want += fil[c, d[i, c]:d[i, c] + nout]
        assert np.array_equal(got[i].astype(np.int64), want), i
