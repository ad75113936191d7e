"""The device's dispersion delays, compiled for the host: the form without
divisions gives the delay of the rounded operations for every accepted input.

The host builds fuse multiply-adds where the source lets them, as the device
build does, and start from a reciprocal cut to 24 bits.  Without inlining the
compiler cannot merge the two forms' operations, so that each shows its own.
"""
import ctypes
import os
import subprocess

import numpy as np
import pytest

import oracle as O
import paper_1511_07343_amd.build as build

SOURCE = """
#include "delays.hpp"
extern "C" void delays(double f_top, double foff, double tsamp, int n, const double *kdm, const int *c, int *fast,
                       int *exact) {
    fdas::Dispersion p{};
    p.f_top = f_top;
    p.foff = foff;
    p.inv_top2 = 1.0 / (f_top * f_top);
    p.tsamp = tsamp;
    p.inv_tsamp = 1.0 / tsamp;
    for (int i = 0; i < n; ++i) {
        fast[i] = fdas::delay_fast(p, kdm[i], c[i]);
        exact[i] = fdas::delay_of(p, kdm[i], c[i]);
    }
}
"""


@pytest.fixture(scope="module", params=[[], ["-fno-inline"]], ids=["inline", "separate"])
def delays(request, tmp_path_factory):
    d = tmp_path_factory.mktemp("delays")
    src, lib = d / "delays.cpp", d / "delays.so"
    src.write_text(SOURCE)
    subprocess.run([build.HIPCC, "-x", "hip", "--offload-host-only", "-O2", "-std=c++17", "-fPIC", "-shared", "-mfma",
                    "-ffp-contract=fast-honor-pragmas", *request.param, "-I", build.CSRC, str(src), "-o", str(lib)],
                   check=True, capture_output=True)
    fn = ctypes.CDLL(os.fspath(lib)).delays
    fn.argtypes = [ctypes.c_double] * 3 + [ctypes.c_int] + [ctypes.c_void_p] * 4

    def run(f_top, foff, tsamp, kdm, c):
        kdm, c = np.ascontiguousarray(kdm, dtype=np.float64), np.ascontiguousarray(c, dtype=np.int32)
        fast, exact = np.empty(len(kdm), dtype=np.int32), np.empty(len(kdm), dtype=np.int32)
        fn(f_top, foff, tsamp, len(kdm), kdm.ctypes.data, c.ctypes.data, fast.ctypes.data, exact.ctypes.data)
        return fast, exact
    return run


@pytest.mark.parametrize("f_top,ratio", [(1500.0, 1.25), (1450.0, 16.0), (800.0, 128.0), (1500.0, 512.0), (1711.3, 4096.0)])
def test_fast_delay_at_rounding_boundaries(delays, f_top, ratio):
    """Products k DM whose delay lies within a few roundings of a half, where
    the form without divisions must not decide by itself."""
    nchan, tsamp = 1021, 64e-6
    foff = f_top * (1.0 - 1.0 / ratio) / (nchan - 1)
    rng = np.random.default_rng(int(ratio))
    c = rng.integers(nchan // 2, nchan, 20000)
    f = f_top - foff * c
    kdm = (rng.integers(1, 200000, len(c)) + 0.5) * tsamp / (1.0 / (f * f) - 1.0 / (f_top * f_top))
    kdm *= 1.0 + 2.0 ** -52 * rng.integers(-6, 7, len(c))
    fast, exact = delays(f_top, foff, tsamp, kdm, c)
    assert np.array_equal(fast, exact)
    for i in range(0, len(c), 200):  # the oracle's delays too (DM 1 of the scaled constant)
        want = np.floor(kdm[i] * (1.0 / (f[i] * f[i]) - 1.0 / (f_top * f_top)) / tsamp + 0.5)
        assert exact[i] == want


def test_delays_match_the_oracle(delays):
    nchan, f_top, foff, tsamp = 257, 1450.0, 1.17, 2.56e-4
    dms = [0.0, 1.0, 55.5, 300.0]
    want = O.dm_delays(nchan, f_top, foff, tsamp, dms)
    for i, dm in enumerate(dms):
        fast, exact = delays(f_top, foff, tsamp, np.full(nchan, 4.148808e3 * dm), np.arange(nchan))
        assert np.array_equal(fast, want[i]) and np.array_equal(exact, want[i])


@pytest.mark.parametrize("f_top,foff,tsamp,dms,nchan", [
    (1500.0, 0.0, 1e-310, [0.0, 10.0, 3e5], 8),    # 1 / tsamp overflows; every channel at f_top, every delay 0
    (1500.0, 0.0, 1e-300, [1.0, 1e9], 8),          # k DM / tsamp overflows
    (1500.0, 10.0, 1e-310, [0.0], 8),
    (1e160, 0.0, 1e-3, [0.0, 50.0], 3),            # f^2 overflows
    (1e160, 1e157, 1e-3, [0.0, 50.0], 3),
    (1e-152, 0.0, 1e-3, [0.0, 50.0], 3),           # f^2 has no finite square of its reciprocal
    (9.9e153, 0.0, 1e-300, [1e3], 3),              # 1 / f^2 is subnormal
    (1500.0, 10.0, float("inf"), [0.0, 50.0], 8),
])
def test_delays_at_the_ends_of_the_range(delays, f_top, foff, tsamp, dms, nchan):
    """Accepted inputs (every delay 0) where a factor overflows or vanishes."""
    c = np.arange(nchan)
    for dm in dms:
        fast, exact = delays(f_top, foff, tsamp, np.full(nchan, 4.148808e3 * dm), c)
        assert np.all(exact == 0)
        assert np.array_equal(fast, exact)
