"""The time-domain search's sample positions, compiled for the host, against
the quadratic's root in higher precision."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

import paper_1511_07343_amd.build as build

SOURCE = """
#include "resample.hpp"
extern "C" void positions(double alpha, long n, double *s) {
    const fdas::DriftPositions p{0.5 * alpha, 1.0 / double(n)};
    for (long i = 0; i < n / 2; ++i) {
        double v, w;
        p.pair(i, v, w);
        s[2 * i] = v;
        s[2 * i + 1] = w;
    }
}
"""


@pytest.fixture(scope="module")
def positions(tmp_path_factory):
    d = tmp_path_factory.mktemp("positions")
    src, lib = d / "positions.cpp", d / "positions.so"
    src.write_text(SOURCE)
    subprocess.run([build.HIPCC, "-x", "hip", "--offload-host-only", "-O2", "-std=c++17", "-fPIC", "-shared", "-mfma",
                    "-ffp-contract=fast-honor-pragmas", "-I", build.CSRC, str(src), "-o", str(lib)],
                   check=True, capture_output=True)
    fn = ctypes.CDLL(os.fspath(lib)).positions
    fn.argtypes = [ctypes.c_double, ctypes.c_long, ctypes.c_void_p]

    def run(alpha, n):
        out = np.empty(n)
        fn(alpha, n, out.ctypes.data)
        return out
    return run


@pytest.mark.parametrize("log2n", [10, 11, 13, 16, 20])
@pytest.mark.parametrize("alpha", [0.0, 1e-9, 0.02, -0.02, 0.25, -0.25, 0.5, -0.5])
def test_positions_to_a_few_roundings(positions, log2n, alpha):
    n = 1 << log2n
    got = positions(alpha, n)
    tau = np.arange(n, dtype=np.longdouble) / n - np.longdouble(0.5)
    want = 2 * tau / (1 + np.sqrt(1 + 2 * np.longdouble(alpha) * tau))
    assert np.finfo(np.longdouble).nmant >= 63
    # v is at most 0.6 in magnitude: a rounding is 1.1e-16; the residual, formed
    # from terms of that size and divided by a slope of 0.7 or more, a few
    assert np.abs(got - want).max() < 5e-16
