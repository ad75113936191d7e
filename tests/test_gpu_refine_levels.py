"""The two forms of the refinement, one launch per level (up to 2048 records)
and one workgroup per record (above), give the same records bit for bit; and
the interpolated power over small and zero drifts, where the response's forms
meet, agrees with a quadrature of the response's defining integral."""
import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu


def _plan(lib, zmax, nz, seg, log2n=16):
    import torch
    bank = lib.make_templates(zmax, 2 * zmax / (nz - 1))
    plan = lib.Plan(bank, 1 << log2n, seg, nharm_max=16, sigma=9.0, median_window=512)
    rng = np.random.default_rng(nz)
    X = (rng.standard_normal(1 << (log2n - 1)) + 1j * rng.standard_normal(1 << (log2n - 1))).astype(np.complex64)
    X[0] = 0
    plan.search(torch.from_numpy(X).cuda(), kind=lib.IN_SPECTRUM)
    return bank, plan, X


def _power(Xh, r, z, h):
    """P(r, z) with A(q, z) = int_0^1 exp(2 pi i [(q - z/2) u + z u^2 / 2]) du by
    Gauss-Legendre quadrature (200 nodes: exact far past 30 cycles)."""
    u, w = np.polynomial.legendre.leggauss(200)
    u, w = (u + 1) / 2, w / 2
    k = np.arange(int(np.ceil(r - h)), int(np.floor(r + h)) + 1)
    a = np.exp(2j * np.pi * ((r - k)[:, None] * u - z / 2 * u + z * u * u / 2)) @ w
    inside = (k >= 0) & (k < len(Xh))
    return abs(np.sum(Xh[k[inside]] * a[inside].conj())) ** 2 / np.sum(np.abs(a) ** 2)


@pytest.mark.parametrize("zmax,nz,seg,levels", [(2.0, 5, 256, 3), (40.0, 41, 256, 6), (200.0, 201, 2048, 1)])
def test_forms_agree_bit_for_bit(gpu_lib, zmax, nz, seg, levels):
    bank, plan, X = _plan(gpu_lib, zmax, nz, seg)
    rng = np.random.default_rng(1)
    n = 2100
    rec = np.zeros(n, dtype=gpu_lib.CAND_DTYPE)
    rec["nharm"] = rng.choice([1, 2, 4, 8, 16], n)
    rec["k"] = rng.integers(0, len(X), n)  # the spectrum's ends among them
    rec["iz"] = rng.integers(0, nz, n)     # and the drift range's
    whole = plan.refine(rec, levels)
    for part in (slice(0, 2048), slice(2048, n), slice(5, 6), slice(100, 165)):
        got = plan.refine(rec[part], levels)
        assert got.tobytes() == whole[part].tobytes()
        assert plan.refine_noalloc(rec[part], levels).tobytes() == got.tobytes()
    plan.close()
    bank.close()


def test_interpolated_power_over_small_drifts(gpu_lib):
    bank, plan, X = _plan(gpu_lib, 8.0, 9, 256, log2n=12)
    Xh = O.normalise(X.astype(np.complex128), 512)
    r, z = np.meshgrid([200.0, 200.25, 1000.5, 5.0, 2040.875], [0.0, 1e-9, -1e-3, 0.01, 0.25, -0.99, 1.0, 1.5, 1.999, 2.0,
                                                               -2.5, 4.5, 7.0, 8.0, -20.0])
    r, z = r.ravel(), z.ravel()
    got = plan.interp_power(r, z, 1)
    want = np.array([_power(Xh, ri, zi, bank.h) for ri, zi in zip(r, z)])
    # the medians of the FP32 powers, 2^-24 each, and FP64 responses
    assert np.all(np.abs(got - want) <= 4 * 2.0 ** -24 * want + 1e-10)
    plan.close()
    bank.close()
