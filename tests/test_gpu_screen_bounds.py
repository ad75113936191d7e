"""How many cells the harmonic-sum screen passes on: those of the 2-bin blocks
whose codes (powers in units of 1/250 of the last threshold, rounded up) add up
to a threshold, no more."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

TERMS = [[16], [8], [4, 12], [2, 6, 10, 14], [1, 3, 5, 7, 9, 11, 13, 15]]  # added at each level


def _flagged_cells(code, izc, code_thr):
    nz, nblk = code.shape
    d = np.arange(nz) - izc
    b = np.arange(nblk, dtype=np.int64)
    total = np.zeros((nz, nblk), dtype=np.int64)
    flagged = np.zeros((nz, nblk), dtype=bool)
    for level, thr in enumerate(code_thr):
        for j in TERMS[level]:
            rows = izc + np.sign(d) * ((np.abs(d) * j + 8) >> 4)
            lo, hi = ((2 * b * j + 8) >> 4) >> 1, (((2 * b + 1) * j + 8) >> 4) >> 1
            total += np.maximum(code[np.ix_(rows, lo)], code[np.ix_(rows, hi)])
        flagged |= total >= thr
    return 2 * int(flagged.sum())


@pytest.mark.parametrize("corr", ["fft", "bf16"])
@pytest.mark.parametrize("log2n,nz,nharm,sigma", [(14, 21, 1, 2.0), (15, 21, 2, 2.5), (15, 21, 4, 3.0), (16, 21, 16, 3.0)])
def test_screen_passes_on_no_more(gpu_lib, log2n, nz, nharm, sigma, corr):
    import torch
    n = 1 << log2n
    x = torch.randn(n, device="cuda", generator=torch.Generator(device="cuda").manual_seed(log2n))
    bank = gpu_lib.make_templates(10.0, 20.0 / (nz - 1))
    plan = gpu_lib.Plan(bank, n, 256, nharm_max=nharm, sigma=sigma, median_window=256, correlator=corr)
    plane = torch.empty((nz, n // 2), device="cuda")
    plan.search(x, plane=plane, cap=1 << 20)
    torch.cuda.synchronize()
    cells = plan.search_counts()[1]
    P = plane.cpu().numpy()
    thr = [np.float32(gpu_lib.threshold(sigma, 1 << l)) for l in range(nharm.bit_length())]
    inv = np.float32(250.0 / np.float64(thr[-1]))
    code_thr = [int(np.floor(np.float64(t) * np.float64(inv) * (1.0 - 1e-5))) for t in thr]
    u = P.astype(np.float64).reshape(nz, -1, 2).max(axis=2) * np.float64(inv)
    # a product within a rounding of a whole number may take either code
    low = _flagged_cells(np.minimum(np.ceil(u * (1.0 - 1e-6)), 255).astype(np.int64), (nz - 1) // 2, code_thr)
    high = _flagged_cells(np.minimum(np.ceil(u * (1.0 + 1e-6) + 1e-6), 255).astype(np.int64), (nz - 1) // 2, code_thr)
    print(low, cells, high)
    assert 0 < low <= cells <= high
    plan.close()
    bank.close()
