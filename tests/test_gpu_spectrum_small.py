"""Spectra of up to 2048 slots, which take all cells through one kernel: every
transform length it has (one to 2048, its tiles of 64 cells down to one), numbers
of cells that leave a tile part empty or give a workgroup several tiles, padding,
and each choice of outputs, against the oracle's spectrum of the same fields.

Bar: 1e-12, the spectrum's own.
"""
import numpy as np
import pytest

import oracle
from paper_2302_14812_amd import workloads as W

pytestmark = pytest.mark.gpu


def _rel(a, b):
    return float(np.linalg.norm(a - b)) / float(np.linalg.norm(b))


@pytest.mark.parametrize("precision", ["fp64", "mixed_twosum"])
@pytest.mark.parametrize("n_t,n_fft,n_c", [
    (1, 0, 67), (2, 0, 5), (3, 0, 130), (8, 0, 64), (13, 32, 33), (40, 0, 1), (100, 0, 17),
    (256, 0, 9), (257, 0, 6), (700, 1024, 3), (1500, 0, 2), (2048, 0, 1), (2000, 0, 1100),
    (16, 0, 40000)])
def test_small_spectrum(precision, n_t, n_fft, n_c):
    import torch

    import paper_2302_14812_amd as radio
    rng = np.random.Generator(np.random.PCG64(1000 * n_t + n_c))
    cells = W.line_cells(1.0e3, n_c, 0.3)
    E = rng.normal(size=(n_c, n_t, 3))
    det = radio.Detector(cells, t0=0.0, dt_det=0.01, n_t=n_t, precision=precision)
    det.load(torch.from_numpy(E).cuda(), torch.from_numpy(E[::-1].copy()).cuda())
    held = det.read()[0].cpu().numpy()
    weights = rng.uniform(0.5, 2.0, size=n_c)
    _, d2o, dwo, dOo = oracle.spectrum(held, 0.01, cells, n_fft=n_fft or None, weights=weights)
    for want in ((True, True, True), (True, False, False), (False, True, False),
                 (False, True, True), (True, False, True)):
        out = det.spectrum(n_fft=n_fft, weights=weights, d2I=want[0], dIdw=want[1], dIdO=want[2])
        torch.cuda.synchronize()
        for got, ref, asked in zip(out[1:], (d2o, dwo, dOo), want):
            assert (got is not None) == asked
            if asked:
                assert _rel(got.cpu().numpy(), ref) <= 1e-12, want
    det.close()
