"""Spectra of 2049 to 4096 slots, one workgroup of 1024 threads a cell at a time: more
cells than the device has workgroups for (a second cell, its slots in flight, sums over
several), fewer, padding, and each choice of outputs, against the oracle's spectrum of
the same fields.

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
@pytest.mark.parametrize("n_t,n_fft,n_c", [(2049, 0, 300), (4096, 0, 601), (4095, 0, 1),
                                           (100, 4096, 5), (3000, 0, 257)])
def test_spectrum_4096(precision, n_t, n_fft, n_c):
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
                 (False, False, True), (False, True, True), (True, False, True)):
        out = det.spectrum(n_fft=n_fft, weights=weights, d2I=want[0], dIdw=want[1], dIdO=want[2])
        torch.cuda.synchronize()
        for got, ref, asked in zip(out[1:], (d2o, dwo, dOo), want):
            assert (got is not None) == asked
            if asked:
                assert _rel(got.cpu().numpy(), ref) <= 1e-12, want
    det.close()
