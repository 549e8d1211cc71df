"""The particle order of a tile at the sizes where its kernel changes form.

Up to 2048 particles a thread keeps its keys in registers; beyond that the keys
are computed per pass.  The histogram covers only the bins the particles'
spread needs, in rounds of 1024.  An order that lost or repeated a particle
would show as a parity error of the double deposit, whose bars are used.
"""
import numpy as np
import pytest

import oracle
from paper_2302_14812_amd import workloads as W

pytestmark = pytest.mark.gpu

from parity import TOL_FP64, check_parity  # noqa: E402


@pytest.mark.parametrize("n_p", [1, 2, 255, 256, 257, 2047, 2048, 2049, 3000])
@pytest.mark.parametrize("spread,n_t", [(1e-3, 64), (3.0, 1500), (3.0, 20000)])
def test_order_holds_every_particle_once(n_p, spread, n_t):
    import torch

    import paper_2302_14812_amd as radio
    chunk = W.random_chunk(n_p, 4, seed=W.BASE_SEED + n_p, spread=spread)
    cells = W.sphere_cap_cells(50.0, [0, 0, 1], [1, 0, 0], 3, 3, 0.3, 0.3)
    t0, dtd = W.arrival_window(cells, chunk, n_t, max_particles=n_p)
    spec = W.DetectorSpec(cells=cells, t0=t0, dt_det=dtd, n_t=n_t)
    det = radio.Detector.from_spec(spec)
    det.deposit(radio.Chunk.from_numpy(chunk))
    E, B = det.read()
    torch.cuda.synchronize()
    Eg, Bg = E.cpu().numpy(), B.cpu().numpy()
    det.close()
    Eo, Bo = oracle.read(oracle.deposit_workload(spec, chunk))
    assert np.isfinite(Eo).all()
    check_parity(Eg, Bg, Eo, Bo, TOL_FP64, f"order n_p={n_p} spread={spread} n_t={n_t}")
