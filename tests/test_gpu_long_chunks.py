"""A chunk whose particle orders (tiles x runs) outnumber one launch's workgroups:
256 electrons x 16416 steps x 66049 cells, an order per tile and run, 4.2e6 of them in
two launches, against the oracle on sampled cells.
"""
import numpy as np
import pytest

import oracle
from paper_2302_14812_amd import workloads as W

pytestmark = pytest.mark.gpu

from parity import TOLS, check_parity  # noqa: E402


def test_orders_in_several_launches():
    import torch

    import paper_2302_14812_amd as radio
    wl = W.undulator_workload(n_particles=256, n_steps=16416, n_side=257, n_t=256)
    tile, _, run = radio.SHAPES[0]
    assert -(-wl.detector.n_cells // tile) * -(-wl.chunk.n_steps // run) > 2**22
    cur = radio.get_tuning()
    try:
        radio.set_tuning(order_budget_mib=8192, shape=0)
        det = radio.Detector.from_spec(wl.detector, precision="mixed")
        det.deposit(radio.Chunk.from_numpy(wl.chunk))
        E, B = det.read()
        torch.cuda.synchronize()
    finally:
        radio.set_tuning(**cur)
    assert det.stats()["slices"] == 1
    at = np.linspace(0, wl.detector.n_cells - 1, 7).astype(int)
    Eg, Bg = E[at].cpu().numpy(), B[at].cpu().numpy()
    det.close()
    Eo, Bo = oracle.read(oracle.deposit_workload(wl.detector, wl.chunk, cell_index=at))
    check_parity(Eg, Bg, Eo, Bo, TOLS["mixed"], "orders in several launches")
