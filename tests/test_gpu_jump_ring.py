"""The large slot ring where a segment crosses several slots, with runs staged in
shorter stretches the more slots they span.

The plasma-mirror sheet over ten periods in ever fewer steps crosses ~1.6 (250
steps) to ~34 (12 steps) of 1024 slots a segment, from a whole run per stretch to
one segment, and beyond what the ring holds at all.  Bars: the parity bars; slots
no segment reaches read exactly zero.
"""
import numpy as np
import pytest

import oracle
from paper_2302_14812_amd import workloads as W

pytestmark = pytest.mark.gpu

from parity import TOLS, check_parity  # noqa: E402

HOLD_PREVIOUS, HOLD_LINEAR, FAR_FIELD = 4, 8, 1
_CACHE = {}


def _case(n_steps, options):
    if (n_steps, options) not in _CACHE:
        wl = W.plasma_mirror_workload(n_particles=150, n_steps=n_steps, n_side=9, n_t=1024)
        spec = wl.detector
        # a window that starts inside the arrivals and ends after them
        spec.t0 += 0.2 * spec.n_t * spec.dt_det
        cnt = np.zeros(2, dtype=np.int64)
        D = oracle.deposit_workload(spec, wl.chunk, options=options, counters=cnt)
        _CACHE[(n_steps, options)] = (spec, wl.chunk) + oracle.read(D) + (cnt,)
    return _CACHE[(n_steps, options)]


@pytest.mark.parametrize("options", [0, HOLD_PREVIOUS, HOLD_LINEAR, FAR_FIELD])
@pytest.mark.parametrize("n_steps", [250, 125, 60, 30, 12])
@pytest.mark.parametrize("precision", ["fp64", "mixed", "mixed_twosum"])
def test_sparse_arrivals(precision, n_steps, options):
    import torch

    import paper_2302_14812_amd as radio
    spec, chunk, Eo, Bo, cnt = _case(n_steps, options)
    det = radio.Detector.from_spec(spec, precision=precision, options=options)
    det.deposit(radio.Chunk.from_numpy(chunk))
    E, B = det.read()
    torch.cuda.synchronize()
    st = det.stats()
    Eg, Bg = E.cpu().numpy(), B.cpu().numpy()
    det.close()
    assert st["large_ring"] > 0.5 * st["interactions"]
    assert (st["clipped"], st["nonmonotone"]) == (cnt[0], cnt[1])
    check_parity(Eg, Bg, Eo, Bo, TOLS[precision], f"sparse {precision} {n_steps} {options}")
    empty = (Eo == 0.0).all(axis=2) & (Bo == 0.0).all(axis=2)
    assert empty.any() and (Eg[empty] == 0.0).all() and (Bg[empty] == 0.0).all()
