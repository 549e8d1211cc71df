"""Weak slots beside strong ones: a slot's sum holds what its own segments deposit,
however strong the field was in the slots next to it.

A sheet whose segments cross a slot or more each, seen by cells close together, with
one electron of 1e16 times the others' charge in the middle of the arrivals.  The
slots that this electron never reaches are compared with the oracle by themselves.
Bar: the precision's parity bar times the cell's largest weak slot (a sum that had
passed through the strong slots in double would be off by about 1e16 * 2^-53, a
whole weak field).
"""
import dataclasses
import math

import numpy as np
import pytest

import oracle
from paper_2302_14812_amd import workloads as W

pytestmark = pytest.mark.gpu

from parity import TOLS  # noqa: E402

STRONG = 1.0e16
HOLD_PREVIOUS, HOLD_LINEAR = 4, 8


def _only(chunk, keep):
    return dataclasses.replace(chunk, x=np.ascontiguousarray(chunk.x[:, :, keep]),
                               u=np.ascontiguousarray(chunk.u[:, :, keep]),
                               q=np.ascontiguousarray(chunk.q[keep]))


def _sheet(n_steps, n_p=4000):
    wl = W.plasma_mirror_workload(n_particles=n_p, n_steps=n_steps, n_side=2, n_t=1024)
    inc = math.pi / 4
    cells = W.sphere_cap_cells(1.0e5, [-math.cos(inc), math.sin(inc), 0.0],
                               [math.sin(inc), math.cos(inc), 0.0], 3, 3, 1e-3, 1e-3)
    spec = W.DetectorSpec(cells=cells, t0=wl.detector.t0, dt_det=wl.detector.dt_det, n_t=1024)
    # the electron in the middle of the sheet as the cells see it
    far = np.linalg.norm(cells.mean(axis=0)[:, None] - wl.chunk.x[:, 0], axis=0)
    strong = int(np.argsort(far)[n_p // 2])
    q = np.full(n_p, -1.0)
    q[strong] = -STRONG
    return spec, dataclasses.replace(wl.chunk, q=q), strong


@pytest.mark.parametrize("options", [0, HOLD_PREVIOUS, HOLD_LINEAR])
@pytest.mark.parametrize("n_steps", [250, 60])
@pytest.mark.parametrize("precision", ["fp64", "mixed", "mixed_twosum"])
def test_weak_slots(precision, n_steps, options):
    import torch

    import paper_2302_14812_amd as radio
    spec, chunk, strong = _sheet(n_steps)
    read = lambda c: oracle.read(oracle.deposit_workload(spec, c, options=options))  # noqa: E731
    Es, Bs = read(_only(chunk, [strong]))
    Eo, Bo = read(_only(chunk, [p for p in range(chunk.n_particles) if p != strong]))
    det = radio.Detector.from_spec(spec, precision=precision, options=options)
    det.deposit(radio.Chunk.from_numpy(chunk))
    E, B = det.read()
    torch.cuda.synchronize()
    Eg, Bg = E.cpu().numpy(), B.cpu().numpy()
    st = det.stats()
    det.close()
    assert st["large_ring"] > 0
    weak = (Es == 0.0).all(axis=2) & (Bs == 0.0).all(axis=2) & (Eo != 0.0).any(axis=2)
    assert weak.sum() > 0.2 * weak.size
    for got, ref in ((Eg, Eo), (Bg, Bo)):
        largest = np.where(weak[..., None], np.abs(ref), 0.0).max(axis=(1, 2))
        off = np.where(weak[..., None], np.abs(got - ref), 0.0).max(axis=(1, 2))
        print(f"[weak] {precision} {n_steps} {options}: {float((off / largest).max()):.2e}",
              flush=True)
        assert (off <= TOLS[precision] * largest).all()
