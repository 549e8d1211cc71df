"""The large slot ring's unusual inputs: states that are not finite, segments that run
backward, windows of about the ring's span, and runs staged in stretches in a batch.

A sheet whose segments cross several slots, seen by cells close together.  Bars: the
parity bars; a particle with a state that is not finite leaves its mark on its own
slots alone.
"""
import dataclasses

import numpy as np
import pytest

import oracle
from paper_2302_14812_amd import workloads as W
from test_gpu_weak_slots import _only, _sheet

pytestmark = pytest.mark.gpu

from parity import TOLS, check_parity  # noqa: E402

PRECISIONS = pytest.mark.parametrize("precision", ["fp64", "mixed", "mixed_twosum"])
HOLD_PREVIOUS, HOLD_LINEAR = 4, 8


def _plain(n_steps, n_p=600):
    spec, chunk, _ = _sheet(n_steps, n_p)
    return spec, dataclasses.replace(chunk, q=np.full(n_p, -1.0))


def _deposit(spec, chunk, precision, options=0):
    import torch

    import paper_2302_14812_amd as radio
    det = radio.Detector.from_spec(spec, precision=precision, options=options)
    det.deposit(radio.Chunk.from_numpy(chunk))
    E, B = det.read()
    torch.cuda.synchronize()
    st = det.stats()
    out = E.cpu().numpy(), B.cpu().numpy()
    det.close()
    assert st["large_ring"] > 0
    return out + (st,)


@PRECISIONS
@pytest.mark.parametrize("options", [0, HOLD_PREVIOUS, HOLD_LINEAR])
@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_state_that_is_not_finite(precision, options, bad):
    spec, chunk = _plain(60)
    p, k = 311, 25
    u = chunk.u.copy()
    u[0, k, p] = bad
    broken = dataclasses.replace(chunk, u=u)
    Eg, Bg, _ = _deposit(spec, broken, precision, options)
    read = lambda c: oracle.read(oracle.deposit_workload(spec, c, options=options))  # noqa: E731
    Eo, Bo = read(chunk)
    # the slots that the particle reaches with the segments about that state
    own = dataclasses.replace(_only(chunk, [p]), x=np.ascontiguousarray(chunk.x[:, k - 2:k + 3, [p]]),
                              u=np.ascontiguousarray(chunk.u[:, k - 2:k + 3, [p]]),
                              first_step=chunk.first_step + k - 2)
    Es, Bs = read(own)
    touched = (Es != 0.0).any(axis=2) | (Bs != 0.0).any(axis=2)
    touched |= np.roll(touched, 1, axis=1) | np.roll(touched, -1, axis=1)  # slots it only grazes
    assert touched.any() and not touched.all()
    for got, ref in ((Eg, Eo), (Bg, Bo)):
        assert np.isfinite(got[~touched]).all()
        ref, got = ref.copy(), got.copy()
        ref[touched] = got[touched] = 0.0
        off = np.abs(got - ref).max(axis=(1, 2))
        assert (off <= TOLS[precision] * np.abs(ref).max(axis=(1, 2))).all()


@PRECISIONS
@pytest.mark.parametrize("options", [0, HOLD_PREVIOUS, HOLD_LINEAR])
@pytest.mark.parametrize("n_steps", [250, 60, 12])
def test_backward_segments(precision, options, n_steps):
    spec, chunk = _plain(n_steps)
    x = chunk.x.copy()
    # every fifth particle is moved away for a third of its states (jumps that light
    # cannot make, there and back)
    x[0, n_steps // 3:2 * n_steps // 3, ::5] += 4.0
    chunk = dataclasses.replace(chunk, x=x)
    Eg, Bg, st = _deposit(spec, chunk, precision, options)
    cnt = np.zeros(2, dtype=np.int64)
    Eo, Bo = oracle.read(oracle.deposit_workload(spec, chunk, options=options, counters=cnt))
    assert cnt[1] > 0 and (st["clipped"], st["nonmonotone"]) == (cnt[0], cnt[1])
    check_parity(Eg, Bg, Eo, Bo, TOLS[precision], f"backward {precision} {options} {n_steps}")


@PRECISIONS
@pytest.mark.parametrize("n_t", [1, 17, 63, 64, 65, 130])
def test_window_of_about_the_ring(precision, n_t):
    spec, chunk = _plain(120)
    # a window of n_t slots inside the arrivals, clipped at both ends
    spec = W.DetectorSpec(cells=spec.cells, t0=spec.t0 + 500.3 * spec.dt_det, dt_det=spec.dt_det,
                          n_t=n_t)
    import torch

    import paper_2302_14812_amd as radio
    det = radio.Detector.from_spec(spec, precision=precision)
    det.deposit(radio.Chunk.from_numpy(chunk))
    E, B = det.read()
    torch.cuda.synchronize()
    st = det.stats()
    Eg, Bg = E.cpu().numpy(), B.cpu().numpy()
    det.close()
    cnt = np.zeros(2, dtype=np.int64)
    Eo, Bo = oracle.read(oracle.deposit_workload(spec, chunk, counters=cnt))
    assert (st["clipped"], st["nonmonotone"]) == (cnt[0], cnt[1])
    check_parity(Eg, Bg, Eo, Bo, TOLS[precision], f"window of {n_t} {precision}")


@PRECISIONS
def test_stretches_in_a_batch(precision):
    import torch

    import paper_2302_14812_amd as radio
    cases = [_plain(n) for n in (250, 120, 60, 30, 12)]  # from whole runs to single segments
    dets = [radio.Detector.from_spec(s, precision=precision) for s, _ in cases]
    radio.deposit_batch(dets, [radio.Chunk.from_numpy(c) for _, c in cases])
    torch.cuda.synchronize()
    for det, (spec, chunk) in zip(dets, cases):
        E, B = det.read()
        torch.cuda.synchronize()
        Eo, Bo = oracle.read(oracle.deposit_workload(spec, chunk))
        assert det.stats()["large_ring"] == det.stats()["interactions"]
        check_parity(E.cpu().numpy(), B.cpu().numpy(), Eo, Bo, TOLS[precision],
                     f"stretches in a batch {precision} {chunk.n_steps}")
        det.close()
