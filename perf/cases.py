"""Performance cases of the radiation deposit: what its users have it do.

A case is a dict of plain values.  listed() gives the named ones, draw(rng)
more of the same ranges; prepare(case, seed) makes what a program holds before
the call (device trajectories and detectors), run(state) is one pass through
the public entry points and returns its whole outputs, work(case) what a pass
cannot do without, exact(case, seed) the same outputs in plain 64-bit torch.

Kinds of pass:

deposit   one shot on a resident detector: reset, deposit a trajectory chunk,
          read E and B.
runtime   the same with the particles pushed on the device first (a run-time
          block of a few steps).
batch     several uneven (detector, chunk) pairs in one call, then every read.
spectrum  spectral post-processing of a resident detector.

Fields of the mixed modes carry single-precision accuracy, and a program that
keeps them stores them as float32; so these passes end with that conversion.
"""
import math

import numpy as np
import torch

import paper_2302_14812_amd as radio

FAR_FIELD, HOLD_PREVIOUS, HOLD_LINEAR = 1, 4, 8
TWO_PI = 2.0 * math.pi
FLOPS = 84.0  # of one (particle, segment, cell) interaction, on the textbook form
EXACT_MOST = 1.0e10  # interactions (times slots a segment touches) exact() takes on


# --------------------------------------------------------------------------
# the cases
# --------------------------------------------------------------------------

def listed():
    return [
        # one charge on a circular orbit before a small plane: the first thing a
        # user tries, and a parameter scan's inner call (latency, launches)
        dict(name="circular_1e", kind="deposit", source="circular", precision="fp64", options=0,
             n_p=1, n_s=2000, n1=32, n2=32, n_t=512),
        # the paper's spectral benchmark: one electron, a long sinusoidal orbit, a
        # line of cells with many slots
        dict(name="sinusoidal_1e", kind="deposit", source="sinusoidal", precision="fp64",
             options=0, n_p=1, n_s=25133, n1=256, n2=1, n_t=65536),
        # undulator ensemble (many segments a slot), the framework's own benchmark in
        # fewer particles and periods, at its own cells and rate of slots
        dict(name="undulator_mixed", kind="deposit", source="undulator", precision="mixed",
             options=0, n_p=1000, n_s=2048, n1=128, n2=128, n_t=1024),
        # the same ensemble in double precision at odd sizes
        dict(name="undulator_fp64_odd", kind="deposit", source="undulator", precision="fp64",
             options=0, n_p=777, n_s=1500, n1=97, n2=61, n_t=750),
        # the higher-order hold rule
        dict(name="undulator_linear_hold", kind="deposit", source="undulator", precision="mixed",
             options=HOLD_LINEAR, n_p=300, n_s=1024, n1=64, n2=64, n_t=512),
        # plasma-mirror sheet: the large configuration's electrons and cells a radian
        # over some of its steps (a slot or two crossed by every segment)
        dict(name="plasma_sheet_mixed", kind="deposit", source="plasma", precision="mixed",
             options=0, n_p=100000, n_s=16, n1=128, n2=128, n_t=4096, stride=1),
        # a chunk of the served stream, double precision, odd sizes
        dict(name="plasma_chunk_fp64", kind="deposit", source="plasma", precision="fp64",
             options=0, n_p=7001, n_s=37, n1=61, n2=83, n_t=4096, stride=1),
        # the sheet sampled four times as coarsely: six slots crossed by a segment
        dict(name="plasma_coarse", kind="deposit", source="plasma", precision="mixed", options=0,
             n_p=5000, n_s=24, n1=64, n2=64, n_t=4096, stride=4),
        # run-time mode: push a block of steps on the device and deposit it
        dict(name="runtime_block", kind="runtime", source="wave", precision="mixed", options=0,
             n_p=10000, n_s=16, n1=128, n2=128, n_t=2048),
        # uneven sets, each with its own detector, in one call
        dict(name="batch_uneven", kind="batch", precision="mixed", n_sets=8, recipe=11),
        # spectra: the paper's benchmark size, and an ordinary detector's
        dict(name="spectrum_long", kind="spectrum", precision="fp64", n1=512, n2=1, n_t=131072,
             weights=False),
        dict(name="spectrum_cap", kind="spectrum", precision="mixed", n1=128, n2=128, n_t=2048,
             weights=True),
    ]


def _logint(rng, lo, hi):
    """Log-uniform whole number in [lo, hi]; mostly odd or ragged sizes."""
    return int(min(hi, max(lo, round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["single", "undulator", "undulator", "plasma", "plasma", "coarse", "runtime",
                       "batch", "spectrum"])
    if kind == "single":
        if rng.random() < 0.5:
            return dict(kind="deposit", source="circular", precision=rng.choice(["fp64", "mixed"]),
                        options=0, n_p=rng.choice([1, 1, 2, 3, 5]), n_s=_logint(rng, 200, 8000),
                        n1=_logint(rng, 8, 64), n2=_logint(rng, 8, 64), n_t=_logint(rng, 64, 2048))
        n_s = _logint(rng, 3000, 25000)
        return dict(kind="deposit", source="sinusoidal", precision=rng.choice(["fp64", "mixed"]),
                    options=0, n_p=1, n_s=n_s, n1=_logint(rng, 16, 256), n2=1,
                    n_t=int(n_s * rng.uniform(1.0, 3.0)))
    if kind == "undulator":
        n_s = _logint(rng, 128, 2048)
        n1, n2 = _logint(rng, 8, 128), _logint(rng, 8, 128)
        n_p = _logint(rng, 20, 5000)
        n_p = max(1, min(n_p, int(2.0e10 / (n_s * n1 * n2))))
        return dict(kind="deposit", source="undulator",
                    precision=rng.choice(["mixed", "mixed", "fp64", "mixed_twosum"]),
                    options=rng.choice([0, 0, 0, FAR_FIELD, HOLD_PREVIOUS, HOLD_LINEAR]),
                    n_p=n_p, n_s=n_s, n1=n1, n2=n2, n_t=max(16, n_s // 2))
    if kind == "plasma":
        n_s = rng.randint(1, 64)
        n1, n2 = _logint(rng, 16, 128), _logint(rng, 16, 128)
        n_p = _logint(rng, 1000, 100000)
        n_p = max(100, min(n_p, int(1.0e10 / (n_s * n1 * n2))))
        return dict(kind="deposit", source="plasma",
                    precision=rng.choice(["mixed", "mixed", "fp64", "mixed_twosum"]), options=0,
                    n_p=n_p, n_s=n_s, n1=n1, n2=n2, n_t=_logint(rng, 1024, 4096), stride=1)
    if kind == "coarse":
        n_s = rng.randint(2, 24)
        n1, n2 = _logint(rng, 16, 64), _logint(rng, 16, 64)
        n_p = _logint(rng, 1000, 10000)
        n_p = max(100, min(n_p, int(4.0e8 / (n_s * n1 * n2))))
        return dict(kind="deposit", source="plasma", precision=rng.choice(["mixed", "fp64"]),
                    options=0, n_p=n_p, n_s=n_s, n1=n1, n2=n2, n_t=_logint(rng, 2048, 4096),
                    stride=rng.choice([2, 3, 4]))
    if kind == "runtime":
        n1, n2 = _logint(rng, 16, 128), _logint(rng, 16, 128)
        return dict(kind="runtime", source="wave", precision=rng.choice(["mixed", "fp64"]),
                    options=0, n_p=_logint(rng, 200, 10000), n_s=rng.choice([8, 16, 16, 32]),
                    n1=n1, n2=n2, n_t=_logint(rng, 512, 2048))
    if kind == "batch":
        return dict(kind="batch", precision=rng.choice(["mixed", "fp64"]),
                    n_sets=rng.randint(2, 6), recipe=rng.randint(100, 10**6))
    n_t = _logint(rng, 256, 65536)
    n_c = _logint(rng, 32, max(33, min(16384, int(3.0e7 / n_t))))
    return dict(kind="spectrum", precision=rng.choice(["fp64", "mixed", "mixed_twosum"]), n1=n_c,
                n2=1, n_t=n_t, weights=rng.random() < 0.5)


def _recipe(case):
    """The sets of a batch: log-uniform particles, uneven steps, cells and slots,
    helical or planar motion over four periods, gamma in [2, 100], K in [0.5, 3]."""
    rng = np.random.Generator(np.random.PCG64(int(case["recipe"])))
    sets = []
    for _ in range(case["n_sets"]):
        s = dict(n_p=int(round(10 ** rng.uniform(1.5, 3.3))), n_s=int(rng.integers(500, 2001)),
                 helical=bool(rng.integers(0, 2)), g0=float(rng.uniform(2.0, 100.0)),
                 K=float(rng.uniform(0.5, 3.0)), side=int(rng.choice([32, 64, 128])),
                 n_t=int(rng.choice([256, 512, 1024, 2048])))
        if s["helical"]:
            s["K"] = min(s["K"], math.sqrt(max((0.98 * s["g0"]) ** 2 - 1.0, 0.0)) * 0.5)
        else:
            s["K"] = min(s["K"], 0.8 * math.sqrt(s["g0"] ** 2 - 1.0))
        s["n_p"] = max(1, min(s["n_p"], int(5.0e9 / (s["n_s"] * s["side"] ** 2))))
        sets.append(s)
    return sets


def work(case):
    if case["kind"] == "spectrum":
        n_c, n_t = case["n1"] * case["n2"], case["n_t"]
        n = 1 << max(0, (n_t - 1).bit_length())
        return {"bytes": 24.0 * n_c * n_t + 8.0 * n_c * (n // 2 + 1),
                "flops": n_c * (3.0 * 2.5 * n * math.log2(n) + 8.0 * n)}
    total = {"bytes": 0.0, "flops": 0.0}
    sets = _recipe(case) if case["kind"] == "batch" else [case]
    for s in sets:
        n_c = s["side"] ** 2 if "side" in s else s["n1"] * s["n2"]
        # trajectories in, the detector's slots once, E and B out (float32 in the mixed modes)
        out = 48.0 if case["precision"] == "fp64" else 24.0
        total["bytes"] += 48.0 * s["n_p"] * (s["n_s"] + 1) + n_c * s["n_t"] * (48.0 + out)
        total["flops"] += FLOPS * s["n_p"] * s["n_s"] * n_c
    return total


# --------------------------------------------------------------------------
# inputs (on the GPU, from the seed)
# --------------------------------------------------------------------------

def _rng(seed):
    return np.random.Generator(np.random.PCG64(seed))


def _dev(a):
    return torch.as_tensor(np.asarray(a, dtype=np.float64), device="cuda")


def _cap(radius, axis, e1, n1, n2, half1, half2):
    """Cells on a cap of a sphere about `axis` (angles +-half1, +-half2), index i2 n1 + i1."""
    axis = np.asarray(axis, dtype=np.float64) / np.linalg.norm(axis)
    e1 = np.asarray(e1, dtype=np.float64)
    e1 = e1 - (e1 @ axis) * axis
    e1 /= np.linalg.norm(e1)
    e2 = np.cross(axis, e1)
    lon = -half1 + (np.arange(n1) + 0.5) * (2.0 * half1 / n1)
    lat = -half2 + (np.arange(n2) + 0.5) * (2.0 * half2 / n2)
    lat, lon = np.meshgrid(lat, lon, indexing="ij")
    d = (np.cos(lat)[..., None] * (np.cos(lon)[..., None] * axis + np.sin(lon)[..., None] * e1)
         + np.sin(lat)[..., None] * e2)
    return np.ascontiguousarray((radius * d).reshape(n1 * n2, 3))


def _corners(cells, n1, n2):
    at = [(n1 // 2, n2 // 2), (0, 0), (n1 - 1, 0), (0, n2 - 1), (n1 - 1, n2 - 1)]
    return _dev(cells[[i2 * n1 + i1 for i1, i2 in at]])


def _window(cells, n1, n2, x, t, n_t, pad):
    """(t0, dt_det) over the arrivals of states x (3, S+1, P) at times t at the
    corner and middle cells, padded by `pad` of the width."""
    lo, hi = math.inf, -math.inf
    for c in _corners(cells, n1, n2):
        tau = t[:, None] + ((c[:, None, None] - x) ** 2).sum(0).sqrt()
        lo, hi = min(lo, float(tau.min())), max(hi, float(tau.max()))
    w = hi - lo
    return lo - pad * w, (1.0 + 2.0 * pad) * w / n_t


def _times(n_s, dt, first=0):
    return torch.arange(first, first + n_s + 1, dtype=torch.float64, device="cuda") * dt


def _simpson(f, t, dt):
    """Integral of f (times -> (S+1, P)) from t[0], at every t."""
    a = f(t)
    m = f(t[:-1] + 0.5 * dt)
    out = torch.zeros_like(a)
    out[1:] = torch.cumsum((a[:-1] + 4.0 * m + a[1:]) * (dt / 6.0), 0)
    return out


def _circular(case, rng):
    gamma, dt, n_s = 5.0, 0.01, case["n_s"]
    beta = math.sqrt(1.0 - 1.0 / gamma**2)
    ph = beta * _times(n_s, dt)[:, None] + _dev(rng.uniform(0.0, TWO_PI, case["n_p"]))
    zero = torch.zeros_like(ph)
    x = torch.stack([torch.cos(ph), torch.sin(ph), zero])
    u = gamma * beta * torch.stack([-torch.sin(ph), torch.cos(ph), zero])
    n1, n2 = case["n1"], case["n2"]
    a1 = -50.0 + (np.arange(n1) + 0.5) * (100.0 / n1)
    a2 = -50.0 + (np.arange(n2) + 0.5) * (100.0 / n2)
    a2, a1 = np.meshgrid(a2, a1, indexing="ij")
    cells = np.stack([a1.ravel(), a2.ravel(), np.full(n1 * n2, 1000.0)], 1)
    return cells, x, u, dt, 0, _window(cells, n1, n2, x, _times(n_s, dt), case["n_t"], 0.002)


def _sinusoidal(case, rng):
    gamma, r_beta, k, dt, n_s = 50.0, 2.0, 0.1, 0.01, case["n_s"]
    K, ph0 = gamma * k * r_beta, float(rng.uniform(0.0, 0.1))
    t = _times(n_s, dt)
    uy = lambda s: K * torch.cos(k * s + ph0)[:, None]  # noqa: E731
    ux = lambda s: torch.sqrt(gamma**2 - 1.0 - uy(s) ** 2)  # noqa: E731
    y = (K / (gamma * k)) * torch.sin(k * t + ph0)[:, None]
    x = torch.stack([_simpson(lambda s: ux(s) / gamma, t, dt), y, torch.zeros_like(y)])
    u = torch.stack([ux(t), uy(t), torch.zeros_like(y)])
    n1, n2 = case["n1"], case["n2"]
    cells = _cap(1.0e5, [1, 0, 0], [0, 0, 1], n1, n2, 0.1, 0.0)
    return cells, x, u, dt, 0, _window(cells, n1, n2, x, t, case["n_t"], 0.01)


def _undulator(n_p, n_s, periods, g0, gs, K, rng):
    gam, x0, y0 = (_dev(rng.normal(m, s, n_p)) for m, s in ((g0, gs), (0.0, 0.1), (0.0, 0.1)))
    gam = torch.clamp(gam, min=math.sqrt(1.0 + 1.2 * K * K))
    dt = periods * TWO_PI / n_s
    t = _times(n_s, dt)
    ux = lambda s: (K * torch.sin(s))[:, None] * torch.ones_like(gam)  # noqa: E731
    uz = lambda s: torch.sqrt(gam**2 - 1.0 - ux(s) ** 2)  # noqa: E731
    x = torch.stack([x0 + (K / gam) * (1.0 - torch.cos(t))[:, None],
                     y0 + torch.zeros(n_s + 1, 1, dtype=torch.float64, device="cuda"),
                     _simpson(lambda s: uz(s) / gam, t, dt)])
    return x, torch.stack([ux(t), torch.zeros_like(x[0]), uz(t)]), dt


def _helix(n_p, n_s, periods, g0, gs, K, rng):
    gam, x0, y0 = (_dev(rng.normal(m, s, n_p)) for m, s in ((g0, gs), (0.0, 0.1), (0.0, 0.1)))
    gam = torch.clamp(gam, min=math.sqrt(1.0 + 1.2 * K * K))
    dt = periods * TWO_PI / n_s
    t = _times(n_s, dt)[:, None]
    uz = torch.sqrt(gam**2 - 1.0 - K * K)
    one = torch.ones_like(gam)
    x = torch.stack([x0 + (K / gam) * torch.sin(t), y0 + (K / gam) * (1.0 - torch.cos(t)),
                     (uz / gam) * t])
    return x, torch.stack([K * torch.cos(t) * one, K * torch.sin(t) * one, uz * torch.ones_like(t)]), dt


def _undulator_case(case, rng):
    # 4096 steps over 20 periods, as the framework's benchmark samples it
    x, u, dt = _undulator(case["n_p"], case["n_s"], case["n_s"] / 204.8, 50.0, 0.5, 1.0, rng)
    n1, n2 = case["n1"], case["n2"]
    # a patch of the benchmark's 128 x 128 cap (+-0.04 rad) at the same cells a radian
    cells = _cap(1.0e5, [0, 0, 1], [1, 0, 0], n1, n2, 0.04 * n1 / 128, 0.04 * n2 / 128)
    t = _times(case["n_s"], dt)
    return cells, x, u, dt, 0, _window(cells, n1, n2, x[:, :, :64], t, case["n_t"], 0.02)


_INC = math.pi / 4
_A = math.sqrt(1.0 - 1.0 / 100.0)  # peak gamma 10


def _plasma(case, rng):
    n_p, n_s = case["n_p"], case["n_s"]
    hw, ky = 10.0 * TWO_PI, math.sin(_INC)
    total = 1000 // case["stride"]  # steps of the whole run (ten laser periods)
    dt = 10.0 * TWO_PI / total
    first = int(rng.integers(0, max(1, total - n_s)))
    y0, z0 = _dev(rng.uniform(-hw, hw, n_p)), _dev(rng.uniform(-hw, hw, n_p))
    du = _dev(rng.normal(0.0, 0.01 * 10.0 * _A, (3, 1, n_p)))
    t = _times(n_s, dt, first)
    bx = _A * torch.cos(t[:, None] - ky * y0)
    u = du + torch.stack([bx / torch.sqrt(1.0 - bx * bx), torch.zeros_like(bx),
                          torch.zeros_like(bx)])
    beta = u / torch.sqrt(1.0 + (u * u).sum(0))
    x = torch.empty_like(u)
    x[0, 0] = _A * (torch.sin(t[0] - ky * y0) + torch.sin(ky * y0))
    x[1, 0], x[2, 0] = y0, z0
    x[:, 1:] = x[:, :1] + torch.cumsum(0.5 * dt * (beta[:, :-1] + beta[:, 1:]), 1)
    # a patch of the 256 x 256 cap about the specular direction at its cells a radian
    n1, n2 = case["n1"], case["n2"]
    cells = _cap(1.0e5, [-math.cos(_INC), math.sin(_INC), 0.0],
                 [math.sin(_INC), math.cos(_INC), 0.0], n1, n2, 0.1 * n1 / 256, 0.1 * n2 / 256)
    # the window of the whole run, at the whole cap's corners
    ts = torch.linspace(0.0, 10.0 * TWO_PI, 201, dtype=torch.float64, device="cuda")
    ys = _dev(np.linspace(-hw, hw, 33))
    xs = _A * (torch.sin(ts[:, None] - ky * ys) + torch.sin(ky * ys))
    path = torch.stack([xs, ys + torch.zeros_like(xs), torch.zeros_like(xs)])
    path = torch.cat([path + _dev([0.0, 0.0, z]).view(3, 1, 1) for z in (-hw, 0.0, hw)], 2)
    cap = _cap(1.0e5, [-math.cos(_INC), math.sin(_INC), 0.0],
               [math.sin(_INC), math.cos(_INC), 0.0], 2, 2, 0.1, 0.1)
    return cells, x, u, dt, first, _window(cap, 2, 2, path, ts, case["n_t"], 0.02)


_WAVE = dict(qm=-1.0, wave_amplitude=1.5, wave_dir=[1.0, 0.0, 0.0], wave_pol=[0.0, 1.0, 0.0],
             wave_omega=1.0, wave_phase=0.0)


def _boris(x0, u0, dt, n_s, first=0):
    """States of electrons in the plane wave _WAVE: half drift, kick, half drift."""
    xs, us = [x0], [u0]
    x, u, h = x0, u0, -0.5 * dt
    for s in range(first, first + n_s):
        xh = x + 0.5 * dt * u / torch.sqrt(1.0 + (u * u).sum(0))
        w = 1.5 * torch.cos((s + 0.5) * dt - xh[0])
        um = torch.stack([u[0], u[1] + h * w, u[2]])
        tz = h * w / torch.sqrt(1.0 + (um * um).sum(0))  # B = k x E along +z
        up0, up1 = um[0] + um[1] * tz, um[1] - um[0] * tz
        sz = 2.0 / (1.0 + tz * tz) * tz
        u = torch.stack([um[0] + up1 * sz, um[1] - up0 * sz + h * w, um[2]])
        x = xh + 0.5 * dt * u / torch.sqrt(1.0 + (u * u).sum(0))
        xs.append(x)
        us.append(u)
    return torch.stack(xs, 1), torch.stack(us, 1)


def _wave(case, rng):
    """A block in the middle of a run-time run: state 0 only; pushed in the pass."""
    dt, first = 0.05, 160
    x0 = _dev(rng.uniform(-2.0, 2.0, (3, case["n_p"])))
    xs, us = _boris(x0, torch.zeros_like(x0), dt, first)
    x = torch.zeros((3, case["n_s"] + 1, case["n_p"]), dtype=torch.float64, device="cuda")
    u = torch.zeros_like(x)
    x[:, 0], u[:, 0] = xs[:, -1], us[:, -1]
    n1, n2 = case["n1"], case["n2"]
    cells = _cap(1.0e4, [1, 0, 0], [0, 1, 0], n1, n2, 0.3 * n1 / 128, 0.3 * n2 / 128)
    cap = _cap(1.0e4, [1, 0, 0], [0, 1, 0], 2, 2, 0.3, 0.3)
    # the window of a run of 1024 steps, from a sample of electrons in longer steps
    xr, _ = _boris(x0[:, :64], torch.zeros_like(x0[:, :64]), 4 * dt, 256)
    return cells, x, u, dt, first, _window(cap, 2, 2, xr, _times(256, 4 * dt), case["n_t"], 0.05)


_SOURCES = dict(circular=_circular, sinusoidal=_sinusoidal, undulator=_undulator_case,
                plasma=_plasma, wave=_wave)


def _inputs(case, seed):
    """[(cells, x, u, q, dt, first_step, t0, dt_det, n_t)] of a case."""
    if case["kind"] != "batch":
        cells, x, u, dt, first, (t0, dtd) = _SOURCES[case["source"]](case, _rng(seed))
        q = torch.full((x.shape[2],), -1.0, dtype=torch.float64, device="cuda")
        return [(cells, x.contiguous(), u.contiguous(), q, dt, first, t0, dtd, case["n_t"])]
    out = []
    for i, s in enumerate(_recipe(case)):
        make = _helix if s["helical"] else _undulator
        x, u, dt = make(s["n_p"], s["n_s"], 4.0, s["g0"], 0.01 * s["g0"], s["K"],
                        _rng(seed + 7919 * i))
        half, side = (1.0 + s["K"]) / s["g0"], s["side"]
        cells = _cap(1.0e4, [0, 0, 1], [1, 0, 0], side, side, half, half)
        t0, dtd = _window(cells, side, side, x[:, :, :64], _times(s["n_s"], dt), s["n_t"], 0.02)
        q = torch.full((s["n_p"],), -1.0, dtype=torch.float64, device="cuda")
        out.append((cells, x.contiguous(), u.contiguous(), q, dt, 0, t0, dtd, s["n_t"]))
    return out


def _signals(case, seed):
    """E and B (n_c, n_t, 3) of a chirped pulse seen at slightly different
    frequencies and phases by the cells, with a weak second component."""
    n_c, n_t = case["n1"] * case["n2"], case["n_t"]
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    rnd = lambda lo, hi: lo + (hi - lo) * torch.rand(  # noqa: E731
        n_c, 1, dtype=torch.float64, device="cuda", generator=g)
    t = torch.linspace(0.0, 1.0, n_t, dtype=torch.float64, device="cuda")
    E = torch.empty((n_c, n_t, 3), dtype=torch.float64, device="cuda")
    w = TWO_PI * n_t / 40.0
    for k, amp in enumerate((1.0, 0.3, 0.05)):
        c, width, f, ph = rnd(0.3, 0.7), rnd(0.05, 0.3), rnd(0.5, 1.5), rnd(0.0, TWO_PI)
        E[:, :, k] = amp * torch.exp(-(((t - c) / width) ** 2)) * torch.cos(w * f * t * (1 + t) + ph)
    return E, torch.stack([-E[..., 1], E[..., 0], 0.1 * E[..., 2]], 2)


def _line(case):
    return _cap(1.0e5, [1, 0, 0], [0, 0, 1], case["n1"], case["n2"], 0.1,
                0.1 if case["n2"] > 1 else 0.0)


_SPEC_DT = 1.0e-3


def _weights(case):
    n = case["n1"] * case["n2"]
    return 0.5 + (np.arange(n) % 17) / 16.0 if case["weights"] else None


# --------------------------------------------------------------------------
# a program's state, and one pass
# --------------------------------------------------------------------------

def prepare(case, seed):
    if case["kind"] == "spectrum":
        det = radio.Detector(_line(case), t0=0.0, dt_det=_SPEC_DT, n_t=case["n_t"],
                             precision=case["precision"])
        det.load(*_signals(case, seed))
        return dict(kind="spectrum", det=det, weights=_weights(case))
    dets, chunks, bufs = [], [], []
    for cells, x, u, q, dt, first, t0, dtd, n_t in _inputs(case, seed):
        dets.append(radio.Detector(cells, t0=t0, dt_det=dtd, n_t=n_t, precision=case["precision"],
                                   options=case.get("options", 0)))
        chunks.append(radio.Chunk(x, u, q, 0.0, dt, first))
        bufs.append([torch.empty((cells.shape[0], n_t, 3), dtype=torch.float64, device="cuda")
                     for _ in range(2)])
    return dict(kind=case["kind"], dets=dets, chunks=chunks, bufs=bufs,
                single=case["precision"] != "fp64")


def _read(state, i):
    E, B = state["dets"][i].read(*state["bufs"][i])
    return (E.float(), B.float()) if state["single"] else (E, B)


def run(state):
    if state["kind"] == "spectrum":
        _, d2I, dIdw, dIdO = state["det"].spectrum(weights=state["weights"])
        return {"d2I": d2I, "dIdw": dIdw, "dIdO": dIdO}
    for det in state["dets"]:
        det.reset()
    if state["kind"] == "batch":
        radio.deposit_batch(state["dets"], state["chunks"])
        return [_read(state, i) for i in range(len(state["dets"]))]
    chunk = state["chunks"][0]
    if state["kind"] == "runtime":
        radio.push(chunk, **_WAVE)
        radio.deposit_batch(state["dets"], state["chunks"])
        E, B = _read(state, 0)
        return {"E": E, "B": B, "x": chunk.x, "u": chunk.u}
    state["dets"][0].deposit(chunk)
    E, B = _read(state, 0)
    return {"E": E, "B": B}


# --------------------------------------------------------------------------
# the same in plain 64-bit torch
# --------------------------------------------------------------------------

def _kinematics(x, u, dt, options):
    """beta, betadot by the hold rule's difference, 1/gamma^2."""
    g2 = 1.0 + (u * u).sum(0)
    beta = u / torch.sqrt(g2)
    bd = torch.zeros_like(beta)
    step = (beta[:, 1:] - beta[:, :-1]) / dt
    bd[:, 1:] = step
    if options & HOLD_PREVIOUS:
        bd[:, 0] = step[:, 0]
    if options & HOLD_LINEAR:
        bd[:, 0] = step[:, 0]
        bd[:, 1:-1] = (beta[:, 2:] - beta[:, :-2]) / (2.0 * dt)
    return beta, bd, 1.0 / g2


def _block_fields(cells, x, beta, bd, g2i, q, t, options):
    """Arrival times (C, S+1, P) and E, B [6] of Eq. 1 at a block of cells."""
    dot = lambda a, b: a[0] * b[0] + a[1] * b[1] + a[2] * b[2]  # noqa: E731
    cross = lambda a, b: [a[1] * b[2] - a[2] * b[1], a[2] * b[0] - a[0] * b[2],  # noqa: E731
                          a[0] * b[1] - a[1] * b[0]]
    c = [cells[:, k, None, None] for k in range(3)]
    if options & FAR_FIELD:
        R = torch.sqrt((c[0] * c[0] + c[1] * c[1]) + c[2] * c[2])
        ri = 1.0 / R
        n = [v * ri for v in c]
        tau = t[None, :, None] + (R - ((x[0] * n[0] + x[1] * n[1]) + x[2] * n[2]))
    else:
        d = [c[k] - x[k] for k in range(3)]
        R = torch.sqrt((d[0] * d[0] + d[1] * d[1]) + d[2] * d[2])
        ri = 1.0 / R
        n = [v * ri for v in d]
        tau = t[None, :, None] + R
    w = [n[k] - beta[k] for k in range(3)]
    kap = 0.5 * (dot(w, w) + g2i)
    a = cross(n, cross(w, [bd[0], bd[1], bd[2]]))
    cv = q * g2i * ri * ri / kap**3
    ca = q * ri / kap**3
    E = [cv * w[k] + ca * a[k] for k in range(3)]
    return tau, E + cross(n, E)


def _exact_deposit(case, inputs):
    cells, x, u, q, dt, first, t0, dtd, n_t = inputs
    opt = case.get("options", 0)
    n_p, n_s = x.shape[2], x.shape[1] - 1
    beta, bd, g2i = _kinematics(x, u, dt, opt)
    t = _times(n_s, dt, first)
    cells = _dev(cells)
    acc = torch.zeros((cells.shape[0] * n_t, 6), dtype=torch.float64, device="cuda")
    per = max(1, int(6.0e6 // (n_s + 1)))
    cb = max(1, min(cells.shape[0], per // min(n_p, per)))
    pb = min(n_p, max(1, per // cb))
    for c0 in range(0, cells.shape[0], cb):
        for p0 in range(0, n_p, pb):
            sl = slice(p0, p0 + pb)
            cell = cells[c0:c0 + cb]
            tau, F = _block_fields(cell, x[:, :, sl], beta[:, :, sl], bd[:, :, sl], g2i[:, sl],
                                   q[sl], t, opt)
            s = (tau - t0) / dtd
            a, b = s[:, :-1], s[:, 1:]
            lo = torch.minimum(a, b).clamp(0.0, n_t)
            hi = torch.maximum(a, b).clamp(0.0, n_t)
            F = torch.stack(F, -1)
            Fa, Fb = F[:, :-1], F[:, 1:]
            if opt & HOLD_PREVIOUS:
                Fb = Fa
            J = lo.floor()
            row = (torch.arange(cell.shape[0], device="cuda") + c0)[:, None, None] * n_t
            for j in range(int((hi.ceil() - J).max())):
                left, right = torch.maximum(lo, J + j), torch.minimum(hi, J + (j + 1))
                on = right > left
                weight = (right - left)[on][:, None]
                f = Fb[on]
                if opt & HOLD_LINEAR:
                    mid = (0.5 * ((left - a) + (right - a)) / (b - a))[on][:, None]
                    f = Fa[on] + (f - Fa[on]) * mid
                acc.index_add_(0, (row + J.long() + j)[on], f * weight)
    acc = acc.view(cells.shape[0], n_t, 6)
    return acc[..., :3].contiguous(), acc[..., 3:].contiguous()


def _exact_spectrum(case, seed):
    E, _ = _signals(case, seed)
    cells = _dev(_line(case))
    n_t, dt = case["n_t"], _SPEC_DT
    N = 1 << max(0, (n_t - 1).bit_length())
    om = TWO_PI * torch.arange(N // 2 + 1, dtype=torch.float64, device="cuda") / (N * dt)
    W = torch.where(om == 0, torch.full_like(om, dt), 2.0 * torch.sin(0.5 * om * dt) / om)
    R2 = (cells * cells).sum(1)
    d2I = torch.empty((E.shape[0], N // 2 + 1), dtype=torch.float64, device="cuda")
    for c0 in range(0, E.shape[0], 256):
        f = torch.fft.rfft(E[c0:c0 + 256].transpose(1, 2).contiguous(), n=N, dim=2)
        d2I[c0:c0 + 256] = (f.real**2 + f.imag**2).sum(1)
    d2I *= (R2 / (4.0 * math.pi**2))[:, None] * W * W
    w = _weights(case)
    w = torch.ones_like(R2) if w is None else _dev(w)
    return {"d2I": d2I, "dIdw": (w[:, None] * d2I).sum(0),
            "dIdO": R2 / (4.0 * math.pi) * (E * E).sum((1, 2)) * dt}


def exact(case, seed):
    if case["kind"] == "spectrum":
        return _exact_spectrum(case, seed)
    slots = {"plasma": 2.5 * case.get("stride", 1), "wave": 3.0, "sinusoidal": 4.0}
    if work(case)["flops"] / FLOPS * slots.get(case.get("source"), 1.3) > EXACT_MOST:
        return None
    inputs = _inputs(case, seed)
    if case["kind"] == "batch":
        return [_exact_deposit(case, i) for i in inputs]
    (i,) = inputs
    if case["kind"] == "runtime":
        x, u = _boris(i[1][:, 0], i[2][:, 0], i[4], case["n_s"], i[5])
        E, B = _exact_deposit(case, (i[0], x, u) + i[3:])
        return {"E": E, "B": B, "x": x, "u": u}
    E, B = _exact_deposit(case, i)
    return {"E": E, "B": B}
