"""Timing cases of the library: what a pass of each is, its inputs, and its
results in float64.

A pass is a stretch of time steps through the public entry points: a shot
(`Shot.record`, `Shot.step`, `Shot.traces`, sometimes `Shot.read`), a batch of
shots (`Batch.add`, `Batch.run`, `Batch.remove`), or the serving loop
(`Server.run`).  Shots and batches continue from a wavefield in flight that
`prepare` writes (as a restart does), so every point of the grid carries signal
from the first step on; each pass takes the next stretch, and its receivers
are set anew, which empties the trace buffer.

Sizes are those of the tests and of the benchmark: the 64^3 parity grid, small
ragged grids, the 128-384 range of the many-shot workload, the 512^3 benchmark
shot in float32 and bf16, and the 1000-wide planes with the 27-cell layer of
the paper's grid (with 256 planes, so that the model is quick to make).
"""
from __future__ import annotations

import math
import random
from types import SimpleNamespace

import numpy as np
import torch

from paper_2009_04619_amd import serve as S
from paper_2009_04619_amd import wave as W

DEV = "cuda:0"
H = 10.0        # grid spacing (m)
F0 = 15.0       # Ricker peak frequency (Hz)
REFL = 1e-3     # the damping profile's target reflection (the default)
MAX_POINTS = 1000 * 1000 * 256      # the largest listed grid
MAX_UPDATES = 512 ** 3 * 100        # the most point updates of a listed pass


def _shot(name, nx, ny, nz, w, steps, storage="f32", nsrc=1, rec="line", eta=False,
          damping=True, sr=False, field=False):
    c = dict(kind="shot", nx=nx, ny=ny, nz=nz, w=w, steps=steps, storage=storage, nsrc=nsrc,
             rec=rec, eta_array=eta, damping=damping, stochastic_round=sr, read_field=field)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the 64^3 parity configuration, 100 steps with a receiver line: the
        # smallest complete run, where launches and latency count
        _shot("c1_64cube_f32", 64, 64, 64, 16, 100),
        # a quick check run on a ragged grid: two sources, scattered
        # receivers, the final field read back
        _shot("ragged_70x45x37_f32_field", 70, 45, 37, 5, 20, nsrc=2, rec="scatter", field=True),
        # a small shot with the user's own damping array, its final field kept
        _shot("eta_array_128x112x96_f32_field", 128, 112, 96, 20, 100, eta=True, field=True),
        # one shot of the many-shot workload, run on its own
        _shot("shot_176x144x160_f32", 176, 144, 160, 20, 100),
        # a mid-size shot of odd width in half precision, stations all over it
        _shot("shot_333x256x272_f16", 333, 256, 272, 20, 50, storage="f16", rec="scatter"),
        # stochastically rounded bf16 storage
        _shot("shot_256x240x256_bf16_sr", 256, 240, 256, 20, 50, storage="bf16", sr=True),
        # a rigid box: no layer (the energy and dispersion studies)
        _shot("box_320x304x288_f32_no_layer", 320, 304, 288, 0, 50, rec="scatter", damping=False),
        # the benchmark shot, float32 and bf16
        _shot("c2_512cube_f32", 512, 512, 512, 20, 100),
        _shot("c2_512cube_bf16", 512, 512, 512, 20, 100, storage="bf16"),
        # the paper's planes: 1000 x 1000 with a 27-cell layer
        _shot("paper_1000x1000x256_f32", 1000, 1000, 256, 27, 25),
        # uneven shots of 128-256 cells advanced together
        dict(kind="batch", name="batch_8_uneven_f32", shots=8, lo=128, hi=256, shape_seed=4000,
             steps=50, storage="f32"),
        # the serving loop: requests of every storage type, set-up to traces
        dict(kind="serve", name="serve_6_mixed", requests=6, lo=96, hi=160, shape_seed=5000,
             smin=120, smax=240),
    ]


def _extent(rng, lo, hi):
    """An extent spread over its logarithm, one in two of them odd."""
    n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    return max(lo, min(hi, n | 1 if rng.random() < 0.5 else n))


def draw(rng):
    r = rng.random()
    if r < 0.12:
        return dict(kind="batch", shots=rng.randint(2, 8), lo=96, hi=rng.choice([160, 192, 224, 256]),
                    shape_seed=rng.randint(0, 1 << 20), steps=rng.randint(20, 50),
                    storage=rng.choice(["f32", "f32", "bf16", "f16"]))
    if r < 0.2:
        return dict(kind="serve", requests=rng.randint(2, 6), lo=64, hi=rng.choice([96, 128, 160]),
                    shape_seed=rng.randint(0, 1 << 20), smin=100, smax=rng.randint(150, 240))
    while True:
        top = math.exp(rng.uniform(math.log(64), math.log(1000)))
        nx, ny, nz = (_extent(rng, max(36, int(top / 2)), max(48, min(1000, int(top)))) for _ in range(3))
        if nx * ny * nz <= MAX_POINTS:
            break
    w = min(rng.choice([5, 10, 16, 20, 20, 20, 27, 32]), min(nx, ny, nz) // 2)
    damping = rng.random() < 0.85
    eta = damping and nx * ny * nz < 1 << 24 and rng.random() < 0.2
    storage = rng.choice(["f32", "f32", "f32", "bf16", "bf16", "f16"])
    steps = min(rng.randint(20, 120), max(10, MAX_UPDATES // (nx * ny * nz)))
    return _shot(None, nx, ny, nz, w if damping else 0, steps, storage=storage,
                 nsrc=rng.choice([1, 1, 1, 2, 3]), rec=rng.choice(["line", "line", "scatter"]),
                 eta=eta, damping=damping, sr=storage == "bf16" and not eta and rng.random() < 0.3,
                 field=nx * ny * nz < 1 << 21 and rng.random() < 0.3)


# ---- inputs ------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) & 0x7FFFFFFF)
    return g


def _axes(nx, ny, nz):
    f = lambda n, s: torch.arange(n, device=DEV, dtype=torch.float32).reshape(s)
    return f(nx, (1, 1, -1)), f(ny, (1, -1, 1)), f(nz, (-1, 1, 1))


def _velocity(nx, ny, nz, g):
    """Eight flat layers of increasing velocity with a smooth 5 % perturbation (m/s)."""
    v, _ = torch.sort(torch.rand(8, device=DEV, generator=g) * 3000.0 + 1500.0)
    cuts, _ = torch.sort(torch.rand(7, device=DEV, generator=g) * nz)
    x, y, z = _axes(nx, ny, nz)
    vel = v[torch.searchsorted(cuts, z.reshape(-1).contiguous())].reshape(-1, 1, 1).expand(nz, ny, nx).clone()
    k = (torch.rand(4, 3, device=DEV, generator=g) * 0.4 - 0.2).tolist()
    p = (torch.rand(4, device=DEV, generator=g) * 6.283).tolist()
    pert = torch.zeros((nz, ny, nx), device=DEV)
    for (a, b, c), ph in zip(k, p):
        pert += torch.cos(a * x + b * y + c * z + ph)
    vel *= 1.0 + 0.025 * pert
    return vel.clamp_(1350.0, 4950.0).float()


def _waves(nx, ny, nz, dt, g, dtype):
    """u at two consecutive times: plane waves of 10 to 30 cells per wavelength."""
    x, y, z = _axes(nx, ny, nz)
    d = torch.randn(5, 3, device=DEV, generator=g)
    d = d / d.norm(dim=1, keepdim=True)
    lam = torch.rand(5, device=DEV, generator=g) * 20.0 + 10.0
    k = (d * (6.283185307 / lam)[:, None]).tolist()
    wdt = (6.283185307 / lam / H * 2500.0 * dt).tolist()
    ph = (torch.rand(5, device=DEV, generator=g) * 6.283).tolist()
    out = []
    for back in (0.0, 1.0):
        u = torch.zeros((nz, ny, nx), device=DEV)
        for (a, b, c), o, p in zip(k, wdt, ph):
            u += 0.2 * torch.cos(a * x + b * y + c * z + p + back * o)
        out.append(u.to(dtype).float())
    return out


def _ricker(n, dt, t0):
    a = (math.pi * F0 * (np.arange(n, dtype=np.float64) * dt - t0)) ** 2
    return ((1.0 - 2.0 * a) * np.exp(-a)).astype(np.float32)


def _eta_array(nx, ny, nz, w, vmax, dt, g):
    """A user's damping array: a cubic ramp per axis, its strength varied smoothly."""
    eta = torch.zeros((nz, ny, nx), device=DEV, dtype=torch.float64)
    d0 = 3.0 * vmax * math.log(1.0 / REFL) / (2.0 * w * H)
    for n, a in zip((nx, ny, nz), _axes(nx, ny, nz)):
        depth = torch.maximum(w - a, a - (n - 1 - w)).clamp_min(0).double() / w
        eta += d0 * dt * depth ** 3
    x, y, z = _axes(nx, ny, nz)
    ph = (torch.rand(2, device=DEV, generator=g) * 6.283).tolist()
    eta *= 1.0 + 0.1 * torch.cos(0.05 * x + 0.07 * y + ph[0]).double() * torch.cos(0.06 * z + ph[1]).double()
    return eta.float()


_TORCH = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}


def _inputs(case, seed, flight=True):
    """Everything a shot is made of: the arrays stay on the GPU as tensors."""
    g = _gen(seed)
    nx, ny, nz, w = case["nx"], case["ny"], case["nz"], case["w"]
    vel = _velocity(nx, ny, nz, g)
    vmax = float(vel.max())
    dt = 0.4 * H / vmax
    s = SimpleNamespace(nx=nx, ny=ny, nz=nz, w=w, dx=H, dy=H, dz=H, dt=dt, steps=case["steps"],
                        vel=vel, vmax=vmax, eta=None, storage=case["storage"],
                        damping=case.get("damping", True), sr=case.get("stochastic_round", False))
    if case.get("eta_array"):
        s.eta = _eta_array(nx, ny, nz, w, vmax, dt, g)
    s.u = _waves(nx, ny, nz, dt, g, _TORCH[case["storage"]]) if flight else None
    r = random.Random(seed)
    k = min(nz - 1, w + 5)
    s.src = [(nx // 2, ny // 2, k)]
    for _ in range(1, case.get("nsrc", 1)):
        s.src.append((r.randrange(nx), r.randrange(ny), r.randrange(nz)))
    # wavefields in flight: the wavelet is at its peak in the middle of the first pass
    t0 = 1.5 / F0 if not flight else 0.5 * s.steps * dt
    s.wavelet = np.stack([_ricker(s.steps, dt, t0 * (1.0 + 0.2 * q)) * 10.0 for q in range(len(s.src))])
    if case.get("rec", "line") == "line":
        s.rec = np.array([(i, ny // 2, k) for i in range(nx)], np.int32)
    else:
        s.rec = np.array([(r.randrange(nx), r.randrange(ny), r.randrange(nz)) for _ in range(64)], np.int32)
    return s


def _make(s):
    """The library's context for a shot in flight."""
    sh = W.Shot(s.nx, s.ny, s.nz, s.w, s.dx, s.dy, s.dz, s.dt, s.vel.cpu().numpy(),
                eta=None if s.eta is None else s.eta.cpu().numpy(), storage=s.storage,
                damping=s.damping, refl=REFL, max_src=len(s.src), max_rec=len(s.rec),
                max_steps=s.steps, device=DEV, stochastic_round=s.sr)
    for q, (i, j, k) in enumerate(s.src):
        sh.inject(i, j, k, s.wavelet[q])
    sh.write(W.WAVE_FIELD_U, s.u[0].cpu().numpy())
    sh.write(W.WAVE_FIELD_UPREV, s.u[1].cpu().numpy())
    return sh


def _members(case):
    """The shots of a batch or of a request stream, as cases of their own."""
    r = random.Random(case["shape_seed"])
    out = []
    for i in range(case.get("shots", case.get("requests", 0))):
        nx, ny, nz = (16 * r.randint(case["lo"] // 16, case["hi"] // 16) for _ in range(3))
        serve = case["kind"] == "serve"
        out.append(dict(nx=nx, ny=ny, nz=nz, w=20,
                        steps=r.randint(case["smin"], case["smax"]) if serve else case["steps"],
                        storage=("f32", "bf16", "f16")[i % 3] if serve else case["storage"]))
    return out


def prepare(case, seed):
    if case["kind"] == "shot":
        s = _inputs(case, seed)
        return dict(kind="shot", shot=_make(s), rec=s.rec, steps=s.steps, field=case["read_field"])
    if case["kind"] == "batch":
        # a batch keeps its tables; its members leave and join again with every pass
        batch = W.Batch(storage=case["storage"], max_shots=case["shots"], device=DEV)
        batch.set_kernel(*S.GpuExecutor.TILES[case["storage"]])
        shots, recs = [], []
        for i, c in enumerate(_members(case)):
            s = _inputs(c, seed * 64 + i)
            shots.append(_make(s))
            recs.append(s.rec)
        return dict(kind="batch", batch=batch, shots=shots, recs=recs, steps=case["steps"])
    jobs = []
    for i, c in enumerate(_members(case)):
        s = _inputs(c, seed * 64 + i, flight=False)
        s.vel = s.vel.cpu().numpy()
        jobs.append((s, c["storage"]))
    return dict(kind="serve", executor=S.GpuExecutor(device=DEV), jobs=jobs)


def run(state):
    if state["kind"] == "shot":
        sh = state["shot"]
        sh.record(state["rec"])
        sh.step(state["steps"])
        out = {"traces": sh.traces()}
        if state["field"]:
            out["u"] = sh.read(W.WAVE_FIELD_U)
        return out
    if state["kind"] == "batch":
        b = state["batch"]
        for sh, rec in zip(state["shots"], state["recs"]):
            sh.record(rec)
            b.add(sh, state["steps"])
        b.run(state["steps"])
        for sh in state["shots"]:
            b.remove(sh)
        return [sh.traces() for sh in state["shots"]]
    reqs = [S.Request(rid=i, arrival=0.0, shot=s, storage=st) for i, (s, st) in enumerate(state["jobs"])]
    done = S.Server(state["executor"], budget_bytes=64 << 30).run(reqs)
    return [r.traces for r in done]


# ---- the work of a pass -------------------------------------------------------
def work(case):
    """State read once and written once, model read once, traces written once;
    operations of every step: 38 for the Laplacian and the update of an inner
    point, 60 for a layer point."""
    if case["kind"] != "shot":
        each = [work(dict(c, kind="shot")) for c in _members(case)]
        return {k: sum(e[k] for e in each) for k in ("bytes", "flops")}
    nx, ny, nz, w = case["nx"], case["ny"], case["nz"], case["w"]
    pts = nx * ny * nz
    layer = pts - (nx - 2 * w) * (ny - 2 * w) * (nz - 2 * w) if case.get("damping", True) else 0
    es = 4 if case["storage"] == "f32" else 2
    per = 4 * es + 4                                # u, u_prev in and out, vp
    nrec = nx if case.get("rec", "line") == "line" else 64
    b = pts * per + layer * (8 + (4 if case.get("eta_array") else 0)) + 8 * nrec * case["steps"]
    if case.get("read_field"):
        b += 4 * pts
    return {"bytes": float(b), "flops": float(case["steps"] * (38 * (pts - layer) + 60 * layer))}


# ---- the same passes in float64 -------------------------------------------------
_WM = (8.0 / 5.0, -1.0 / 5.0, 8.0 / 315.0, -1.0 / 560.0)


def _ramps(s):
    """Per axis (x, y, z): the profile t(i) for i = -1..n."""
    out = []
    for n in (s.nx, s.ny, s.nz):
        i = torch.arange(-1, n + 1, device=DEV, dtype=torch.float64)
        depth = torch.maximum(s.w - i, i - (n - 1 - s.w)).clamp_min(0)
        out.append(3.0 * s.vmax * math.log(1.0 / REFL) / (2.0 * s.w * H) * (depth / s.w) ** 2)
    return out


def _exact_shot(s, field):
    nx, ny, nz, w = s.nx, s.ny, s.nz, s.w
    pad = lambda: torch.zeros((nz + 8, ny + 8, nx + 8), device=DEV, dtype=torch.float64)
    view = lambda a, dz=0, dy=0, dx=0: a[4 + dz:4 + dz + nz, 4 + dy:4 + dy + ny, 4 + dx:4 + dx + nx]
    cur, prev = pad(), pad()
    if s.u is not None:
        view(cur).copy_(s.u[0])
        view(prev).copy_(s.u[1])
    vel = s.vel if torch.is_tensor(s.vel) else torch.from_numpy(s.vel).to(DEV)
    vp = (vel.double() * s.dt) ** 2
    damp = s.damping and w > 0
    if damp:
        shapes = ((1, 1, -1), (1, -1, 1), (-1, 1, 1))
        q = 1.0 / (4.0 * H * H)
        if s.eta is None:
            t = _ramps(s)
            eta = sum((s.dt * a[1:-1]).reshape(sh) for a, sh in zip(t, shapes))
            dq = [(s.dt * q * (a[2:] - a[:-2])).reshape(sh) for a, sh in zip(t, shapes)]
        else:
            e = torch.zeros((nz + 2, ny + 2, nx + 2), device=DEV, dtype=torch.float64)
            e[1:-1, 1:-1, 1:-1] = s.eta
            eta = e[1:-1, 1:-1, 1:-1].clone()
            dq = [q * (e[1:-1, 1:-1, 2:] - e[1:-1, 1:-1, :-2]), q * (e[1:-1, 2:, 1:-1] - e[1:-1, :-2, 1:-1]),
                  q * (e[2:, 1:-1, 1:-1] - e[:-2, 1:-1, 1:-1])]
        layer = torch.ones((nz, ny, nx), device=DEV, dtype=torch.bool)
        layer[w:nz - w, w:ny - w, w:nx - w] = False
        eta = torch.where(layer, eta, torch.zeros((), device=DEV, dtype=torch.float64))
        phi = torch.zeros((nz, ny, nx), device=DEV, dtype=torch.float64)
    ri = [torch.tensor(s.rec[:, a].astype(np.int64), device=DEV) for a in range(3)]
    wav = torch.from_numpy(s.wavelet).to(DEV).double()
    rows = []
    for n in range(s.steps):
        u = view(cur)
        lap = u * (-205.0 / 72.0 * 3.0 / (H * H))
        for m, c in enumerate(_WM, 1):
            for d in ((0, 0, m), (0, m, 0), (m, 0, 0)):
                lap.add_(view(cur, *d), alpha=c / (H * H))
                lap.add_(view(cur, *(-v for v in d)), alpha=c / (H * H))
        if damp:
            lap += phi
        lap *= vp
        lap += u
        lap -= view(prev)
        if damp:
            lap.addcmul_(eta * eta, u, value=-1.0)
            lap /= 1.0 + 2.0 * eta
            gr = dq[0] * (view(cur, 0, 0, 1) - view(cur, 0, 0, -1))
            gr += dq[1] * (view(cur, 0, 1, 0) - view(cur, 0, -1, 0))
            gr += dq[2] * (view(cur, 1, 0, 0) - view(cur, -1, 0, 0))
            phi -= gr
            phi /= 1.0 + eta
            phi *= layer
        lap += u
        view(prev).copy_(lap)
        cur, prev = prev, cur
        u = view(cur)
        for q_ in range(len(s.src)):    # in order: sources may share a cell
            i, j, k = s.src[q_]
            u[k, j, i] += vp[k, j, i] * wav[q_, n]
        rows.append(u[ri[2], ri[1], ri[0]])
    out = {"traces": torch.stack(rows)}
    if field:
        out["u"] = view(cur).clone()
    return out


def exact(case, seed):
    if case["kind"] == "shot":
        return _exact_shot(_inputs(case, seed), case["read_field"])
    flight = case["kind"] == "batch"
    return [_exact_shot(_inputs(c, seed * 64 + i, flight=flight), False)["traces"]
            for i, c in enumerate(_members(case))]
