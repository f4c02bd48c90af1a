"""Performance cases: the calls a program makes of this package, over the range
of sizes it makes them at, with inputs made from a seed and 64-bit values of
what the calls return.

A case is a dict of plain values. `kind` says which public calls one pass makes:

  forward   Plan.forward                       (modelling: data of a model)
  gradient  Plan.forward(save) + l2_misfit + Plan.backward
            (one evaluation of misfit and gradient, what every inversion repeats)
  born      Plan.born                          (one application of the linearised map)
  batch     Batch.forward(save) + l2_misfit + Batch.backward of uneven models
  mlp       MLPVelocity.forward + backward + step  (one training iteration)

`physics` is acoustic, elastic, acoustic_vd or vti; `nsrc` > 1 makes encoded
shots; `keep_b` stores that many checkpoint segments in place of recomputing.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2604_14189_amd as sw
from paper_2604_14189_amd.mlp import MLPVelocity

PHYSICS = {"acoustic": sw.ACOUSTIC, "elastic": sw.ELASTIC, "acoustic_vd": sw.ACOUSTIC_VD,
           "vti": sw.VTI}
# grid spacing, time step, peak frequency and velocity range of each physics, as
# in the package's workloads (VTI: the horizontal speed stays below 4700 m/s)
SCALES = {"acoustic": (10.0, 1e-3, 8.0, 1500.0, 4700.0),
          "elastic": (5.0, 0.5e-3, 15.0, 1800.0, 4500.0),
          "acoustic_vd": (10.0, 1e-3, 8.0, 1500.0, 4700.0),
          "vti": (10.0, 1e-3, 8.0, 1500.0, 4100.0)}


def _case(kind, physics, nx, nz, nt, shots, *, pml=40, nrec=0, nsrc=1, ckpt=50, keep_b=0, fs=0,
          models=1, name=None):
    c = {"kind": kind, "physics": physics, "nx": nx, "nz": nz, "nt": nt, "shots": shots,
         "pml": pml, "nrec": nrec or nx, "nsrc": nsrc, "ckpt": ckpt, "keep_b": keep_b, "fs": fs,
         "models": models}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # one shot over a small model: a quick look at an acquisition or a parameter,
        # and the smallest call, where launches and latency are all there is
        _case("forward", "acoustic", 200, 200, 1000, 1, pml=20, name="forward_200x200_1shot"),
        # a ragged small target with a thin pad, as the tests and quick trials use
        _case("gradient", "acoustic", 150, 77, 240, 3, pml=10, nrec=41, ckpt=17,
              name="gradient_150x77_3shots"),
        # one shot of the benchmark model: stochastic inversion, one shot a step
        _case("gradient", "acoustic", 1000, 300, 500, 1, name="gradient_1000x300_1shot"),
        # the benchmark's gradient (64 shots) over a short record, most segments stored
        _case("gradient", "acoustic", 1000, 300, 300, 64, keep_b=5,
              name="gradient_1000x300_64shots"),
        # source encoding: 64 sources in 8 supershots, every segment recomputed
        _case("gradient", "acoustic", 1000, 300, 400, 8, nsrc=8, name="encoded_1000x300_8x8"),
        # linearised modelling, the forward half of a least-squares migration iteration
        _case("born", "acoustic", 1000, 300, 300, 32, name="born_1000x300_32shots"),
        # eight uneven models advanced together (325x225 ... 1200x400)
        _case("batch", "acoustic", 1200, 400, 150, 24, models=8, name="batch_8_uneven"),
        # elastic inversion under a free surface
        _case("gradient", "elastic", 600, 300, 300, 32, pml=30, fs=1, keep_b=3,
              name="elastic_600x300_32shots"),
        # elastic modelling of a small model, padded on all sides
        _case("forward", "elastic", 90, 70, 400, 3, pml=10, nrec=23, ckpt=23,
              name="elastic_forward_90x70"),
        # variable-density acoustic inversion
        _case("gradient", "acoustic_vd", 1000, 300, 200, 16, name="vd_1000x300_16shots"),
        # anisotropic (VTI) inversion
        _case("gradient", "vti", 1000, 300, 150, 16, name="vti_1000x300_16shots"),
        # one training iteration of the network velocity model on the benchmark's grid
        _case("mlp", "acoustic", 1000, 300, 1, 1, name="mlp_1000x300"),
    ]


# relative time of a cell-step of each kind, used only to bound a drawn case
COST = {("forward", "acoustic"): 0.4, ("gradient", "acoustic"): 1.0, ("born", "acoustic"): 1.0,
        ("batch", "acoustic"): 1.0, ("forward", "elastic"): 1.2, ("gradient", "elastic"): 6.0,
        ("forward", "acoustic_vd"): 1.0, ("gradient", "acoustic_vd"): 4.5,
        ("forward", "vti"): 1.2, ("gradient", "vti"): 5.0}
MOST_CELL_STEPS = 6e9  # of an acoustic gradient; below the largest listed cases


def _between(rng, lo, hi):
    """A whole number between lo and hi, spread evenly over its logarithm."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind, physics = rng.choice([
        ("forward", "acoustic"), ("gradient", "acoustic"), ("gradient", "acoustic"),
        ("gradient", "acoustic"), ("born", "acoustic"), ("batch", "acoustic"),
        ("forward", "elastic"), ("gradient", "elastic"), ("gradient", "acoustic_vd"),
        ("gradient", "vti"), ("mlp", "acoustic")])
    nx, nz = _between(rng, 80, 1200), _between(rng, 60, 400)
    if kind == "mlp":
        while nx * nz > 300000:
            nx, nz = _between(rng, 80, 1200), _between(rng, 60, 400)
        return _case("mlp", "acoustic", nx, nz, 1, 1)
    pml = rng.choice([10, 20, 30, 40])
    shots, nt = _between(rng, 1, 64), _between(rng, 150, 800)
    nsrc = rng.choice([1, 1, 4, 8]) if physics == "acoustic" and kind != "batch" else 1
    fs = rng.choice([0, 1]) if physics in ("elastic", "acoustic_vd") else 0
    ckpt = rng.choice([17, 25, 50])
    models = rng.choice([2, 4, 8]) if kind == "batch" else 1
    cells = (nx + 2 * pml) * (nz + 2 * pml) * models * COST[(kind, physics)]
    while shots > 1 and cells * shots * nt > MOST_CELL_STEPS:
        shots -= 1
    while nt > 150 and cells * shots * nt > MOST_CELL_STEPS:
        nt -= 10
    keep_b = rng.choice([0, 2, (nt + ckpt - 1) // ckpt]) if kind == "gradient" else 0
    nrec = rng.choice([nx, max(1, nx // 2), max(1, nx // 7)])
    return _case(kind, physics, nx, nz, nt, shots, pml=pml, nrec=nrec, nsrc=nsrc, ckpt=ckpt,
                 keep_b=keep_b, fs=fs, models=models)


# ------------------------------------------------------------------ inputs
def _members(case):
    """The plans of a case: itself, or the uneven models of a batch."""
    if case["kind"] != "batch":
        return [case]
    out, n = [], case["models"]
    for m in range(n):
        f = (m + 1) / n
        nx = max(80, int(case["nx"] * (1 + 5 * f) / 6))
        out.append(dict(case, nx=nx, nz=max(60, int(case["nz"] * (1 + f) / 2)),
                        nt=max(100, int(case["nt"] * (3 + f) / 4)),
                        shots=max(1, int(case["shots"] * (1 + f) / 2)),
                        nrec=min(case["nrec"], nx), seed_offset=101 * m))
    return out


def _layers(nx, nz, vmin, vmax, rng):
    """Velocity growing with depth in layers, with Gaussian anomalies of 10 %."""
    top = np.sort(rng.uniform(0, nz, 7))
    v = np.linspace(vmin, vmax, 8)[np.searchsorted(top, np.arange(nz) + 0.5)][:, None]
    pert = np.zeros((nz, nx))
    for _ in range(20):
        r, cx, cz = rng.uniform(5, 30), rng.uniform(0, nx), rng.uniform(0, nz)
        gx = np.exp(-((np.arange(nx) - cx) ** 2) / (2 * r * r))
        gz = np.exp(-((np.arange(nz) - cz) ** 2) / (2 * r * r))
        pert += rng.choice([-0.1, 0.1]) * gz[:, None] * gx[None, :]
    return np.clip(v * (1 + pert), vmin, vmax)


def _model(c, rng):
    """[nparam][nz][nx] of the case's physics (float32)."""
    _, _, _, vmin, vmax = SCALES[c["physics"]]
    vp = _layers(c["nx"], c["nz"], vmin, vmax, rng)
    if c["physics"] == "acoustic":
        m = vp[None]
    elif c["physics"] == "elastic":
        m = np.stack([vp, vp / 1.73 * (1 + rng.uniform(-0.05, 0.05, vp.shape)),
                      310.0 * vp ** 0.25])
    elif c["physics"] == "acoustic_vd":
        m = np.stack([vp, 310.0 * vp ** 0.25])
    else:  # eta 0 in the top rows, where sources and receivers sit
        ramp = np.clip((np.arange(c["nz"])[:, None] - 20) / 40.0, 0.0, 1.0)
        m = np.stack([vp, 1.02 * vp, 0.12 * ramp * np.ones_like(vp)])
    return m.astype(np.float32)


def _problem(c, seed):
    """Everything of one plan that is made on the host."""
    rng = np.random.default_rng([seed, c.get("seed_offset", 0)])
    h, dt, f0, _, vmax = SCALES[c["physics"]]
    ns, nsrc, nt, depth = c["shots"], c["nsrc"], c["nt"], min(5, c["nz"] - 1)
    n = ns * nsrc
    xs = np.floor((np.arange(n) + 0.5) * c["nx"] / n).astype(np.int32)
    src = np.stack([xs, np.full(n, depth, np.int32)], 1)
    rx = np.floor((np.arange(c["nrec"]) + 0.5) * c["nx"] / c["nrec"]).astype(np.int32)
    rec = np.stack([rx, np.full(len(rx), depth, np.int32)], 1)
    rec = np.ascontiguousarray(np.broadcast_to(rec, (ns,) + rec.shape))
    a = (math.pi * f0 * (np.arange(nt) * dt - 1.5 / f0)) ** 2
    wav = np.broadcast_to((1 - 2 * a) * np.exp(-a), (n, nt)) * rng.uniform(0.8, 1.2, (n, 1))
    if nsrc > 1:  # sources of a supershot interleave along the line, with random signs
        src = np.ascontiguousarray(src.reshape(nsrc, ns, 2).transpose(1, 0, 2))
        wav = (wav * rng.choice([-1.0, 1.0], (n, 1))).reshape(ns, nsrc, nt)
    vmax = 4700.0 if c["physics"] == "vti" else vmax  # the fastest (horizontal) speed
    return {"h": h, "dt": dt, "f0": f0, "vmax": vmax, "src": src, "rec": rec,
            "wav": np.ascontiguousarray(wav, dtype=np.float32), "model": _model(c, rng)}


def _plan(c, p):
    return sw.Plan(nx=c["nx"], nz=c["nz"], h=p["h"], dt=p["dt"], nt=c["nt"], pml=c["pml"],
                   src_xz=p["src"], rec_xz=p["rec"], pml_vmax=p["vmax"], pml_f0=p["f0"],
                   ckpt_every=c["ckpt"], physics=PHYSICS[c["physics"]], free_surface=c["fs"])


def _observed(c, p, seed):
    """Stand-in for recorded data: noise in the band of the source, at the
    strength of the modelled data (float32, on the GPU)."""
    g = torch.Generator(device="cuda").manual_seed(seed * 7919 + c.get("seed_offset", 0) + 1)
    shape = (c["shots"], c["nt"], c["nrec"])
    if c["physics"] in ("elastic", "acoustic_vd"):
        shape += (2,)
        scale = 3e-2 * p["dt"] ** 2 / p["h"] ** 3 / 2000.0
    else:
        scale = 0.3 * p["dt"] ** 2 / p["h"] ** 2
    x = torch.randn(shape, generator=g, device="cuda")
    f = torch.fft.rfftfreq(c["nt"], d=p["dt"], device="cuda") / p["f0"]
    band = (f * f * torch.exp(1 - f * f)).view((1, -1) + (1,) * (len(shape) - 2))
    x = torch.fft.irfft(torch.fft.rfft(x, dim=1) * band, n=c["nt"], dim=1)
    return (x * (scale / x.std())).contiguous()


def _network(case, seed):
    """Frequencies, weights, Adam moments in mid-training and dJ/dv."""
    rng = np.random.default_rng(seed)
    B = rng.normal(0.0, 10.0, (64, 2)).astype(np.float32)
    shapes = [(256, 128), (256,), (256, 256), (256,), (256, 256), (256,), (256, 256), (256,),
              (256,), (1,)]
    theta = [rng.uniform(-1, 1, s) / math.sqrt(s[-1] if len(s) == 2 else 256) for s in shapes]
    theta = np.concatenate([t.ravel() for t in theta]).astype(np.float32)
    m = rng.normal(0.0, 1e-2, theta.shape).astype(np.float32)
    v2 = rng.uniform(1e-4, 1e-3, theta.shape).astype(np.float32)
    dv = _layers(case["nx"], case["nz"], -1.0, 1.0, rng)
    dv = (dv + rng.normal(0.0, 0.2, dv.shape)) * 1e-5
    return B, theta, m, v2, dv.astype(np.float32)


ADAM = {"t": 100, "lr": 1e-4, "b1": 0.9, "b2": 0.999, "eps": 1e-8}


def prepare(case, seed):
    if case["kind"] == "mlp":
        B, theta, m, v2, dv = _network(case, seed)
        net = MLPVelocity(case["nx"], case["nz"], B, theta)
        net.m.copy_(torch.from_numpy(m))
        net.v2.copy_(torch.from_numpy(v2))
        net.t = ADAM["t"]
        return {"kind": "mlp", "net": net, "dv": torch.from_numpy(dv).cuda()}
    state = {"kind": case["kind"], "plans": [], "models": [], "wavs": [], "obs": [], "d": [],
             "g": [], "r": []}
    for c in _members(case):
        p = _problem(c, seed)
        plan = _plan(c, p)
        if c["keep_b"]:
            plan.set_tuning(keep_b=c["keep_b"])
        state["plans"].append(plan)
        state["models"].append(torch.from_numpy(p["model"]).cuda())
        state["wavs"].append(torch.from_numpy(p["wav"]).cuda())
        state["d"].append(torch.empty(plan.gathers_shape(), device="cuda"))
        if c["kind"] in ("gradient", "batch"):
            state["obs"].append(_observed(c, p, seed))
            state["r"].append(torch.empty(plan.gathers_shape(), device="cuda"))
            state["g"].append(torch.empty((plan.nparam, c["nz"], c["nx"]), device="cuda"))
        if c["kind"] == "born":
            dv = 0.02 * (p["model"][0] - p["model"][0].mean())
            state["dmodel"] = torch.from_numpy(dv.astype(np.float32)).cuda()
    if case["kind"] == "batch":
        state["batch"] = sw.Batch(state["plans"])
    else:
        state["plans"][0].reserve_workspace(case["kind"] != "forward")
    return state


def run(state):
    kind = state["kind"]
    if kind == "mlp":
        net = state["net"]
        v = net.forward()
        g = net.backward(state["dv"])
        net.step(g, lr=ADAM["lr"])
        return {"v": v, "g": g, "theta": net.theta}
    plan, model, wav = state["plans"][0], state["models"][0], state["wavs"][0]
    if kind == "forward":
        return {"d": plan.forward(model, wav, out=state["d"][0])}
    if kind == "born":
        return {"d": plan.born(model, state["dmodel"], wav, out=state["d"][0])}
    if kind == "gradient":
        d = plan.forward(model, wav, save=True, out=state["d"][0])
        r, J = sw.l2_misfit(d, state["obs"][0], resid=state["r"][0])
        return {"d": d, "J": J, "g": plan.backward(r, out=state["g"][0])}
    ds = state["batch"].forward(state["models"], state["wavs"], save=True, out=state["d"])
    rs, Js = [], []
    for d, obs, buf in zip(ds, state["obs"], state["r"]):
        r, J = sw.l2_misfit(d, obs, resid=buf)
        rs.append(r)
        Js.append(J)
    return {"d": ds, "J": Js, "g": state["batch"].backward(rs, out=state["g"])}


# ------------------------------------------------------------------ work
def _padded(c):
    top = 0 if c["fs"] else c["pml"]
    return c["nx"] + 2 * c["pml"], c["nz"] + top + c["pml"]


# state planes of one cell (4-byte words) that a time step reads and writes, and
# the operations of its update; the adjoint step moves as much and adds the
# gradient's product; a gradient takes a forward and an adjoint step per step
STEP = {"acoustic": (3, 45), "elastic": (10, 100), "acoustic_vd": (6, 60), "vti": (9, 80)}


def work(case):
    if case["kind"] == "mlp":
        n = case["nx"] * case["nz"]
        weights = 128 * 256 + 3 * 256 * 256 + 256
        # forward 1, backward 2 products per weight; the features and, for the
        # backward, the four hidden layers (bf16) written and read once
        return {"flops": 6.0 * n * weights, "bytes": n * (2 * 128 + 2 * 4 * 512 + 12.0)
                + 28.0 * weights}
    total = {"bytes": 0.0, "flops": 0.0}
    for c in _members(case):
        NX, NZ = _padded(c)
        words, ops = STEP[c["physics"]]
        passes = {"forward": 1, "born": 2}.get(c["kind"], 2)
        steps = float(NX * NZ) * c["shots"] * c["nt"] * passes
        ncomp = 2 if c["physics"] in ("elastic", "acoustic_vd") else 1
        data = 4.0 * c["shots"] * c["nt"] * (c["nrec"] * ncomp * (3 if passes == 2 else 1)
                                             + c["nsrc"])
        total["bytes"] += 4 * words * steps + data
        total["flops"] += ops * steps
    return total


# ------------------------------------------------------------------ 64-bit values
# Every spatial derivative is a banded matrix applied along x (from the right) or
# z (from the left), zero outside the padded grid; gradients are torch's own
# derivatives of the time step, one checkpoint segment at a time.
F64 = {"dtype": torch.float64, "device": "cuda"}


def _band(n, taps, rows=None):
    """n x n matrix with weight w at column (row + offset) for each tap; `rows`
    replaces the taps of some rows."""
    m = np.zeros((n, n))
    for i in range(n):
        for off, w in (rows or {}).get(i, taps):
            if 0 <= i + off < n:
                m[i, i + off] += w
    return torch.from_numpy(m).cuda()


def _profile(n, lo, hi, shift, c, p):
    """C-PML coefficients a, b at the nodes i + shift of an axis of n cells."""
    x = np.arange(n) + shift
    xi = np.zeros(n)
    L = np.ones(n)
    if lo:
        xi = np.where(x < lo, (lo - x) * p["h"], xi)
        L = np.where(x < lo, lo * p["h"], L)
    if hi:
        on = (x > n - 1 - hi) & (xi == 0)
        xi = np.where(on, (x - (n - 1 - hi)) * p["h"], xi)
        L = np.where(on, hi * p["h"], L)
    xi = np.minimum(xi, L)
    d = -3.0 * p["vmax"] * math.log(1e-3) / (2 * L) * (xi / L) ** 2
    alpha = math.pi * p["f0"] * (1 - xi / L)
    b = np.exp(-(d + alpha) * p["dt"])
    a = np.where(d > 0, d / np.where(d > 0, d + alpha, 1.0) * (b - 1), 0.0)
    return torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda()


class _Exact:
    """The recurrence of one plan in 64 bits: coefficients of the model, a time
    step of the state, and what the receivers record."""

    def __init__(self, c, p):
        self.c, self.p = c, p
        self.NX, self.NZ = _padded(c)
        P, top = c["pml"], 0 if c["fs"] else c["pml"]
        at = lambda xz: torch.from_numpy(  # noqa: E731
            ((xz[..., 1] + top).astype(np.int64) * self.NX + xz[..., 0] + P)).cuda()
        self.src = at(p["src"]).view(c["shots"], -1)
        self.rec = at(p["rec"])
        self.wav = torch.from_numpy(p["wav"]).cuda().double().view(c["shots"], -1, c["nt"])
        self.ix = torch.from_numpy(np.clip(np.arange(self.NX) - P, 0, c["nx"] - 1)).cuda()
        self.iz = torch.from_numpy(np.clip(np.arange(self.NZ) - top, 0, c["nz"] - 1)).cuda()
        ax, bx = _profile(self.NX, P, P, 0.0, c, p)
        az, bz = _profile(self.NZ, top, P, 0.0, c, p)
        self.ax, self.bx, self.az, self.bz = ax, bx, az[:, None], bz[:, None]
        self.staggered = c["physics"] in ("elastic", "acoustic_vd")
        h, n = p["h"], (self.NX, self.NZ)
        if self.staggered:
            axh, bxh = _profile(self.NX, P, P, 0.5, c, p)
            azh, bzh = _profile(self.NZ, top, P, 0.5, c, p)
            self.axh, self.bxh, self.azh, self.bzh = axh, bxh, azh[:, None], bzh[:, None]
            u, w = 9 / 8, -1 / 24
            plus = [(1, u), (0, -u), (2, w), (-1, -w)]
            minus = [(0, u), (-1, -u), (1, w), (-2, -w)]
            fs = bool(c["fs"])
            self.xp = _band(n[0], plus).t().contiguous() / h
            self.xm = _band(n[0], minus).t().contiguous() / h
            # below a free surface: odd images of tzz and txz, second-order velocity rows
            self.zp_t = _band(n[1], plus, fs and {0: [(1, u + w), (0, -u), (2, w)]}) / h
            self.zm_t = _band(n[1], minus, fs and {0: [(0, 2 * u), (1, 2 * w)],
                                                   1: [(0, u), (-1, w - u), (1, w)]}) / h
            self.zp_v = _band(n[1], plus, fs and {0: [(1, 1.0), (0, -1.0)]}) / h
            self.zm_v = _band(n[1], minus, fs and {0: [], 1: [(0, 1.0), (-1, -1.0)]}) / h
        else:
            k2 = (8 / 5, -1 / 5, 8 / 315, -1 / 560)
            k1 = (4 / 5, -1 / 5, 4 / 105, -1 / 280)
            t2 = [(s * (k + 1), a) for k, a in enumerate(k2) for s in (1, -1)] + [(0, -205 / 72)]
            t1 = [(s * (k + 1), s * b) for k, b in enumerate(k1) for s in (1, -1)]
            self.d2x, self.d2z = _band(n[0], t2).t().contiguous() / h ** 2, _band(n[1], t2) / h ** 2
            self.d1x, self.d1z = _band(n[0], t1).t().contiguous() / h, _band(n[1], t1) / h

    def zero(self):
        n = 13 if self.staggered else 8 if self.c["physics"] == "vti" else 6
        return [torch.zeros((self.c["shots"], self.NZ, self.NX), **F64) for _ in range(n)]

    def coefs(self, model):
        """Coefficient planes of a model [nparam][nz][nx] in 64 bits."""
        m = model.index_select(1, self.iz).index_select(2, self.ix)
        dt = self.p["dt"]
        if self.c["physics"] == "acoustic":
            return [(m[0] * dt) ** 2]
        if self.c["physics"] == "vti":
            P, c = self.c["pml"], self.c
            inside = torch.zeros((self.NZ, self.NX), **F64)
            inside[P:P + c["nz"], P:P + c["nx"]] = 1
            vv, v, eta = m[0], m[1], m[2] * inside
            return [(1 + 2 * eta) * (v * dt) ** 2, (vv * dt) ** 2,
                    2 * eta * (v * vv) ** 2 * dt ** 2]
        fluid = self.c["physics"] == "acoustic_vd"
        vp, vs, rho = (m[0], torch.zeros_like(m[0]), m[1]) if fluid else (m[0], m[1], m[2])
        right = torch.arange(1, self.NX + 1, device="cuda").clamp(max=self.NX - 1)
        down = torch.arange(1, self.NZ + 1, device="cuda").clamp(max=self.NZ - 1)
        mu, lam = rho * vs ** 2, rho * (vp ** 2 - 2 * vs ** 2)
        bx = 2 * dt / (rho + rho.index_select(1, right))
        bz = 2 * dt / (rho + rho.index_select(0, down))
        mxz = torch.zeros_like(mu)
        if not fluid:
            r = 1 / mu
            r = r + r.index_select(1, right)
            mxz = 4 * dt / (r + r.index_select(0, down))
        l2m = lam + 2 * mu
        cxx_x, cxx_z, czz_x, czz_z = dt * l2m, dt * lam, dt * lam, dt * l2m
        if self.c["fs"]:
            low = torch.ones((self.NZ, 1), **F64)
            low[0] = 0
            cxx_x = cxx_x * low + dt * 4 * mu * (lam + mu) / l2m * (1 - low)
            cxx_z, czz_x, czz_z = cxx_z * low, czz_x * low, czz_z * low
        return [bx, bz, mxz, cxx_x, cxx_z, czz_x, czz_z]

    def inject(self, f, n, scale):
        flat = f.reshape(f.shape[0], -1)
        return flat.scatter_add(1, self.src, scale * self.wav[:, :, n]).view_as(f)

    def record(self, f):
        return f.reshape(f.shape[0], -1).gather(1, self.rec)

    def laplace(self, p1, psx, psz, zex, zez):
        psx = self.bx * psx + self.ax * (p1 @ self.d1x)
        psz = self.bz * psz + self.az * (self.d1z @ p1)
        qx, qz = p1 @ self.d2x + psx @ self.d1x, self.d2z @ p1 + self.d1z @ psz
        zex, zez = self.bx * zex + self.ax * qx, self.bz * zez + self.az * qz
        return qx + zex, qz + zez, psx, psz, zex, zez

    def step(self, st, cf, n, source=True):
        """(new state, recorded values, background bracket B) of step n."""
        p = self.p
        if not self.staggered:
            p0, p1 = st[0], st[1]
            bx, bz, psx, psz, zex, zez = self.laplace(p1, *st[2:6])
            w = (p["dt"] / p["h"]) ** 2
            if self.c["physics"] == "acoustic":
                B = bx + bz
                pn = 2 * p1 - p0 + cf[0] * B
                rest = []
            else:
                f0, f1 = st[6], st[7]
                B = None
                mixed = (self.d2z @ f1) @ self.d2x
                pn = 2 * p1 - p0 + cf[0] * bx + cf[1] * bz - cf[2] * mixed
                rest = [f1, 2 * f1 - f0 + p["dt"] ** 2 * p1]
            if source:
                pn = self.inject(pn, n, w)
            return [p1, pn, psx, psz, zex, zez] + rest, self.record(pn), B
        vx, vz, txx, tzz, txz, pa, pb, pc, pd, pe, pf, pg, ph = st
        bx, bz, mxz, cxx_x, cxx_z, czz_x, czz_z = cf
        ga, gb, gc, gd = txx @ self.xp, self.zm_t @ txz, txz @ self.xm, self.zp_t @ tzz
        pa, pb = self.bxh * pa + self.axh * ga, self.bz * pb + self.az * gb
        pc, pd = self.bx * pc + self.ax * gc, self.bzh * pd + self.azh * gd
        vx = vx + bx * (ga + pa + gb + pb)
        vz = vz + bz * (gc + pc + gd + pd)
        ge, gf, gg, gh = vx @ self.xm, self.zm_v @ vz, self.zp_v @ vx, vz @ self.xp
        pe, pf = self.bx * pe + self.ax * ge, self.bz * pf + self.az * gf
        pg, ph = self.bzh * pg + self.azh * gg, self.bxh * ph + self.axh * gh
        exx, ezz = ge + pe, gf + pf
        txx = txx + cxx_x * exx + cxx_z * ezz
        tzz = tzz + czz_x * exx + czz_z * ezz
        txz = txz + mxz * (gg + pg + gh + ph)
        w = p["dt"] / p["h"] ** 2
        txx, tzz = self.inject(txx, n, w), self.inject(tzz, n, w)
        if self.c["fs"]:
            tzz = torch.cat([torch.zeros_like(tzz[:, :1]), tzz[:, 1:]], 1)
        return ([vx, vz, txx, tzz, txz, pa, pb, pc, pd, pe, pf, pg, ph],
                torch.stack([self.record(vx), self.record(vz)], -1), None)

    def forward(self, model, every=0):
        """Gathers, and the state entering every `every`-th step."""
        cf, st, d, kept = self.coefs(model), self.zero(), [], []
        for n in range(self.c["nt"]):
            if every and n % every == 0:
                kept.append(st)
            st, r, _ = self.step(st, cf, n)
            d.append(r)
        return torch.stack(d, 1), kept

    def gradient(self, model, obs, every=20):
        nt = self.c["nt"]
        with torch.no_grad():
            d, kept = self.forward(model, every)
        resid = d - obs
        gst, gcf = self.zero(), None
        leaf = model.clone().requires_grad_()
        cf = self.coefs(leaf)
        for k in range(len(kept) - 1, -1, -1):
            start = [x.requires_grad_() for x in kept.pop()]
            cl = [x.detach().clone().requires_grad_() for x in cf]
            st, loss = start, 0.0
            for n in range(k * every, min(nt, (k + 1) * every)):
                st, r, _ = self.step(st, cl, n)
                loss = loss + (r * resid[:, n]).sum()
            loss = loss + sum((a * b).sum() for a, b in zip(st, gst))
            got = torch.autograd.grad(loss, start + cl, allow_unused=True)
            gst = [torch.zeros_like(x) if g is None else g for x, g in zip(start, got)]
            gc = [torch.zeros_like(x) if g is None else g
                  for x, g in zip(cl, got[len(start):])]
            gcf = gc if gcf is None else [a + b for a, b in zip(gcf, gc)]
        on = [(x, g) for x, g in zip(cf, gcf) if x.requires_grad]
        g, = torch.autograd.grad([x for x, _ in on], leaf, [g for _, g in on])
        return {"d": d, "J": 0.5 * (resid * resid).sum(), "g": g}

    def born(self, model, dmodel):
        dt = self.p["dt"]
        with torch.no_grad():
            cf = self.coefs(model)
            m, dm = (x.index_select(1, self.iz).index_select(2, self.ix)
                     for x in (model, dmodel[None]))
            dC = 2 * m[0] * dm[0] * dt ** 2
            st, ds, d = self.zero(), self.zero(), []
            for n in range(self.c["nt"]):
                st, _, B = self.step(st, cf, n)
                ds, _, _ = self.step(ds, cf, n, source=False)
                ds[1] = ds[1] + dC * B
                d.append(self.record(ds[1]))
        return {"d": torch.stack(d, 1)}


def _seconds(c):
    """Rough time of the 64-bit values of one plan."""
    NX, NZ = _padded(c)
    derivs = {"acoustic": 6, "vti": 8}.get(c["physics"], 8)
    steps = float(NX * NZ) * c["shots"] * c["nt"] * {"forward": 1, "born": 2}.get(c["kind"], 5)
    per_cell = derivs * (NX + NZ) / 3e13 + derivs * 6 * 16 / 3e12
    launches = c["nt"] * derivs * 6 * 12e-6 * (1 if c["kind"] == "forward" else 4)
    return steps * per_cell + launches


def _exact_mlp(case, seed):
    B, theta, m, v2, dv = (torch.from_numpy(x).cuda().double() for x in _network(case, seed))
    nx, nz = case["nx"], case["nz"]
    x = torch.arange(nx, **F64).repeat(nz) / max(nx - 1, 1)
    z = torch.arange(nz, **F64).repeat_interleave(nx) / max(nz - 1, 1)
    ph = 2 * math.pi * torch.stack([x, z], 1) @ B.t()
    leaf = theta.clone().requires_grad_()
    sizes = [256 * 128, 256] + [65536, 256] * 3 + [256, 1]
    w = torch.split(leaf, sizes)
    a = torch.cat([torch.cos(ph), torch.sin(ph)], 1)
    for k in range(4):
        a = torch.relu(a @ w[2 * k].view(256, -1).t() + w[2 * k + 1])
    v = 1500.0 + 3200.0 * torch.sigmoid(a @ w[8] + w[9])
    g, = torch.autograd.grad((v * dv.view(-1)).sum(), leaf)
    t, b1, b2 = ADAM["t"] + 1, ADAM["b1"], ADAM["b2"]
    m, v2 = b1 * m + (1 - b1) * g, b2 * v2 + (1 - b2) * g * g
    new = theta - ADAM["lr"] * (m / (1 - b1 ** t)) / (torch.sqrt(v2 / (1 - b2 ** t)) + ADAM["eps"])
    return {"v": v.detach().view(nz, nx), "g": g, "theta": new}


def exact(case, seed):
    if case["kind"] == "mlp":
        return _exact_mlp(case, seed)
    members = _members(case)
    if sum(_seconds(c) for c in members) > 22.0:
        return None
    out = []
    for c in members:
        p = _problem(c, seed)
        model = torch.from_numpy(p["model"]).cuda().double()
        e = _Exact(c, p)
        if c["kind"] == "forward":
            with torch.no_grad():
                out.append({"d": e.forward(model)[0]})
        elif c["kind"] == "born":
            dv = 0.02 * (p["model"][0] - p["model"][0].mean())
            out.append(e.born(model, torch.from_numpy(dv.astype(np.float32)).cuda().double()))
        else:
            out.append(e.gradient(model, _observed(c, p, seed).double()))
    if case["kind"] != "batch":
        return out[0]
    return {k: [o[k] for o in out] for k in ("d", "J", "g")}
