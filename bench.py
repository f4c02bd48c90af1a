"""Benchmark: acoustic FWI gradient (forward + checkpointed adjoint) on one GPU.

    python bench.py [--gpus 1] [--steps K] [--warmup W]

Workload: the 1000x300 layered-plus-anomaly model (8 layers, 20 Gaussian
anomalies of +-10 %), dx = 10 m, dt = 1 ms, 3000 steps, 40-cell C-PML (padded
1080x380), 64 Ricker (8 Hz) shots at depth 5 and 1000 receivers per shot,
checkpoints every 50 steps. One step = forward of all 64 shots with
checkpointing, L2 misfit against observed data, and the adjoint pass that
returns the model gradient. Inputs are resident in HBM before timing starts.

Metric: fwd+adj Gcell-updates/s = 2 * shots * NX * NZ * nt / step time (padded
cells counted; recomputation is overhead, not work). Prints one JSON line.
"""
from __future__ import annotations

import argparse
import gc
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

import numpy as np  # noqa: E402

HBM_PEAK_GBS = 8000.0
WORKLOAD = "layered1000x300"
METRIC = "Gcell-updates/s fwd+adj; batched vs per-shot FWI gradient time at 1e-4 rel err"

# Traffic past L2 of the dominant kernel per launch (32 shots of 1080 x 380 cells,
# one launch for the whole grid), from rocprofv3 FETCH_SIZE and WRITE_SIZE runs of
# this benchmark, each scaled by what the same counter reads for a plain device copy
# of known size (--calibrate-copy). The counters do not tell what of it the
# last-level cache serves. Keyed by kernel class and padded cells of a launch; valid
# only while the kernel source hashes to the recorded value.
TRAFFIC = {
    ("adj_xpml", 32 * 1080 * 380): {"bytes_per_launch": 445883999, "source": "d1aff81a08f928a7"},
}


def _source_hash() -> str:
    """Hash of the one-launch kernels' source and the headers it compiles against
    (the traffic figures hold only for that code)."""
    import hashlib
    h = hashlib.sha256()
    for name in ("acoustic_wide.hip", "acoustic_two.h", "fd.h", "internal.h"):
        with open(os.path.join(ROOT, "paper_2604_14189_amd", "csrc", name), "rb") as f:
            h.update(f.read())
    return h.hexdigest()[:16]


# FP64 oracle values for one shot of the headline workload (traces and sampled
# gradient cells, written by tests/golden/make_golden.py from the oracle alone)
GOLDEN = os.path.join(ROOT, "tests", "golden", "layered1000x300_shot37.npz")


def oracle_parity(torch, plan, w, v_true, wav):
    """The timed configuration (the same plan: tiling, stored segments and
    workspace) against the stored oracle values of one shot: a forward on the
    true model and the gradient for a band-limited residual on that shot only,
    compared on complete receiver traces and 20 000 sampled gradient cells
    (relative L2), outside the timed region."""
    import synth
    if not os.path.exists(GOLDEN):
        return None
    gold = np.load(GOLDEN)
    s = int(gold["shot"])
    d = plan.forward(v_true, wav, save=True)
    tr = torch.as_tensor(gold["trace_idx"], device="cuda")
    dt_ = d[s][:, tr].double().cpu().numpy()
    resid = torch.zeros_like(d)
    resid[s] = torch.tensor(
        synth.bandlimited_noise((1, w.nt, w.nrec), w.f0, w.dt, s)[0].astype(np.float32),
        device="cuda")
    g = plan.backward(resid).double().cpu().numpy()[0]
    cells = gold["grad_cells"]

    def rel(a, b):
        return float(np.linalg.norm(a - b) / np.linalg.norm(b))

    gn = float(gold["grad_norm"])
    return {"shot": s, "traces_rel_l2": rel(dt_, gold["traces"]),
            "gradient_rel_l2": rel(g.ravel()[cells], gold["grad"]),
            "gradient_norm_rel": abs(float(np.linalg.norm(g)) - gn) / gn, "tolerance": 1e-4,
            "reference": "FP64 oracle, tests/golden/layered1000x300_shot37.npz: 8 complete "
                         "traces, 20 000 sampled gradient cells and the gradient norm"}


def calibrate_copy(nbytes=1 << 30, reps=3):
    """A plain device-to-device copy of known size, for scaling the HBM byte
    counters (run under rocprofv3 --pmc)."""
    import torch
    src = torch.ones(nbytes // 4, dtype=torch.float32, device="cuda")
    dst = torch.empty_like(src)
    for _ in range(reps):
        dst.copy_(src)
    torch.cuda.synchronize()
    print(json.dumps({"calibrate_copy_bytes_read": nbytes, "bytes_written": nbytes,
                      "reps": reps, "kernel": "torch copy_"}), flush=True)


def _cpu_model() -> str:
    try:
        with open("/proc/cpuinfo") as f:
            for line in f:
                if line.startswith("model name"):
                    return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return "unknown"


def cpu_baseline(w, nt_s=100, reps=3):
    """The FP64 oracle on the host cores, on a bounded sample of the workload,
    in the metric's unit (fwd+adj Gcell-updates/s): `cores` shots (one per host
    thread, up to 16) for `nt_s` of the steps, forward + checkpointed gradient,
    the median of `reps` runs; and the same on one thread with one shot."""
    import oracle
    from synth.cases import case_from_workload, f32
    import synth

    oracle.lib()
    cores = os.cpu_count() or 1
    try:
        cores = len(os.sched_getaffinity(0))
    except Exception:
        pass
    cores = max(1, min(cores, 16, w.nshots))
    NX, NZ = w.NX, w.NZ

    def rate(nshot, nthreads):
        shots = list(range(0, w.nshots, max(1, w.nshots // nshot)))[:nshot]
        case = case_from_workload(w, shots=shots, nt=nt_s)
        case.nt = nt_s
        pb = case.oracle_problem(oracle, nthreads=nthreads)
        resid = f32(synth.bandlimited_noise((len(shots), nt_s, w.nrec), w.f0, w.dt, 5))
        ts = []
        for _ in range(reps):
            t0 = time.perf_counter()
            oracle.ac_gradient(pb, case.v, case.src, case.wav, case.rec, resid)
            ts.append(time.perf_counter() - t0)
        t = float(np.median(ts))
        return 2.0 * len(shots) * NX * NZ * nt_s / t / 1e9, t

    v, t = rate(cores, cores)
    v1, t1 = rate(1, 1)
    return {"value": v, "unit": "Gcell-updates/s", "cores": cores, "kind": "oracle",
            "cpu": _cpu_model(), "one_thread_value": v1,
            "sample": f"{cores} of {w.nshots} shots x {nt_s} of {w.nt} steps on {cores} "
                      f"threads (one shot per thread), forward + checkpointed adjoint gradient "
                      f"(k=50), FP64, median of {reps}: {t:.2f} s; one thread, one shot: "
                      f"{t1:.2f} s"}


FIT_LOG = []  # one entry per fit_keep_b call, reported with the results
T_START = time.perf_counter()


def progress(what: str):
    """One line on stderr as each measurement ends (stdout holds only the
    result line)."""
    print(f"[bench {time.perf_counter() - T_START:7.1f} s] {what}", file=sys.stderr, flush=True)


def _free_bytes(torch):
    """Device memory a new workspace can take: what the device reports free,
    plus what torch's allocator holds cached but unused (a workspace is a
    torch tensor, so it can take a cached block; the allocator may keep a
    very large freed block rather than return it to the device)."""
    free, _ = torch.cuda.mem_get_info()
    return free + max(0, torch.cuda.memory_reserved() - torch.cuda.memory_allocated())


def fit_keep_b(torch, plan, nt, ckpt, reserve=8 << 30):
    """Use the HBM: store B'^n of as many checkpoint segments as the free
    memory holds after the rest of the workspace and `reserve` bytes for the
    gathers, residuals and temporaries, so that the backward recomputes only
    the others. The workspace is allocated here; on an allocation failure the
    count steps down. Returns the count set on the plan."""
    t = dict(plan.tuning)
    nseg = -(-nt // ckpt)

    def ws(k):  # the plan's backward workspace with k stored segments (host-side layout)
        t["keep_b"] = k
        plan.set_tuning(**t)
        return plan.workspace_bytes(True)

    plan.release_workspace()
    gc.collect()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    free = _free_bytes(torch)
    budget = free - reserve
    # a stored segment costs its B'^n planes less the checkpoint it no longer
    # needs; the first one also takes over the recomputation's B'^n buffer,
    # so the workspace grows with the count from one stored segment on: the
    # largest count that fits, by bisection
    keep = 0
    if ws(1) <= budget:
        lo, hi = 1, nseg
        while lo < hi:
            mid = (lo + hi + 1) // 2
            if ws(mid) <= budget:
                lo = mid
            else:
                hi = mid - 1
        keep = lo
    log = {"free_GiB": round(free / 2**30, 1),
           "torch_reserved_GiB": round(torch.cuda.memory_reserved() / 2**30, 1),
           "torch_allocated_GiB": round(torch.cuda.memory_allocated() / 2**30, 1),
           "first_try": keep, "failed_tries": 0}
    FIT_LOG.append(log)
    while True:
        t["keep_b"] = keep
        plan.set_tuning(**t)
        try:
            plan.reserve_workspace(True)
            log["keep_b"] = keep
            return keep
        except torch.OutOfMemoryError:
            plan.release_workspace()
            torch.cuda.empty_cache()
            log["failed_tries"] += 1
            if keep == 0:
                raise
            keep = max(0, keep - 2)


def fit_batch_keep_b(torch, batch, plans, nsegs, reserve=8 << 30):
    """Stored segments for a batch: every plan stores the same fraction of its
    checkpoint segments (rounded down), the largest fraction whose workspace
    leaves `reserve` bytes of the free memory. The workspace is allocated
    here; on an allocation failure the fraction steps down. Returns the
    per-plan counts."""
    tun = [dict(p.tuning) for p in plans]

    def ws_at(f):
        for p, t, ns in zip(plans, tun, nsegs):
            t["keep_b"] = int(f * ns)
            p.set_tuning(**t)
        return batch.workspace_bytes(True)

    batch._work = None
    gc.collect()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    free = _free_bytes(torch)
    lo, hi = 0.0, 1.0
    if ws_at(1.0) <= free - reserve:
        lo = 1.0
    else:
        for _ in range(30):
            mid = 0.5 * (lo + hi)
            lo, hi = (mid, hi) if ws_at(mid) <= free - reserve else (lo, mid)
    log = {"batch": True, "free_GiB": round(free / 2**30, 1), "first_fraction": round(lo, 4),
           "failed_tries": 0}
    FIT_LOG.append(log)
    f = lo
    while True:
        need = ws_at(f)
        try:
            batch._work = torch.empty(need, dtype=torch.uint8, device="cuda")
            break
        except torch.OutOfMemoryError:
            batch._work = None
            torch.cuda.empty_cache()
            log["failed_tries"] += 1
            if f == 0.0:
                raise
            f = max(0.0, f - 0.05)
    log["keep_b"] = [p.tuning["keep_b"] for p in plans]
    return log["keep_b"]


def per_shot_compare(sw, torch, w, v0, wav, d_obs, nsample, tuning, t_batched):
    """The same FWI gradient through the per-shot path: one single-shot plan
    per shot, its kernels launched once per shot per step (no batching, no
    graph), timed on `nsample` shots spread over the line and scaled to all
    shots. A single shot's B'^n planes fit in HBM many times over, so each
    single-shot plan stores them for all its segments. Also checks that the
    per-shot gradients sum to the batched gradient of the same shots."""
    from synth.cases import case_from_workload
    shots = sorted(set(np.linspace(0, w.nshots - 1, nsample).round().astype(int).tolist()))
    cs = case_from_workload(w, shots=shots)
    bp = cs.plan()
    bp.set_tuning(*tuning)
    idx = torch.tensor(shots, device=wav.device)
    d = bp.forward(v0, wav[idx].contiguous(), save=True)
    r, _ = sw.l2_misfit(d, d_obs[idx].contiguous())
    g_batch = bp.backward(r).double()
    bp.release_workspace()
    del bp
    nseg = -(-w.nt // w.ckpt_every)

    def one(s):
        p1 = case_from_workload(w, shots=[s]).plan()
        p1.set_tuning(*tuning, keep_b=nseg)
        d = p1.forward(v0, wav[s:s + 1], save=True)
        r, _ = sw.l2_misfit(d, d_obs[s:s + 1])
        g = p1.backward(r)
        p1.release_workspace()
        return g

    one(shots[0])  # warm-up: kernels loaded, workspace block cached
    torch.cuda.synchronize()
    g_sum = torch.zeros_like(g_batch)
    t0 = time.perf_counter()
    for s in shots:
        g_sum += one(s).double()
    torch.cuda.synchronize()
    t = (time.perf_counter() - t0) / len(shots)
    err = float(torch.linalg.norm(g_sum - g_batch) / torch.linalg.norm(g_batch))
    est = t * w.nshots
    return {"shots_timed": len(shots), "s_per_shot": round(t, 4),
            "per_shot_gradient_s": round(est, 3), "batched_gradient_s": round(t_batched, 3),
            "speedup": round(est / t_batched, 2), "grad_rel_err_vs_batched": err}


def _sync_time(torch, fn):
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    out = fn()
    torch.cuda.synchronize()
    return out, time.perf_counter() - t0


def _median_time(torch, fn, reps=3):
    """(last output, median seconds, all samples) of `reps` timed calls."""
    ts, out = [], None
    for _ in range(reps):
        out, t = _sync_time(torch, fn)
        ts.append(t)
    return out, float(np.median(ts)), [round(x, 4) for x in ts]


def batched_uneven(sw, torch, tuning=None):
    """The eight uneven layered models (200x200 ... 1200x400, 16-48 shots, 2000-4000
    steps, 256 shots): one FWI gradient of all of them through one Batch (one
    launch per kernel kind and step for every model) against the per-shot path
    (single-shot plans, kernels launched once per shot per step), timed on the
    middle shot of each model and scaled by its shot count. The tiling and
    time-blocking depth come from the batch autotuner (before timing) unless
    `tuning` (rz, pml_rz, use_graph, tblock) is given; the per-shot plans use the
    same."""
    import synth
    from synth.cases import case_from_workload
    ws = synth.batched_workloads()
    plans, v0s, wavs, dobs = [], [], [], []
    for w in ws:
        case = case_from_workload(w)
        p = case.plan()
        if tuning is not None:
            p.set_tuning(*tuning)
        wav = torch.tensor(case.wav, dtype=torch.float32, device="cuda")
        d = p.forward(torch.tensor(case.v, dtype=torch.float32, device="cuda"), wav).clone()
        p.release_workspace()
        plans.append(p)
        v0s.append(torch.tensor(synth.smooth(case.v, 20.0), dtype=torch.float32, device="cuda"))
        wavs.append(wav)
        dobs.append(d)
    batch = sw.Batch(plans)
    if tuning is None:
        ch = batch.autotune(v0s, wavs, steps=20)
        tuning = (ch["rz"], ch["pml_rz"], 0, ch["tblock"])
    # the workspace, with as many stored segments as fit, is allocated before
    # timing (inputs and state resident in HBM)
    nsegs = [-(-w.nt // w.ckpt_every) for w in ws]
    keeps = fit_batch_keep_b(torch, batch, plans, nsegs)

    # fixed gathers, residual and gradient buffers: a captured graph stays valid
    gath = [torch.empty(p.gathers_shape(), device="cuda") for p in plans]
    res = [torch.empty_like(g) for g in gath]
    grads = [torch.empty(p._model_shape(), device="cuda") for p in plans]

    def grad():
        ds = batch.forward(v0s, wavs, save=True, out=gath)
        for d, o, r in zip(ds, dobs, res):
            sw.l2_misfit(d, o, resid=r)
        return batch.backward(res, out=grads)

    grad()
    _, t_batch, t_eager_all = _median_time(torch, grad)
    g_eager = [g.clone() for g in grads]
    batch.set_graph(True)
    grad()  # capture
    _, t_graph, t_graph_all = _median_time(torch, grad)
    nodes = batch.graph_nodes()
    same = all(bool(torch.equal(a, b)) for a, b in zip(g_eager, grads))
    batch.set_graph(False)
    batch._work = None
    t_shot = 0.0
    for w, v0, wav, do, nseg in zip(ws, v0s, wavs, dobs, nsegs):
        s = w.nshots // 2
        p1 = case_from_workload(w, shots=[s]).plan()
        p1.set_tuning(*tuning, keep_b=nseg)  # one shot's planes all fit

        def one():
            d = p1.forward(v0, wav[s:s + 1], save=True)
            return p1.backward(sw.l2_misfit(d, do[s:s + 1])[0])

        _, t1 = _sync_time(torch, one)
        p1.release_workspace()
        t_shot += t1 * w.nshots
    cells = sum(2.0 * w.nshots * w.NX * w.NZ * w.nt for w in ws)
    return {"models": len(ws), "shots": sum(w.nshots for w in ws),
            "batched_gradient_s": round(t_batch, 3), "samples_s": t_eager_all,
            "batched_Gcell_per_s": round(cells / t_batch / 1e9, 2),
            "graph": {"gradient_s": round(t_graph, 3), "samples_s": t_graph_all,
                      "Gcell_per_s": round(cells / t_graph / 1e9, 2),
                      "launches_forward_graph": nodes[0], "launches_backward_graph": nodes[1],
                      "graph_launches_per_gradient": 2,
                      "bitwise_equal_to_eager": same},
            "per_shot_gradient_s_est": round(t_shot, 3), "speedup": round(t_shot / t_batch, 2),
            "tuning": {"rz": tuning[0], "pml_rz": tuning[1], "tblock": tuning[3]},
            "keep_b": keeps, "segments": nsegs,
            "per_shot_sample": "middle shot of each model, scaled by its shot count"}


# Algorithmic bytes per cell of one elastic step (interior cells; the C-PML
# memory variables of the strips come on top): forward velocity kernel 36 B
# (read txx, tzz, txz, vx, vz, bx, bz; write vx, vz) and stress kernel 44 B
# (read vx, vz, txx, tzz, txz and the coefficients cxx_x, cxx_z, mxz; write the
# stresses); the storing forward adds the five trace planes (20 B); the
# reverse kernels 76 B (stress adjoints, three coefficients, velocity adjoints,
# three traces and three gradient partials read; velocity adjoints and the
# partials written) and 64 B (velocity adjoints, bx, bz, stress adjoints, two
# traces and two partials read; stress adjoints and the partials written).
EL_STEP_BYTES = {"fwd_int": 80, "rec_int": 100, "adj_int": 140}
# The fluid kernels of the variable-density plans (vs = 0: no txz, mxz, exz or
# mu partials): forward 32 + 32 B (velocity: txx, tzz, vx, vz, bx, bz read,
# vx, vz written; stress: vx, vz, txx, tzz, cxx_x, cxx_z read, txx, tzz
# written), storing forward + four trace planes (16 B), reverse 48 + 56 B
# (stress adjoints, two coefficients, velocity adjoints, two traces and the
# lambda partial read, velocity adjoints and the partial written; velocity
# adjoints, bx, bz, stress adjoints, two traces and two partials read, stress
# adjoints and the partials written).
VD_STEP_BYTES = {"fwd_int": 64, "rec_int": 80, "adj_int": 104}


def el_step_kernels(torch, plan, grad, step_cells, step_bytes=EL_STEP_BYTES):
    """Per-step kernel times of a staggered-grid plan (velocity and stress with
    the receivers, or the two reverse kernels with the residual injection), from
    one more gradient timed every 10th launch pair, with their algorithmic GB/s.
    The library's groups of shots (fields of up to 170 MiB) are timed one by one;
    the times here are those of all the groups of a step."""
    NX, NZ = plan.padded()
    shots = step_cells // (NX * NZ)
    fit = max((170 << 20) // ((16 if step_bytes is VD_STEP_BYTES else 20) * NX * NZ), 1)
    groups = -(-shots // fit)
    groups = -(-shots // -(-shots // groups))
    plan.set_profiling(True, 10)
    grad()
    torch.cuda.synchronize()
    kt = plan.kernel_times()
    plan.set_profiling(False)
    out = {}
    for cls, nbytes in step_bytes.items():
        n, ms = kt.get(cls, (0, 0.0))
        if n:
            us = 1e3 * ms / n * groups
            out[cls] = {"steps_timed": n, "avg_us": round(us, 1), "bytes_per_cell": nbytes,
                        "algorithmic_GBps": round(nbytes * step_cells / us / 1e3, 1)}
    return out


def elastic_gradient(sw, torch, nt=0):
    """Elastic velocity-stress FWI gradient (vp, vs, rho) on the 600x300
    free-surface workload: 32 shots, 4000 steps (nt > 0: that many, for
    profiling), checkpoints every 50."""
    import synth
    from synth.cases import el_case_from_workload
    w = synth.workload("elastic600x300")
    if nt:
        w = w.replace(nt=nt)
    case = el_case_from_workload(w)
    plan = case.plan()
    wav = torch.tensor(case.wav, dtype=torch.float32, device="cuda")
    m_true = torch.tensor(case.model, dtype=torch.float32, device="cuda")
    d_obs = plan.forward(m_true, wav).clone()
    m0 = torch.tensor(np.stack([synth.smooth(c, 20.0) for c in case.model]), dtype=torch.float32,
                      device="cuda")
    keep = fit_keep_b(torch, plan, w.nt, w.ckpt_every)

    def grad():
        d = plan.forward(m0, wav, save=True)
        return plan.backward(sw.l2_misfit(d, d_obs)[0])

    grad()
    _, t, ts = _median_time(torch, grad)
    NX, NZ = plan.padded()
    cells = 2.0 * w.nshots * NX * NZ * w.nt
    kernels = el_step_kernels(torch, plan, grad, w.nshots * NX * NZ)
    plan.release_workspace()
    return {"workload": "elastic600x300", "padded": f"{NX}x{NZ}", "shots": w.nshots,
            "nt": w.nt, "keep_b": keep, "gradient_s": round(t, 3), "samples_s": ts,
            "Gcell_per_s": round(cells / t / 1e9, 2), "step_kernels": kernels}


def born_modelling(sw, torch, case, w, v_true, v0, wav):
    """Born (tangent-linear) modelling on the 1000x300 workload, all shots:
    the background (two-step passes over the deep tiles) and the perturbation
    (dv = true - smooth model; single steps) advance together; and iterations
    of least-squares RTM (fwi.LSRTM.step: Born modelling of the search
    direction, background forward with checkpoints, gradient of the residual,
    float64 inner products) on the Born data of dv."""
    plan = case.plan()
    dv = (v_true - v0).contiguous()

    def born():
        return plan.born(v0, dv, wav)

    born()
    _, t_born, tb = _median_time(torch, born)
    keep = fit_keep_b(torch, plan, w.nt, w.ckpt_every)

    from paper_2604_14189_amd import fwi
    ls = fwi.LSRTM(plan, v0, wav, plan.born(v0, dv, wav).clone())

    def lsrtm():
        return ls.step()

    lsrtm()
    _, t_it, ti = _median_time(torch, lsrtm)
    resid_rel = ls.history[-1] / ls.history[0]
    NX, NZ = plan.padded()
    plan.release_workspace()
    cells = float(w.nshots) * NX * NZ * w.nt
    return {"workload": "layered1000x300", "shots": w.nshots, "nt": w.nt,
            "born_s": round(t_born, 3), "born_samples_s": tb, "lsrtm_samples_s": ti,
            "born_Gcell_per_s": round(cells / t_born / 1e9, 2),
            "wavefield_Gcell_per_s": round(2.0 * cells / t_born / 1e9, 2),
            "lsrtm_iteration_s": round(t_it, 3), "lsrtm_keep_b": keep,
            "lsrtm_iterations": len(ls.history) - 1, "lsrtm_residual_rel": round(resid_rel, 4),
            "note": "a Born cell-step advances the background and the perturbation"}


def encoded_gradient(sw, torch, nsuper=8):
    """Source encoding on the 1000x300 layered workload: its 64 sources, with
    random signs, encoded into `nsuper` supershots of 64/nsuper sources each
    (every receiver of the line records every supershot), 3000 steps. One FWI
    gradient (observed data: the same encoding on the true model)."""
    import synth
    from synth.cases import case_from_workload
    w = synth.workload(WORKLOAD)
    case = case_from_workload(w)
    k = w.nshots // nsuper
    src = case.src.reshape(nsuper, k, 2)
    signs = np.random.default_rng(7).choice([-1.0, 1.0], size=(nsuper, k, 1))
    wav = torch.tensor((case.wav.reshape(nsuper, k, w.nt) * signs).astype(np.float32),
                       device="cuda")
    plan = sw.Plan(nx=w.nx, nz=w.nz, h=w.h, dt=w.dt, nt=w.nt, pml=w.pml, src_xz=src,
                   rec_xz=case.rec[:nsuper], pml_vmax=case.vmax, pml_f0=w.f0, pml_R=w.pml_R,
                   ckpt_every=w.ckpt_every)
    v_true = torch.tensor(case.v, dtype=torch.float32, device="cuda")
    v0 = torch.tensor(synth.smooth(case.v, 20.0), dtype=torch.float32, device="cuda")
    d_obs = plan.forward(v_true, wav).clone()
    keep = fit_keep_b(torch, plan, w.nt, w.ckpt_every)

    def grad():
        d = plan.forward(v0, wav, save=True)
        return plan.backward(sw.l2_misfit(d, d_obs)[0])

    grad()
    _, t, ts = _median_time(torch, grad)
    NX, NZ = plan.padded()
    plan.release_workspace()
    cells = 2.0 * nsuper * NX * NZ * w.nt
    return {"workload": "layered1000x300", "sources": w.nshots, "supershots": nsuper,
            "sources_per_supershot": k, "nt": w.nt, "keep_b": keep, "gradient_s": round(t, 3),
            "samples_s": ts,
            "Gcell_per_s": round(cells / t / 1e9, 2)}


def acoustic_vd_gradient(sw, torch, nt=0):
    """First-order variable-density acoustic FWI gradient (vp, rho) on the
    1000x300 layered workload (64 shots, 3000 steps (nt > 0: that many, for
    profiling), 40-cell C-PML), with rho = 310 vp^0.25: the staggered kernels'
    fluid variants (vs = 0)."""
    import synth
    w = synth.workload(WORKLOAD)
    if nt:
        w = w.replace(nt=nt)
    vp = np.asarray(w.true_model(), np.float32)
    model = torch.tensor(np.stack([vp, 310.0 * vp ** 0.25]), dtype=torch.float32, device="cuda")
    m0 = torch.tensor(np.stack([synth.smooth(c, 20.0) for c in model.cpu().numpy()]),
                      dtype=torch.float32, device="cuda")
    plan = sw.Plan(nx=w.nx, nz=w.nz, h=w.h, dt=w.dt, nt=w.nt, pml=w.pml, src_xz=w.sources(),
                   rec_xz=w.receivers(), pml_vmax=w.pml_vmax(), pml_f0=w.f0, pml_R=w.pml_R,
                   ckpt_every=w.ckpt_every, physics=sw.ACOUSTIC_VD)
    wav = torch.tensor(w.wavelets(np.float32), device="cuda")
    d_obs = plan.forward(model, wav).clone()
    keep = fit_keep_b(torch, plan, w.nt, w.ckpt_every)

    def grad():
        d = plan.forward(m0, wav, save=True)
        return plan.backward(sw.l2_misfit(d, d_obs)[0])

    grad()
    _, t, ts = _median_time(torch, grad)
    NX, NZ = plan.padded()
    kernels = el_step_kernels(torch, plan, grad, w.nshots * NX * NZ, VD_STEP_BYTES)
    plan.release_workspace()
    cells = 2.0 * w.nshots * NX * NZ * w.nt
    return {"workload": "layered1000x300, rho = 310 vp^0.25", "shots": w.nshots, "nt": w.nt,
            "keep_b": keep, "gradient_s": round(t, 3), "samples_s": ts,
            "Gcell_per_s": round(cells / t / 1e9, 2), "step_kernels": kernels}


def vti_gradient(sw, torch, nt=0):
    """Pseudo-acoustic VTI FWI gradient (vv, v, eta) on the 1000x300 grid with
    the layered benchmark's shots and receivers (64 shots, 3000 steps (nt > 0:
    that many, for profiling), 40-cell C-PML), eta up to 0.12 below an
    isotropic top zone; initial model the 20-cell smoothing of the true one.
    Checkpoints every 50 steps; the saving forward stores the traces of as
    many of the last segments as the free HBM holds, the backward recomputes
    the others."""
    import synth
    w = synth.workload("vti1000x300")
    if nt:
        w = w.replace(nt=nt)
    m_true = np.asarray(w.true_model(), np.float32)
    model = torch.tensor(m_true, device="cuda")
    m0 = torch.tensor(np.stack([synth.smooth(c, 20.0) for c in m_true]).astype(np.float32),
                      device="cuda")
    plan = sw.Plan(nx=w.nx, nz=w.nz, h=w.h, dt=w.dt, nt=w.nt, pml=w.pml, src_xz=w.sources(),
                   rec_xz=w.receivers(), pml_vmax=w.pml_vmax(), pml_f0=w.f0, pml_R=w.pml_R,
                   ckpt_every=w.ckpt_every, physics=sw.VTI)
    wav = torch.tensor(w.wavelets(np.float32), device="cuda")
    d_obs = plan.forward(model, wav).clone()
    keep = fit_keep_b(torch, plan, w.nt, w.ckpt_every)

    def grad():
        d = plan.forward(m0, wav, save=True)
        return plan.backward(sw.l2_misfit(d, d_obs)[0])

    grad()
    plan.set_profiling(True, 10)
    _, t, ts = _median_time(torch, grad)
    kt = plan.kernel_times()
    plan.set_profiling(False)
    NX, NZ = plan.padded()
    plan.release_workspace()
    cells = 2.0 * w.nshots * NX * NZ * w.nt
    per = w.nshots * NX * NZ
    # algorithmic bytes per cell-update: forward reads cx, cz, cm (4 B each),
    # P^{n-1} and G^{n-1} (8 B each, float64), P^n and G^n (8 each) once, and
    # writes P^{n+1} and G^{n+1} (8 each): 60 B; the recompute also writes
    # Bx', Bz', D2x'D2z'G (+12 B); the adjoint reads lambda^{n+1},
    # lambda^{n+2} (8 B), mu^{n+1}, mu^{n+2} (16, float64), cx, cz, cm (12),
    # the three traces (12) and the partials g (12, written only on a
    # segment's first step), and writes lambda^n (4), mu^n (8) and g (12): 84 B
    kb = {"fwd_int": 60.0, "rec_int": 72.0, "adj_int": 84.0}
    kern = {}
    for name, b in kb.items():
        n, ms = kt[name]
        if n:
            avg = ms / n / 1e3
            kern[name] = {"avg_us": round(avg * 1e6, 1),
                          "algorithmic_GBps": round(b * per / avg / 1e9, 1)}
    return {"workload": "vti1000x300", "padded": f"{NX}x{NZ}", "shots": w.nshots, "nt": w.nt,
            "keep_b": keep, "gradient_s": round(t, 3), "samples_s": ts, "Gcell_per_s": round(cells / t / 1e9, 2),
            "kernels": kern}


def mlp_throughput(torch):
    """MLP velocity model at 300,000 points: forward, backward and Adam step
    (bf16 MFMA, float32 accumulation)."""
    import synth
    from paper_2604_14189_amd.mlp import MLPVelocity
    rng = np.random.default_rng(0)
    P = 230657
    theta = (rng.uniform(-1, 1, P) * 0.06).astype(np.float32)
    net = MLPVelocity(1000, 300, synth.rff_frequencies(seed=0), theta)
    dv = torch.full((300, 1000), 1e-3, device="cuda")
    for _ in range(3):
        net.forward()
        net.step(net.backward(dv))
    reps = 20
    _, tf = _sync_time(torch, lambda: [net.forward() for _ in range(reps)])
    _, tb = _sync_time(torch, lambda: [net.backward(dv) for _ in range(reps)])
    g = net.backward(dv)
    _, ta = _sync_time(torch, lambda: [net.step(g) for _ in range(reps)])
    M = 300000
    f_fwd = 2.0 * M * (128 * 256 + 3 * 256 * 256 + 256)
    f_bwd = 2.0 * M * (128 * 256 + 3 * 256 * 256 + 256) + 2.0 * M * 3 * 256 * 256
    return {"points": M, "forward_ms": round(tf / reps * 1e3, 3),
            "backward_ms": round(tb / reps * 1e3, 3), "adam_ms": round(ta / reps * 1e3, 3),
            "forward_TFLOPs": round(f_fwd / (tf / reps) / 1e12, 1),
            "backward_TFLOPs": round(f_bwd / (tb / reps) / 1e12, 1)}


# padded cells of a group of shots (kGroupCells of the library)
GROUP_CELLS = 13600000


def kernel_report(plan, w, kt):
    """Per-class kernel figures of an acoustic gradient and the roofline of the
    dominant class (the most time per gradient), from the plan's sampled HIP
    event timings `kt` ({class: (launches, total ms)})."""
    NX, NZ = plan.padded()
    # Algorithmic bytes per cell-update: interior kernel forward 16 B (read
    # p^n, p^{n-1}, Cs; write p^{n+1}), recompute 20 B (+ write B^n), adjoint
    # 28 B (read lambda^{n+1}, lambda^{n+2}, Cs, B^n, g; write lambda^n, g),
    # 24 B on the first step of a segment (g written, not read). The C-PML
    # kernels move the same per cell plus 16 B per C-PML axis at each strip cell
    # (psi and zeta read and written). A two-step pass over a deep cell moves
    # 20 B forward (read p^n, p^{n-1}, Cs; write p^{n+1}, p^{n+2}), 28 B in the
    # recompute (+ B^n, B^{n+1}) and 36 B adjoint (read lambda^{n+1},
    # lambda^{n+2}, Cs, B^n, B^{n-1}, g; write lambda^n, lambda^{n-1}, g), 32 B
    # on a segment's first pair. Its "effective" rate counts the bytes of the
    # two single steps it replaces.
    k = w.ckpt_every
    t = plan.tiles()
    TZ = t["rows"]
    wz = (t["x1"] - t["x0"]) * 64                       # z-frame columns
    n_deep = t["deep"]
    int_cells = t["interior"] * 64 * TZ
    deep_cells = n_deep * 64 * TZ
    ring_cells = int_cells - deep_cells
    z_cells = wz * (t["z0"] * TZ + NZ - t["z1"] * TZ) if t["interior"] else 0
    x_cells = NX * NZ - int_cells - z_cells
    P = w.pml
    z_strip = 2 * P * wz if t["interior"] else 0        # z-strip cells in the z frame
    x_strip = 2 * P * NZ + 2 * P * NX - z_strip         # strip cells (per axis) in the x frame
    base = {"fwd": 16.0, "rec": 20.0, "adj": (28.0 * (k - 1) + 24.0) / k}
    pairs = k // 2
    deep_b = {"fwd": 20.0, "rec": 28.0, "adj": (36.0 * (pairs - 1) + 32.0) / max(pairs, 1)}
    per_launch, effective = {}, {}
    for ph, b in base.items():
        # single-step interior launches cover the ring tiles when two-step
        # passes run (every launch of the class in this configuration)
        per_launch[ph + "_int"] = b * (ring_cells if n_deep else int_cells) * w.nshots
        per_launch[ph + "_zpml"] = (b * z_cells + 16.0 * z_strip) * w.nshots
        per_launch[ph + "_xpml"] = (b * x_cells + 16.0 * x_strip) * w.nshots
        per_launch[ph + "_deep"] = deep_b[ph] * deep_cells * w.nshots
        effective[ph + "_deep"] = 2.0 * b * deep_cells * w.nshots
    # Steps that take one launch for the whole grid are timed as the x frame, one
    # launch for each group of shots whose fields fit the last-level cache.
    group = None
    if all(v[0] == 0 for kk, v in kt.items() if not kk.endswith("_xpml")):
        groups = -(-w.nshots // max(GROUP_CELLS // (NX * NZ), 1))
        group = -(-w.nshots // groups) * NX * NZ
        for ph, b in base.items():
            per_launch[ph + "_xpml"] = ((b * NX * NZ + 16.0 * 2 * P * (NX + NZ)) *
                                        w.nshots / groups)
    # Dominant kernel: the class with the largest time per step, its average
    # launch time (the timer samples every 10th step's launches, so sampled
    # totals are not comparable) halved for a two-step pass (one launch per
    # two steps). Every adjoint class runs on all steps of the reverse sweep,
    # so among them this orders the time per gradient; they lead it.
    runs = {kk: (0.5 if kk.endswith("_deep") else 1.0) for kk in kt}
    est = {kk: (vv[1] / vv[0]) * runs[kk] for kk, vv in kt.items() if vv[0] > 0}
    ranked = sorted(est, key=lambda kk: -est[kk])

    def roofline_of(cls):
        launches, tot_ms = kt[cls]
        avg_s = tot_ms / launches / 1e3
        # algorithmic bytes per launch: the per-cell-update figure times the
        # cell-updates one launch makes (two per cell for a two-step pass, T = 2;
        # the fraction may then exceed what the pass itself moves)
        T = 2 if cls.endswith("_deep") else 1
        bytes_per_launch = effective.get(cls, per_launch[cls])
        achieved = bytes_per_launch / avg_s / 1e9
        tr = TRAFFIC.get((cls, group))
        traffic = tr["bytes_per_launch"] if tr and tr["source"] == _source_hash() else None
        # the fields of a group of shots stay in the last-level cache from step to
        # step, B' and the gradient partial stream from HBM: `frac` is then a rate
        # against the HBM peak and no HBM utilisation
        return {"bound": "last-level cache and hbm" if group else "hbm", "achieved": round(achieved, 1), "peak": HBM_PEAK_GBS,
                "unit": "GB/s", "frac": round(achieved / HBM_PEAK_GBS, 4), "traffic": traffic,
                "kernel": cls, "T": T, "avg_launch_us": round(avg_s * 1e6, 2),
                "algorithmic_bytes_per_launch": int(bytes_per_launch),
                "pass_bytes_per_launch": int(per_launch[cls]),
                "pass_frac": round(per_launch[cls] / avg_s / 1e9 / HBM_PEAK_GBS, 4)}

    roof = None
    if ranked and ranked[0] in per_launch:
        roof = roofline_of(ranked[0])
        # the adjoint two-step pass and the adjoint z-frame kernel take about
        # the same time per gradient; the runner-up is reported beside the
        # dominant class, with its time relative to it
        if len(ranked) > 1 and ranked[1] in per_launch:
            ru = roofline_of(ranked[1])
            roof["runner_up"] = {"kernel": ru["kernel"], "frac": ru["frac"], "T": ru["T"],
                                 "avg_launch_us": ru["avg_launch_us"],
                                 "time_per_gradient_vs_dominant":
                                     round(est[ranked[1]] / est[ranked[0]], 3)}
    kernels = {}
    for name, (nl, ms) in kt.items():
        if nl > 0 and name in per_launch:
            avg = ms / nl / 1e3
            kernels[name] = {"launches": nl, "total_ms": round(ms, 3),
                             "avg_us": round(avg * 1e6, 2),
                             "algorithmic_GBps": round(per_launch[name] / avg / 1e9, 1)}
            if name in effective:
                kernels[name]["effective_step_GBps"] = round(effective[name] / avg / 1e9, 1)

    return roof, kernels, t


def cell_updates_of(plan, w) -> float:
    """fwd+adj cell-updates of one gradient: 2 x shots x padded cells x steps."""
    NX, NZ = plan.padded()
    return 2.0 * w.nshots * NX * NZ * w.nt


def shots256(sw, torch, args):
    """The layered 1000x300 gradient with 256 shots (the workload's 64 shot
    positions made four times as dense): the fields of one step (four planes of
    256 x 1080 x 380) far exceed the 256 MB MALL, so the kernels stream from
    HBM. Stored segments sized as for the headline; the dominant kernel's
    roofline from sampled HIP events."""
    import synth
    from synth.cases import case_from_workload
    w = synth.workload(WORKLOAD).replace(nshots=256)
    case = case_from_workload(w)
    plan = case.plan()
    plan.set_tuning(rz=args.rz, pml_rz=args.pml_rz, tblock=args.tblock)
    v_true = torch.tensor(case.v, dtype=torch.float32, device="cuda")
    v0 = torch.tensor(synth.smooth(case.v, 20.0), dtype=torch.float32, device="cuda")
    wav = torch.tensor(case.wav, dtype=torch.float32, device="cuda")
    d_obs = plan.forward(v_true, wav).clone()
    plan.release_workspace()
    # 256 shots' gathers, residuals and the misfit's gathers take about 9 GiB
    keep = fit_keep_b(torch, plan, w.nt, w.ckpt_every, reserve=16 << 30)

    def step():
        d = plan.forward(v0, wav, save=True)
        return plan.backward(sw.l2_misfit(d, d_obs)[0])

    step()
    plan.set_profiling(True, period=10)
    _, t, ts = _median_time(torch, step, reps=2)
    kt = plan.kernel_times()
    plan.set_profiling(False)
    roof, kern, _ = kernel_report(plan, w, kt)
    plan.release_workspace()
    return {"workload": "layered1000x300, 256 shots", "shots": w.nshots, "nt": w.nt,
            "keep_b": keep, "gradient_s": round(t, 3), "samples_s": ts,
            "Gcell_per_s": round(cell_updates_of(plan, w) / t / 1e9, 2), "roofline": roof,
            "kernels": {k: v["algorithmic_GBps"] for k, v in kern.items()}}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=3)
    ap.add_argument("--warmup", type=int, default=1)
    ap.add_argument("--rz", type=int, default=8)
    ap.add_argument("--pml-rz", type=int, default=4)
    ap.add_argument("--tblock", type=int, default=2, help="steps per pass on deep interior tiles")
    ap.add_argument("--keep-b", type=int, default=-1,
                    help="checkpoint segments whose B'^n the forward stores (-1: as many as "
                         "fit in 80%% of free device memory)")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--nt", type=int, default=0, help="override the step count (testing)")
    ap.add_argument("--per-shot-sample", type=int, default=4,
                    help="shots timed through the per-shot path (0: skip)")
    ap.add_argument("--no-extras", action="store_true",
                    help="skip every measurement beside the headline gradient (the "
                         "checkpoint-recompute figure, 256 shots, Born, encoded, batched, "
                         "elastic, variable density, VTI, MLP)")
    ap.add_argument("--only", choices=["born", "encoded", "batched_uneven", "elastic",
                                       "acoustic_vd", "mlp", "vti", "shots256"],
                    help="run one of the extra measurements alone (profiling) and print it")
    ap.add_argument("--calibrate-copy", action="store_true",
                    help="only run a 1 GiB device copy (counter calibration)")
    args = ap.parse_args()
    if args.gpus != 1:
        print(json.dumps({"error": "this benchmark runs on one GPU only; partitioning "
                          "the shots over several GPUs is not implemented",
                          "n_gpus": args.gpus}))
        sys.exit(2)

    if args.calibrate_copy:
        calibrate_copy()
        return

    import torch
    import paper_2604_14189_amd as sw
    import synth
    from synth.cases import case_from_workload

    if args.only:
        if args.only == "born":
            wb = synth.workload(WORKLOAD)
            cb = case_from_workload(wb)
            vt = torch.tensor(cb.v, dtype=torch.float32, device="cuda")
            vs = torch.tensor(synth.smooth(cb.v, 20.0), dtype=torch.float32, device="cuda")
            wv = torch.tensor(cb.wav, dtype=torch.float32, device="cuda")
            res = born_modelling(sw, torch, cb, wb, vt, vs, wv)
        elif args.only == "batched_uneven":
            res = batched_uneven(sw, torch)
        elif args.only == "elastic":
            res = elastic_gradient(sw, torch, args.nt)
        elif args.only == "acoustic_vd":
            res = acoustic_vd_gradient(sw, torch, args.nt)
        elif args.only == "encoded":
            res = encoded_gradient(sw, torch)
        elif args.only == "vti":
            res = vti_gradient(sw, torch, args.nt)
        elif args.only == "shots256":
            res = shots256(sw, torch, args)
        else:
            res = mlp_throughput(torch)
        print(json.dumps({args.only: res}), flush=True)
        return

    w = synth.workload(WORKLOAD)
    if args.nt:
        w = w.replace(nt=args.nt)
    case = case_from_workload(w)
    dev = torch.device("cuda:0")
    plan = case.plan()
    plan.set_tuning(rz=args.rz, pml_rz=args.pml_rz, tblock=args.tblock)
    NX, NZ = plan.padded()
    v_true = torch.tensor(case.v, dtype=torch.float32, device=dev)
    v0 = torch.tensor(synth.smooth(case.v, 20.0), dtype=torch.float32, device=dev)
    wav = torch.tensor(case.wav, dtype=torch.float32, device=dev)
    obs_plan = case.plan()
    d_obs = obs_plan.forward(v_true, wav).clone()
    obs_plan.release_workspace()
    del obs_plan
    torch.cuda.synchronize()
    # the workspace is reserved after the inputs so that, once released, its
    # segment holds no other tensor and goes back to the device
    if args.keep_b < 0:
        keep = fit_keep_b(torch, plan, w.nt, w.ckpt_every)
    else:
        keep = args.keep_b
        plan.set_tuning(rz=args.rz, pml_rz=args.pml_rz, tblock=args.tblock, keep_b=keep)

    def step():
        d = plan.forward(v0, wav, save=True)
        resid, J = sw.l2_misfit(d, d_obs)
        g = plan.backward(resid)
        return g, J

    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    plan.set_profiling(True, period=10)  # every 10th step's launches
    t0 = time.perf_counter()
    for _ in range(args.steps):
        g, J = step()
    torch.cuda.synchronize()
    dt = (time.perf_counter() - t0) / args.steps
    kt = plan.kernel_times()
    plan.set_profiling(False)

    cell_updates = 2.0 * w.nshots * NX * NZ * w.nt
    value = cell_updates / dt / 1e9
    progress(f"headline: {args.steps} gradients, {dt:.3f} s each, {value:.1f} Gcell/s")
    parity = None
    if not args.nt:
        parity = oracle_parity(torch, plan, w, v_true, wav)
        if parity:
            progress(f"oracle parity: traces {parity['traces_rel_l2']:.2e}, "
                     f"gradient {parity['gradient_rel_l2']:.2e}")
    per_shot = None
    if args.per_shot_sample > 0:
        plan.release_workspace()
        torch.cuda.empty_cache()
        per_shot = per_shot_compare(sw, torch, w, v0, wav, d_obs, args.per_shot_sample,
                                    (args.rz, args.pml_rz, 0, args.tblock), dt)
        progress("per-shot path")

    roof, kernels, t = kernel_report(plan, w, kt)

    # the same gradient with every checkpoint segment recomputed (no stored B'^n)
    recompute = None
    if not args.nt and not args.no_extras:
        plan.release_workspace()
        torch.cuda.empty_cache()
        plan.set_tuning(keep_b=0)
        plan.reserve_workspace(True)
        step()
        _, t_rc, t_rc_all = _median_time(torch, step)
        recompute = {"keep_b": 0, "gradient_s": round(t_rc, 3), "samples_s": t_rc_all,
                     "Gcell_per_s": round(cell_updates_of(plan, w) / t_rc / 1e9, 2)}
        progress(f"checkpoint-recompute gradient {t_rc:.3f} s")

    out = {
        "metric": METRIC,
        "value": round(value, 3),
        "unit": "Gcell-updates/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(dt * 1e3, 2),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32",
        "data": "synthetic",
        "config": {"workload": WORKLOAD, "nx": w.nx, "nz": w.nz, "padded": f"{NX}x{NZ}",
                   "nt": w.nt, "shots": w.nshots, "receivers": w.nrec, "pml": w.pml,
                   "ckpt_every": w.ckpt_every, "keep_b": keep, "rz": args.rz, "pml_rz": args.pml_rz, "tblock": args.tblock, "misfit_J": float(J.item())},
        "model_grid_value": round(value * w.nx * w.nz / (NX * NZ), 3),
        "roofline": roof,
        "oracle_parity": parity,
        "per_shot": per_shot,
        "checkpoint_recompute": recompute,
        "kernels": kernels,
        "tiles": t,
    }
    if not args.no_extras and not args.nt:
        plan.release_workspace()
        del plan
        torch.cuda.empty_cache()
        out["shots256"] = shots256(sw, torch, args)
        progress("256 shots")
        torch.cuda.empty_cache()
        out["born"] = born_modelling(sw, torch, case, w, v_true, v0, wav)
        progress("born")
        torch.cuda.empty_cache()
        out["encoded"] = encoded_gradient(sw, torch)
        progress("encoded")
        torch.cuda.empty_cache()
        out["batched_uneven"] = batched_uneven(sw, torch)
        progress("batched uneven")
        torch.cuda.empty_cache()
        out["elastic"] = elastic_gradient(sw, torch)
        progress("elastic")
        torch.cuda.empty_cache()
        out["acoustic_vd"] = acoustic_vd_gradient(sw, torch)
        progress("acoustic_vd")
        torch.cuda.empty_cache()
        out["vti"] = vti_gradient(sw, torch)
        progress("vti")
        out["mlp"] = mlp_throughput(torch)
        progress("mlp")
    out["keep_b_fits"] = FIT_LOG
    if not args.no_cpu_baseline:
        out["cpu_baseline"] = cpu_baseline(w)
        progress("cpu baseline")
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
