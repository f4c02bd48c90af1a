"""Acoustic steps in one launch over the whole grid (the path of the default
tiling) against the launches by tile set (a named tiling, tblock 1), bit for bit:
the two do the same operations in the same order."""
import numpy as np
import pytest
import torch

import synth
from synth import cases

pytestmark = pytest.mark.gpu


def _inputs(nx, nz, pml, nshots, nsrc, seed):
    case = cases.random_case(seed, nx=nx, nz=nz, pml=pml, nt=46, nshots=nshots,
                             nrec=min(23, nx), ckpt=10)
    if nsrc > 1:
        rng = np.random.default_rng(seed)
        case.src = np.stack([rng.integers(0, nx, (nshots, nsrc)),
                             rng.integers(0, nz, (nshots, nsrc))], 2).astype(np.int32)
        case.src[0, 1] = case.src[0, 0]          # coincident sources
        case.rec[0, 0] = case.src[0, 0]          # a receiver on a source cell
        case.wav = cases.f32(np.stack([[synth.ricker(12.0 + s + k, 46, 1e-3)
                                        for k in range(nsrc)] for s in range(nshots)]))
    return case


def _run(case, tblock, keep_b=0):
    plan = case.plan()
    plan.set_tuning(tblock=tblock, keep_b=keep_b)
    v = torch.tensor(case.v, dtype=torch.float32, device="cuda")
    wav = torch.tensor(case.wav, dtype=torch.float32, device="cuda")
    d = plan.forward(v, wav, save=True)
    r = torch.linspace(-1.0, 1.0, d.numel(), device="cuda").view(d.shape).sin().contiguous()
    g = plan.backward(r)
    if keep_b:  # Born modelling's workspace is that of a plan without stored segments
        return d, g
    return d, g, plan.born(v, (v * 0.01).contiguous(), wav)


# grids smaller and larger than a piece (64 x 8), one past its edges, odd and
# even widths and pads (an odd one makes 2-column items cross the edges), no
# pad, a pad larger than the model
@pytest.mark.parametrize("nx,nz,pml,nsrc", [
    (64, 16, 0, 1), (65, 17, 0, 1), (44, 28, 10, 1), (45, 29, 10, 1), (46, 27, 9, 1),
    (47, 30, 9, 2), (1, 1, 7, 1), (3, 5, 40, 1), (4, 4, 40, 1), (150, 77, 10, 3),
    (149, 78, 13, 1), (202, 60, 20, 4), (129, 120, 5, 1), (7, 200, 12, 1)])
def test_one_launch_steps_bitwise(nx, nz, pml, nsrc):
    case = _inputs(nx, nz, pml, 2, nsrc, seed=nx + nz)
    for keep_b in (0, 2):
        for a, b in zip(_run(case, 2, keep_b), _run(case, 1, keep_b)):
            assert torch.equal(a, b)


@pytest.mark.parametrize("odd", [False, True])
def test_one_launch_batch_bitwise(odd):
    """Batches of even plans only, and with odd ones among them (ten plans: two
    launches a step)."""
    import paper_2604_14189_amd as sw
    sizes = [(44 + 2 * q + (odd and q % 3 == 1), 30 + q, 6 + 2 * (q % 3)) for q in range(10)]
    members = [_inputs(nx, nz, P, 1 + q % 2, 1, seed=q) for q, (nx, nz, P) in enumerate(sizes)]
    plans = [m.plan() for m in members]
    batch = sw.Batch(plans)
    vs = [torch.tensor(m.v, dtype=torch.float32, device="cuda") for m in members]
    ws = [torch.tensor(m.wav, dtype=torch.float32, device="cuda") for m in members]
    ds = batch.forward(vs, ws, save=True)
    gs = batch.backward([d.clone() for d in ds])
    for m, v, w, d, g in zip(members, vs, ws, ds, gs):
        plan = m.plan()
        plan.set_tuning(tblock=1)
        d1 = plan.forward(v, w, save=True)
        assert torch.equal(d, d1)
        assert torch.equal(g, plan.backward(d1.clone()))
