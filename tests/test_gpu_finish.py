"""GPU: the kernels that start and finish a gradient, against the FP64 oracle at
the parity tests' tolerances: the sums over the padded cells that repeat a model
cell (a wave per border cell, a thread per inner one) on models that are all
border, one cell wide or have one inner cell, with no pad and with a pad larger
than the model; and the injection of the last residuals with more receivers
than one chunk of 256, most of them coincident, within a chunk and across."""
import numpy as np
import pytest

import synth
from tests.helpers import f32, random_case, random_el_case, rel_l2

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SEIS_TOL = 1e-5
GRAD_TOL = 1e-4
SIZES = [(1, 1, 40), (1, 9, 5), (9, 1, 5), (2, 2, 3), (2, 7, 33), (3, 3, 9), (70, 4, 0),
         (33, 65, 1)]


def _dev(a):
    return torch.as_tensor(np.asarray(a, dtype=np.float32), device="cuda").contiguous()


def _check(case, plan, model, gradient, comp=()):
    d = plan.forward(_dev(model), _dev(case.wav), save=True)
    resid = f32(synth.bandlimited_noise((case.nshots, case.nt, case.nrec) + comp, 15.0, case.dt, 3))
    g = plan.backward(_dev(resid)).double().cpu().numpy()
    gref, _, dref = gradient(model, case.src, case.wav, case.rec, resid, want_gathers=True)
    gref = np.asarray(gref).reshape(g.shape)
    assert rel_l2(d.double().cpu().numpy(), dref) <= SEIS_TOL
    # against the largest plane: by symmetry, one of them is zero up to rounding
    # on a single cell
    big = max(np.linalg.norm(b) for b in gref)
    assert max(np.linalg.norm(a - b) for a, b in zip(g, gref)) <= GRAD_TOL * big


def _case(nx, nz, pml, nrec=600):
    c = random_case(nx + nz, nx=nx, nz=nz, pml=pml, nt=40, nshots=2, nrec=nrec, ckpt=16)
    c.rec[:, 3] = c.src
    return c


@pytest.mark.parametrize("nx,nz,pml", SIZES)
def test_acoustic(orc, nx, nz, pml):
    c = _case(nx, nz, pml)
    pb = c.oracle_problem(orc)
    _check(c, c.plan(), c.v, lambda *a, **k: orc.ac_gradient(pb, *a, **k))


@pytest.mark.parametrize("nx,nz,pml", SIZES)
def test_vti(orc, nx, nz, pml):
    import paper_2604_14189_amd as sw
    c = _case(nx, nz, pml)
    rng = np.random.default_rng(nx)
    c.model = f32(np.stack([c.v, 1.05 * c.v, rng.uniform(0.0, 0.1, c.v.shape)]))
    c.vmax = 4500.0
    pb = c.oracle_problem(orc)
    plan = sw.Plan(nx=nx, nz=nz, h=c.h, dt=c.dt, nt=c.nt, pml=pml, src_xz=c.src, rec_xz=c.rec,
                   pml_vmax=c.vmax, pml_f0=c.f0, pml_R=c.R, ckpt_every=c.ckpt, physics=sw.VTI)
    _check(c, plan, c.model, lambda *a, **k: orc.vti_gradient(pb, *a, **k))


@pytest.mark.parametrize("fs", [0, 1])
@pytest.mark.parametrize("nx,nz,pml", SIZES)
def test_elastic(orc, nx, nz, pml, fs):
    c = random_el_case(nx + nz, fs=fs, nx=nx, nz=nz, pml=pml, nt=60, nshots=2, nrec=300, ckpt=25)
    pb = c.oracle_problem(orc)
    _check(c, c.plan(), c.model, lambda *a, **k: orc.el_gradient(pb, *a, **k), (2,))
