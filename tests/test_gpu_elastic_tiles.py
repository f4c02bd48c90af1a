"""GPU: the staggered-grid steps where their 64 x 16 tiles and four-column items
end, elastic and first-order acoustic, with and without a free surface, against
the FP64 oracle at the parity tests' tolerances: widths of every remainder of 4,
narrower than an item, a tile and one column less and more; heights likewise;
pads that end inside, at and next to a tile's edge, none, and one wider than the
model; receivers too few for the directory over tile rows, and many on one row,
on tile corners and on each other."""
import numpy as np
import pytest

import synth
from tests.helpers import f32, random_el_case, rel_l2

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SEIS_TOL = 1e-5
GRAD_TOL = 1e-4


def _dev(a):
    return torch.as_tensor(np.asarray(a, dtype=np.float32), device="cuda").contiguous()


@pytest.mark.parametrize("fluid", [False, True])
@pytest.mark.parametrize("fs", [0, 1])
@pytest.mark.parametrize("nx,nz,pml,nrec", [
    (64, 16, 0, 40), (63, 15, 0, 2), (65, 17, 0, 40), (66, 18, 0, 40), (4, 3, 0, 2),
    (3, 40, 0, 9), (2, 5, 0, 9), (44, 26, 10, 40), (47, 31, 16, 9), (45, 29, 9, 300),
    (108, 47, 10, 40), (5, 6, 33, 2), (130, 34, 3, 300)])
def test_tile_edges(orc, nx, nz, pml, nrec, fs, fluid):
    import paper_2604_14189_amd as sw
    c = random_el_case(nx + nz, fs=fs, nx=nx, nz=nz, pml=pml, nt=70, nshots=2, nrec=nrec, ckpt=27)
    rng = np.random.default_rng(nx)
    for k in range(nrec // 3):  # a row of receivers, and receivers around tile corners
        c.rec[:, -1 - k] = [rng.integers(0, nx), nz // 2]
    if nrec > 8:
        for k, (x, z) in enumerate([(63, 15), (64, 16), (64, 15), (63, 16)]):
            c.rec[:, 3 + k] = [min(max(x - pml, 0), nx - 1),
                               min(max(z - (0 if fs else pml), 0), nz - 1)]
    if fluid:
        c.model[1] = 0.0
    plan = sw.Plan(nx=nx, nz=nz, h=c.h, dt=c.dt, nt=c.nt, pml=pml, src_xz=c.src, rec_xz=c.rec,
                   pml_vmax=c.vmax, pml_f0=c.f0, pml_R=c.R, ckpt_every=c.ckpt,
                   physics=sw.ACOUSTIC_VD if fluid else sw.ELASTIC, free_surface=fs)
    planes = [0, 2] if fluid else [0, 1, 2]
    d = plan.forward(_dev(c.model[planes]), _dev(c.wav), save=True)
    resid = f32(synth.bandlimited_noise((2, c.nt, nrec, 2), 15.0, c.dt, 3))
    g = plan.backward(_dev(resid)).double().cpu().numpy()
    gref, _, dref = orc.el_gradient(c.oracle_problem(orc), c.model, c.src, c.wav, c.rec, resid,
                                    want_gathers=True)
    gref = np.asarray(gref).reshape((3, nz, nx))[planes]
    assert rel_l2(d.double().cpu().numpy(), dref) <= SEIS_TOL
    big = max(np.linalg.norm(b) for b in gref)
    assert max(np.linalg.norm(a - b) for a, b in zip(g, gref)) <= GRAD_TOL * big


@pytest.mark.parametrize("fluid", [False, True])
def test_groups_of_shots(fluid):
    """Two groups of shots (23 of 520 x 1040 cells, fields of 249 or 199 MB) give
    every shot's gathers and the sum of the shots' gradients that two calls of half
    of the shots give: the gathers bit for bit, the gradients to float32 rounding
    (their float64 sums over shots are rounded once or twice)."""
    import paper_2604_14189_amd as sw
    c = random_el_case(5, fs=0, nx=500, nz=1020, pml=10, nt=27, nshots=23, nrec=40, ckpt=9)
    if fluid:
        c.model[1] = 0.0
    model = _dev(c.model[[0, 2]] if fluid else c.model)
    outs = []
    for lo, hi in ((0, 23), (0, 12), (12, 23)):
        plan = sw.Plan(nx=c.nx, nz=c.nz, h=c.h, dt=c.dt, nt=c.nt, pml=c.pml, src_xz=c.src[lo:hi],
                       rec_xz=c.rec[lo:hi], pml_vmax=c.vmax, pml_f0=c.f0, pml_R=c.R,
                       ckpt_every=c.ckpt, physics=sw.ACOUSTIC_VD if fluid else sw.ELASTIC,
                       free_surface=0)
        d = plan.forward(model, _dev(c.wav[lo:hi]), save=True).clone()
        outs.append((d, plan.backward(torch.cos(1e3 * d).contiguous()).double().clone()))
    assert torch.equal(outs[0][0], torch.cat([outs[1][0], outs[2][0]]))
    whole, parts = outs[0][1], outs[1][1] + outs[2][1]
    eps, tiny = torch.finfo(torch.float32).eps, torch.finfo(torch.float32).tiny
    scale = torch.abs(outs[1][1]) + torch.abs(outs[2][1]) + torch.abs(whole)
    assert bool((torch.abs(whole - parts) <= eps * scale + tiny).all())
