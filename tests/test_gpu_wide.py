"""Acoustic steps in one launch, of four-column items and of two-column ones at
the sides of sizes that are no multiples of 4 (the default tiling's path), against
the launches by tile set (a named tiling, tblock 1), bit for bit: the two do the
same operations in the same order. Grids smaller and larger than a 64 x 16 piece, ending at and next to its
edges, with no pad and with one larger than the model; encoded shots; batches;
and a call whose shots go through the steps in groups."""
import pytest
import torch

from synth import cases
from tests.test_gpu_grid import _inputs, _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,nz,pml,nsrc", [
    (64, 16, 0, 1), (68, 17, 0, 3), (60, 15, 0, 1), (4, 1, 0, 1), (4, 3, 40, 1), (44, 28, 12, 1),
    (48, 33, 4, 2), (148, 77, 20, 1), (200, 61, 40, 4), (8, 200, 12, 1), (300, 24, 8, 1),
    # not multiples of 4: two-column pieces at the sides (no four-column one between
    # them, one, some), with no pad too
    (300, 40, 10, 2), (301, 40, 9, 1), (302, 33, 9, 3), (263, 40, 0, 1), (258, 19, 0, 1),
    (170, 50, 11, 1), (1, 3, 7, 1)])
def test_bitwise(nx, nz, pml, nsrc):
    case = _inputs(nx, nz, pml, 3, nsrc, seed=nx + nz)
    for keep_b in (0, 2):
        for a, b in zip(_run(case, 2, keep_b), _run(case, 1, keep_b)):
            assert torch.equal(a, b)


@pytest.mark.parametrize("nx,ckpt", [(1000, 8), (1001, 13)])
def test_groups_bitwise(nx, ckpt):
    """35 shots of 1080 x 380 cells: two groups in the forward and the adjoint,
    three in Born modelling."""
    case = cases.random_case(7, nx=nx, nz=300, pml=40, nt=30, nshots=35, nrec=29, ckpt=ckpt)
    for keep_b in (0, 1):
        for a, b in zip(_run(case, 2, keep_b), _run(case, 1, keep_b)):
            assert torch.equal(a, b)


# ten plans of aligned sizes (two launches a step); plans that advance in parts: one
# by itself in groups of its shots, two together (one ends first), one by itself
@pytest.mark.parametrize("sizes", [
    [(44 + 4 * q, 30 + q, 4 * (q % 3), 1 + q % 2, 46) for q in range(10)],
    [(1000, 300, 40, 35, 20), (999, 300, 9, 20, 23), (200, 200, 20, 2, 30), (1000, 300, 40, 30, 30)]])
def test_batch_bitwise(sizes):
    import paper_2604_14189_amd as sw
    members = [cases.random_case(q, nx=nx, nz=nz, pml=P, nt=nt, nshots=ns, nrec=min(23, nx), ckpt=9)
               for q, (nx, nz, P, ns, nt) in enumerate(sizes)]
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
