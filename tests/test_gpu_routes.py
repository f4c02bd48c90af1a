"""Which of the acoustic kernels a call takes, and that the choice keeps every bit:
calls near the lines of the dispatch against the launches by tile set (a named
tiling, tblock 1)."""
import pytest
import torch

from synth import cases
from tests.test_gpu_grid import _inputs, _run

pytestmark = pytest.mark.gpu


def _batch(members):
    """Gathers and gradients of the members in one batch."""
    import paper_2604_14189_amd as sw
    plans = [m.plan() for m in members]
    vs = [torch.tensor(m.v, dtype=torch.float32, device="cuda") for m in members]
    ws = [torch.tensor(m.wav, dtype=torch.float32, device="cuda") for m in members]
    batch = sw.Batch(plans)
    ds = batch.forward(vs, ws, save=True)
    gs = batch.backward([torch.linspace(-1.0, 1.0, d.numel(), device="cuda").view(d.shape).sin()
                         .contiguous() for d in ds])
    return list(zip(ds, gs))


# a padded grid of one column (the one-launch kernels take two columns at least), and
# the narrowest that they take
@pytest.mark.parametrize("nx,nz", [(1, 1), (1, 2), (1, 5), (1, 40), (2, 1), (2, 3), (3, 2)])
def test_narrowest_grids_bitwise(nx, nz):
    case = _inputs(nx, nz, 0, 3, 1, seed=nx + nz)
    for keep_b in (0, 2):
        for a, b in zip(_run(case, 2, keep_b), _run(case, 1, keep_b)):
            assert torch.equal(a, b)


def test_narrowest_grids_in_a_batch_bitwise():
    members = [_inputs(nx, nz, pml, 2, 1, seed=nx + nz)
               for nx, nz, pml in ((1, 40, 0), (60, 30, 10), (1, 3, 0), (1, 3, 7))]
    for m, (d, g) in zip(members, _batch(members)):
        d1, g1 = _run(m, 1)[:2]
        assert torch.equal(d, d1) and torch.equal(g, g1)


def _one_launch(run, plan):
    """Whether the steps of run(plan) took one launch for the whole grid (timed as
    x-frame launches) and not one for each tile set."""
    plan.set_profiling(True)
    run(plan)
    torch.cuda.synchronize()
    n = {k: v[0] for k, v in plan.kernel_times().items()}
    plan.set_profiling(False)
    return sum(n.values()) == sum(v for k, v in n.items() if k.endswith("_xpml"))


# sizes that are not multiples of 4 on both sides of the lines in pieces of
# two-column items: 161 columns take 120 a shot on 320 rows, 162 (even) too
@pytest.mark.parametrize("nx,nshots,forward,gradient", [
    (141, 62, True, True), (141, 63, False, True), (141, 66, False, True),
    (141, 67, False, False), (142, 166, True, True), (142, 167, False, False),
    (144, 84, True, True)])
def test_lines_of_unaligned_sizes(nx, nshots, forward, gradient):
    """One launch or tile sets, and the bits of both with and without stored
    segments (Born modelling, untimed, by its bits)."""
    case = cases.random_case(3, nx=nx, nz=300, pml=10 if nx != 144 else 8, nt=8, nshots=nshots,
                             nrec=9, ckpt=3)
    v = torch.tensor(case.v, dtype=torch.float32, device="cuda")
    wav = torch.tensor(case.wav, dtype=torch.float32, device="cuda")
    r = torch.ones((case.nshots, case.nt, case.nrec), device="cuda")

    def grad(plan):
        plan.forward(v, wav, save=True)
        plan.backward(r)
    assert _one_launch(lambda p: p.forward(v, wav), case.plan()) == forward
    assert _one_launch(grad, case.plan()) == gradient
    ref = case.plan()
    ref.set_tuning(tblock=1)
    assert torch.equal(case.plan().forward(v, wav), ref.forward(v, wav))
    for keep_b in (0, 1):
        for a, b in zip(_run(case, 2, keep_b), _run(case, 1, keep_b)):
            assert torch.equal(a, b)


# narrow grids without interior tiles: 28 pieces a shot (line 1250 and 7000)
@pytest.mark.parametrize("nx,nshots", [(101, 44), (101, 45), (102, 250), (102, 251)])
def test_lines_of_narrow_sizes_bitwise(nx, nshots):
    case = cases.random_case(4, nx=nx, nz=90, pml=10, nt=9, nshots=nshots, nrec=9, ckpt=4)
    for a, b in zip(_run(case, 2), _run(case, 1)):
        assert torch.equal(a, b)


def test_batch_of_both_ways_bitwise():
    """Plans that go by tile sets together (unaligned, many shots), one of them
    between and one after plans that go alone in one launch."""
    members = [cases.random_case(q, nx=nx, nz=nz, pml=P, nt=nt, nshots=ns, nrec=9, ckpt=9)
               for q, (nx, nz, P, ns, nt) in enumerate([
                   (101, 90, 10, 50, 20), (1000, 300, 40, 33, 14), (99, 80, 9, 60, 17),
                   (1000, 300, 40, 33, 12), (87, 75, 10, 70, 23)])]
    batch = _batch(members)
    for m, (d, g) in zip(members, batch):
        d1, g1 = _run(m, 1)[:2]
        assert torch.equal(d, d1) and torch.equal(g, g1)


# staggered plans, 640 x 320 cells: a group holds the fields of 43 (fluid 54) shots, a
# modelling call goes as one with the fields and memory variables of 47 (60)
@pytest.mark.parametrize("fluid,nshots,groups", [
    (False, 44, 2), (False, 48, 2), (False, 43, 1), (True, 57, 2), (True, 63, 2), (True, 54, 1)])
def test_groups_of_staggered_calls(fluid, nshots, groups):
    """Modelling calls are split into groups of shots only where their fields and
    memory variables do not fit, saving calls where their fields do not; the gathers
    are the same bits."""
    import paper_2604_14189_amd as sw
    c = cases.random_el_case(5, fs=1, nx=600, nz=300, pml=20, nt=9, nshots=nshots, nrec=9,
                             ckpt=8)
    model = torch.tensor(c.model[[0, 2]] if fluid else c.model, dtype=torch.float32, device="cuda")
    wav = torch.tensor(c.wav, dtype=torch.float32, device="cuda")
    plan = sw.Plan(nx=c.nx, nz=c.nz, h=c.h, dt=c.dt, nt=c.nt, pml=c.pml, src_xz=c.src,
                   rec_xz=c.rec, pml_vmax=c.vmax, pml_f0=c.f0, pml_R=c.R, ckpt_every=c.ckpt,
                   physics=sw.ACOUSTIC_VD if fluid else sw.ELASTIC, free_surface=1)

    def steps(save):
        plan.set_profiling(True)
        d = plan.forward(model, wav, save=save).clone()
        torch.cuda.synchronize()
        n = plan.kernel_times()["fwd_int"][0]
        plan.set_profiling(False)
        return d, n
    d0, n0 = steps(False)
    d1, n1 = steps(True)
    assert n1 == c.nt * groups
    assert n0 == c.nt * (2 if nshots in (48, 63) else 1)
    assert torch.equal(d0, d1)


# encoded shots: fewer sources than lanes of a wave, one more, more than two waves
# hold; widths and pads of every kind of piece
@pytest.mark.parametrize("nsrc", [2, 64, 65, 130])
@pytest.mark.parametrize("nx,nz,pml", [
    (44, 28, 12), (45, 29, 10), (46, 27, 10), (300, 40, 10), (301, 17, 9), (5, 1, 3)])
def test_many_sources_bitwise(nx, nz, pml, nsrc):
    case = _inputs(nx, nz, pml, 2, nsrc, seed=nx + nz)
    case.src[1, 0] = case.src[1, nsrc - 1]   # coincident, first and last
    if nsrc > 64:
        case.src[1, 63] = case.src[1, 64]
    for a, b in zip(_run(case, 2), _run(case, 1)):
        assert torch.equal(a, b)


@pytest.mark.parametrize("nsrc,nshots,forward", [(8, 108, True), (8, 109, False), (2, 83, True),
                                                 (2, 84, False)])
def test_lines_of_encoded_shots(nsrc, nshots, forward):
    case = _inputs(141, 300, 10, nshots, nsrc, seed=3)
    v = torch.tensor(case.v, dtype=torch.float32, device="cuda")
    wav = torch.tensor(case.wav, dtype=torch.float32, device="cuda")
    assert _one_launch(lambda p: p.forward(v, wav), case.plan()) == forward
    ref = case.plan()
    ref.set_tuning(tblock=1)
    assert torch.equal(case.plan().forward(v, wav), ref.forward(v, wav))
