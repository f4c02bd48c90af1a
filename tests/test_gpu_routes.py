"""Which of the acoustic kernels a call takes, and that the choice keeps every bit:
calls near the lines of the dispatch against the launches by tile set (a named
tiling, tblock 1)."""
import pytest
import torch

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
