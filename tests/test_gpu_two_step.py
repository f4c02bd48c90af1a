"""Two-step passes over the deep tiles under tilings that still take them (the
default one takes one launch for the whole grid): the bits of single steps, and the
passes did run (their kernel class has launches)."""
import numpy as np
import pytest

import synth
from tests.helpers import case_from_workload, f32

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _dev(a):
    return torch.as_tensor(np.asarray(a, dtype=np.float32), device="cuda").contiguous()


def _plan(case, **tuning):
    plan = case.plan()
    plan.set_tuning(**tuning)
    plan.set_profiling(True)
    return plan


def _launches(plan):
    torch.cuda.synchronize()
    return {k: n for k, (n, _) in plan.kernel_times().items()}


@pytest.mark.parametrize("rz,prz", [(4, 4), (8, 2)])
def test_born_background_bitwise(rz, prz):
    """The background in two-step passes (an odd number of steps: one single step at
    the end), the perturbation in single steps."""
    case = case_from_workload(synth.batched_workloads()[1], shots=[0, 7], nt=121)
    v, wav = _dev(case.v), _dev(case.wav)
    rng = np.random.default_rng(9)
    dv = _dev(f32(20.0 * rng.standard_normal((case.nz, case.nx))))
    out = []
    for tblock in (1, 2):
        plan = _plan(case, rz=rz, pml_rz=prz, tblock=tblock)
        out.append(plan.born(v, dv, wav).clone())
        assert _launches(plan)["fwd_deep"] == (case.nt // 2 if tblock == 2 else 0)
    assert torch.any(out[0] != 0)
    assert torch.equal(out[0], out[1])
    assert torch.equal(case.plan().born(v, dv, wav), out[0])


@pytest.mark.parametrize("rz,prz,ckpt", [(8, 2, 17), (8, 8, 50), (4, 2, 17)])
def test_gradient_bitwise(rz, prz, ckpt):
    """Segments of odd and even length, forward, recomputation and reverse."""
    case = case_from_workload(synth.workload("interface200"), nt=130)
    case.ckpt = ckpt
    v, wav = _dev(case.v), _dev(case.wav)
    r = _dev(synth.bandlimited_noise((case.nshots, case.nt, case.nrec), 10.0, case.dt, 5))
    out = []
    for tblock in (1, 2):
        plan = _plan(case, rz=rz, pml_rz=prz, tblock=tblock)
        out.append((plan.forward(v, wav, save=True).clone(), plan.backward(r).clone()))
        n = _launches(plan)
        for kind in ("fwd_deep", "rec_deep", "adj_deep"):
            assert (n[kind] > 0) == (tblock == 2), kind
    for a, b in zip(*out):
        assert torch.equal(a, b)
    plan = case.plan()
    assert torch.equal(plan.forward(v, wav, save=True), out[0][0])
    assert torch.equal(plan.backward(r), out[0][1])
