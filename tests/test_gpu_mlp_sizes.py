"""The fused MLP kernels at the edges of their tiles (128 points a work-group,
1024 points a chunk, the two output tilings of dW) against the bf16-emulating
oracle.

The gradient is compared on the kernel's own activations and pre-activation
gradients (the same discrete bf16 and ReLU decisions), so only float32 sums
differ: a sum of K terms is within K 2^-24 of its terms' magnitudes, and the
chunks hold at most 1024 terms, so 1024 * 2^-24 = 6.1e-5 bounds the relative
error of a block without cancellation; 1e-4 is the repository's bound for it."""
import numpy as np
import pytest

import synth
from oracle import mlp as omlp
from tests.helpers import f32, rel_l2
from tests.mlp_decisions import gradient_on_decisions

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("nx,nz", [(1, 1), (127, 1), (128, 1), (129, 1), (1025, 1), (33, 97),
                                   (512, 257)])
def test_sizes(nx, nz):
    from paper_2604_14189_amd import mlp
    M = nx * nz
    B = f32(synth.rff_frequencies(seed=3))
    theta = f32(omlp.init_params(4) +
                0.01 * np.random.default_rng(5).standard_normal(omlp.n_params()))
    net = mlp.MLPVelocity(nx, nz, B, theta)
    v = net.forward().double().cpu().numpy().ravel()
    dv = f32(np.random.default_rng(6).standard_normal(M) * 1e-3)
    g = net.backward(torch.tensor(dv.reshape(nz, nx), dtype=torch.float32, device="cuda"))
    g = g.double().cpu().numpy()
    hs = [h.double().cpu().numpy() for h in net.activations()]
    dzs = [d.double().cpu().numpy() for d in net.pre_activation_grads()]
    feats = ((net.feats.view(M, 128).to(torch.int32) << 16).view(torch.float32)
             .double().cpu().numpy())
    p = omlp.unpack(theta)
    prev = feats
    for l in range(4):  # a layer from the kernel's previous one: within one bf16 rounding
        z = np.maximum(prev @ omlp.bf16(p[2 * l]).T + p[2 * l + 1], 0.0)
        assert rel_l2(hs[l], z) <= 2.0 ** -8
        prev = hs[l]
    s = 1.0 / (1.0 + np.exp(-(hs[3] @ omlp.bf16(p[8]) + p[9][0])))
    assert rel_l2(v - 1500.0, 3200.0 * s) <= 1e-5
    for l in (3, 2, 1):
        t = (dzs[l] @ omlp.bf16(p[2 * l])) * (hs[l - 1] > 0)
        assert rel_l2(dzs[l - 1], t) <= 2.0 ** -8
    gref = gradient_on_decisions(theta, [feats] + hs, s, dzs, dv)
    o = 0
    for shape in omlp.SHAPES:
        n = int(np.prod(shape))
        assert rel_l2(g[o:o + n], gref[o:o + n]) <= 1e-4
        o += n
