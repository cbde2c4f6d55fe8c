"""Surrogate training bit for bit. Adam divides by the gradient's own size, so a gradient that is
rounded another way is a visibly different network some hundred steps on: the stored gradient and
weights hold the roundings that the training kernels write out (which products of the second
layer's bias sums are fused, gelu_derivative, the two projections). They were stored from the
kernel that took 64 samples per wavefront, whose results the present one keeps."""
import os

import numpy as np
import pytest

from paper_2609_28679_amd import inputs

pytestmark = pytest.mark.gpu

GOLDEN = os.path.join(os.path.dirname(__file__), "golden", "mlp_training.npz")


def training(torch, b):
    """Gradient of 200 samples, and the weights after 200 steps of 130 samples out of 1000."""
    rng = np.random.default_rng(20)
    x = rng.standard_normal((1000, 12)).astype(np.float32)
    x[:, 11] = 1.5
    t = (0.5 * rng.standard_normal((1000, 9))).astype(np.float32)
    X, T = torch.from_numpy(x).cuda(), torch.from_numpy(t).cuda()
    tr = b.Trainer(b.pack_mlp(inputs.mlp_init(3)))
    g = torch.empty(b.MLP_NPARAM, dtype=torch.float32, device="cuda")
    loss = tr.grad(X[:200].contiguous(), T[:200].contiguous(), g)
    tr.train(X, T, 130, 200)
    w = tr.weights()
    tr.close()
    return dict(gradient=g.cpu().numpy(), loss=np.float32(loss), weights=w)


def test_gradient_and_weights_of_a_training():
    import torch
    from paper_2609_28679_amd import binding as b
    got = training(torch, b)
    with np.load(GOLDEN) as want:
        for k in want.files:
            assert np.array_equal(got[k], want[k]), (k, float(np.abs(got[k] - want[k]).max()))
