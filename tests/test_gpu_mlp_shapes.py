"""Surrogate training and forward pass at the edges of their work split: 16 samples per wavefront
and 64 per workgroup, samples that wrap around the training set, the two forward splits."""
import numpy as np
import pytest

from oracle import mlp
from paper_2609_28679_amd import inputs

pytestmark = pytest.mark.gpu


def _data(n, seed):
    rng = np.random.default_rng(seed)
    x = rng.standard_normal((n, 12)).astype(np.float32)
    x[:, 11] = 1.5
    return x, (0.5 * rng.standard_normal((n, 9))).astype(np.float32)


@pytest.mark.parametrize("n", [1, 15, 16, 17, 63, 64, 65, 129, 513])
def test_gradient_of_any_batch(n):
    import torch
    from paper_2609_28679_amd import binding as b
    x, t = _data(n, n)
    blob = b.pack_mlp(inputs.mlp_init(4))
    tr = b.Trainer(blob)
    g = torch.full((b.MLP_NPARAM,), np.nan, dtype=torch.float32, device="cuda")
    loss = tr.grad(torch.from_numpy(x).cuda(), torch.from_numpy(t).cuda(), g)
    tr.close()
    p64 = b.unpack_mlp(blob)
    y, cache = mlp.forward(p64, x.astype(np.float64), bf16=True)
    exp = mlp.backward(p64, cache, y, t.astype(np.float64), bf16=True)
    assert loss == pytest.approx(mlp.loss(y, t.astype(np.float64)), rel=1e-3)
    # Same bfloat16 roundings on both sides, but a float32 sum may land on the other side of one:
    # such an activation is 2^-8 off, one of 64, so 5e-4 of a layer's gradient at one sample. Four
    # of them are allowed; a lost or doubled sample is 1/n >= 2e-3 at these sizes.
    for name, got, want in zip(["W1", "b1", "W2", "b2", "W3", "b3"], b.unpack_mlp(g.cpu().numpy()), exp):
        err = np.sqrt(((got - want) ** 2).sum() / (want ** 2).sum())
        assert err <= (2e-3 if n < 100 else 5e-4), (name, err)


def test_training_wraps_around_the_samples():
    import torch
    from paper_2609_28679_amd import binding as b
    x, t = _data(10, 1)
    blob = b.pack_mlp(inputs.mlp_init(5))
    X, T = torch.from_numpy(x).cuda(), torch.from_numpy(t).cuda()
    # one batch of 37 from 10 samples is samples 0..9 three times and 0..6, then on from 7
    order = np.arange(2 * 37) % 10
    small, full = b.Trainer(blob), b.Trainer(blob)
    small.train(X, T, 37, 2)
    full.train(X[order].contiguous(), T[order].contiguous(), 37, 2)
    assert np.array_equal(small.weights(), full.weights())
    small.close()
    full.close()


def test_forward_splits_agree():
    import torch
    from paper_2609_28679_amd import binding as b
    n = 4096 * 64 + 77  # above 4096 workgroups of 64 samples: 64 samples per wavefront
    x, _ = _data(n, 2)
    X = torch.from_numpy(x).cuda()
    tr = b.Trainer(b.pack_mlp(inputs.mlp_init(6)))
    whole = torch.full((n, 9), np.nan, device="cuda")
    tr.forward(X, whole)
    for a, e in ((0, 1), (1, 64), (64, 200), (200, 70000), (n - 130, n)):
        part = torch.full((e - a, 9), np.nan, device="cuda")
        tr.forward(X[a:e].contiguous(), part)
        assert torch.equal(part, whole[a:e]), (a, e)
    tr.close()
