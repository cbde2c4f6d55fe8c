"""Contexts on streams other than torch's: the per-thread default stream, whose handle means
another queue in every thread."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

PER_THREAD = 2  # hipStreamPerThread


@pytest.mark.parametrize("nx,ny", [(601, 400), (1013, 701), (4099, 3051)])
def test_readouts_on_the_per_thread_stream(monkeypatch, nx, ny):
    """Read-outs without totals, which are what would wait for the stream first: fields and
    populations of the current state, several times over as the state goes on."""
    import torch
    from paper_2609_28679_amd import binding
    rng = np.random.default_rng(nx)
    rho = 1.0 + 0.01 * rng.standard_normal((ny, nx))
    u = 0.02 * rng.standard_normal((2, ny, nx))
    ref = binding.Lattice(rho, u, storage="fp64")
    torch.cuda.synchronize()
    monkeypatch.setattr(binding, "current_stream_handle", lambda: PER_THREAD)
    lat = binding.Lattice(rho, u, storage="fp64")
    for n in (0, 40, 7):
        lat.step(n)
        ref.step(n)
        r, v = np.empty_like(rho), np.empty_like(u)
        assert binding.load().lbm_moments(lat.ctx, binding._dptr(r), binding._dptr(v), None, None) == 0
        rr, rv, _, _ = ref.moments()
        assert np.array_equal(r, rr) and np.array_equal(v, rv), n
    if nx < 4000:
        assert np.array_equal(lat.populations()[0], ref.populations()[0])
    lat.close()
    ref.close()
