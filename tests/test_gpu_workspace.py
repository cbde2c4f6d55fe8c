"""Caller workspaces without what only the fastest steps need: accepted, with the same results."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


# bytes that hold the populations, diagnostics scratch and the read-out fields
@pytest.mark.parametrize("kw,nx,ny,least", [
    (dict(), 64, 64, 728320),
    (dict(wall_y=True), 65, 2000, 14872320),
    (dict(storage="fp64"), 1001, 515, 59049216),
    (dict(model="ddf", storage="fp16"), 2000, 2051, 534363392),  # nothing to leave out
    (dict(model="ddf", phi=2), 2000, 2051, 769832192),
])
def test_least_workspace(monkeypatch, kw, nx, ny, least):
    import torch  # noqa: F401  (its HIP runtime is the one that the library takes)
    from paper_2609_28679_amd import binding
    rng = np.random.default_rng(nx)
    rho = 1.0 + 0.01 * rng.standard_normal((ny, nx))
    u = 0.03 * rng.standard_normal((2, ny, nx))
    T = 1.0 / rho if kw.get("model") == "ddf" else None
    lib = binding.load()
    sizes = []
    size_of = lib.lbm_workspace_size

    def capped(p, n):
        rc = size_of(p, n)
        sizes.append(n._obj.value)
        n._obj.value = least
        return rc

    full = binding.Lattice(rho, u, T, tau=0.8, diag_every=7, **kw)
    monkeypatch.setattr(lib, "lbm_workspace_size", capped)
    small = binding.Lattice(rho, u, T, tau=0.8, diag_every=7, **kw)
    monkeypatch.setattr(lib, "lbm_workspace_size", size_of)
    assert sizes[0] >= least
    full.step(23)
    small.step(23)
    for a, b in zip(full.moments(), small.moments()):
        assert a is None or np.array_equal(a, b)
    assert np.array_equal(full.populations()[0], small.populations()[0])
    # the records of other windows are sums in another order
    np.testing.assert_allclose(small.diag_history(), full.diag_history(), rtol=1e-12,
                               atol=1e-12 * rho.size)
    full.close()
    small.close()
