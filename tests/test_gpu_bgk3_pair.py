"""Isothermal D3Q27, two steps per launch, on lattices that take it: bit for bit against calls of one
step, with tiles cut by the last row and column, few and many planes, and recorded totals."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,nz", [(64, 64, 64), (100, 100, 20), (129, 50, 41), (27, 130, 90),
                                      (65, 1003, 4), (700, 9, 64), (66, 20, 200)])
def test_two_steps_equal_single_steps(nx, ny, nz):
    from paper_2609_28679_amd import binding
    rng = np.random.default_rng(nx)
    rho = 1.0 + 0.01 * rng.standard_normal((nz, ny, nx))
    u = 0.03 * rng.standard_normal((3, nz, ny, nx))
    kw = dict(lattice="D3Q27", tau=0.6, streaming="two", diag_every=7)
    many, single = binding.Lattice(rho, u, **kw), binding.Lattice(rho, u, **kw)
    for n in (4, 9, 2):
        many.step(n)
        for _ in range(n):
            single.step(1)
        assert np.array_equal(many.populations()[0], single.populations()[0]), n
    assert np.array_equal(many.diag_history(), single.diag_history())
    for force in ((1e-5, 0.0, 0.0), (0.0, 0.0, 0.0)):  # one step per launch under the force
        many.set_force(force)
        single.set_force(force)
        many.step(4)
        for _ in range(4):
            single.step(1)
        assert np.array_equal(many.populations()[0], single.populations()[0]), force
        for a, b in zip(many.moments(), single.moments()):
            assert a is None or np.array_equal(a, b)
    many.close()
    single.close()
