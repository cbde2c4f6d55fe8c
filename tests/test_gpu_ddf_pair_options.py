"""Double distribution, D2Q9, two steps per launch: the van der Waals fluid between NEQ walls, both
readings of their density, and sources that change between calls. As in the one-step kernel, bit
for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

OPTIONS = {
    "plain": ({}, (0.8, 1.0), 0.9),
    "transport": (dict(prandtl=0.71, eta_over_mu=1.0), (0.8, 1.0), 0.9),
    "nophi": (dict(phi=0), (0.8, 1.0), 0.9),
    "vdw": (dict(vdw=(0.27, 0.2)), (1.38, 1.45), 1.4),  # above the critical temperature of 1.2
}


def _lattice(nx, ny, T0, **kw):
    from paper_2609_28679_amd import binding
    rng = np.random.default_rng(nx)
    y, x = np.mgrid[0:ny, 0:nx]
    u = 0.03 * np.stack([np.sin(2 * np.pi * y / ny), np.cos(2 * np.pi * x / nx)])
    u += 1e-3 * rng.standard_normal(u.shape)
    T = T0 + 0.01 * np.cos(2 * np.pi * x / nx)
    rho = np.ones_like(T) if "vdw" in kw else 1.0 / T
    return binding.Lattice(rho, u, T, model="ddf", tau=0.6, **kw)


def _same(pair, single):
    for a, b in zip(pair.populations(), single.populations()):
        assert np.array_equal(a, b), float(np.abs(a - b).max())


@pytest.mark.parametrize("option", sorted(OPTIONS))
@pytest.mark.parametrize("density", ["pressure", "literal"])
@pytest.mark.parametrize("nx,ny", [(250, 2801), (499, 2003), (1100, 701)])
def test_walls_equal_single_steps(option, density, nx, ny):
    kw, wall_T, T0 = OPTIONS[option]
    walls = dict(u=((-0.05, 0.0), (0.05, 0.0)), T=wall_T, density=density)
    pair, single = (_lattice(nx, ny, T0, neq_walls=walls, **kw) for _ in range(2))
    for n in (4, 3):
        pair.step(n)
        for _ in range(n):
            single.step(1)
        _same(pair, single)
    pair.close()
    single.close()


@pytest.mark.parametrize("option", ["sources", "transport", "vdw"])
@pytest.mark.parametrize("walls", [False, True])
@pytest.mark.parametrize("nx,ny", [(1100, 1001), (200, 6001), (30001, 48)])
def test_extended_collisions_equal_single_steps(option, walls, nx, ny):
    """Lattices on which these collisions take two steps per launch."""
    kw, _, T0 = OPTIONS.get(option, (dict(force=(1e-5, 2e-6), heat_source=1e-6), None, 0.9))
    pair, single = (_lattice(nx, ny, T0, wall_y=walls, **kw) for _ in range(2))
    for n in (4, 3):
        pair.step(n)
        for _ in range(n):
            single.step(1)
        _same(pair, single)
    pair.close()
    single.close()


@pytest.mark.parametrize("walls", [False, True])
def test_sources_that_change_between_calls(walls):
    pair, single = (_lattice(1100, 1001, 0.9, wall_y=walls, diag_every=9) for _ in range(2))
    for n, force, heat in ((4, (1e-5, 2e-6), 0.0), (5, (1e-5, 2e-6), 1e-6), (6, (0.0, 0.0), 1e-6),
                           (4, (0.0, 0.0), 0.0), (1, (0.0, 1e-5), 0.0), (2, (0.0, 0.0), 0.0)):
        for lat in (pair, single):
            lat.set_force(force)
            lat.set_heat_source(heat)
        pair.step(n)
        for _ in range(n):
            single.step(1)
        _same(pair, single)
        for a, b in zip(pair.moments(), single.moments()):
            assert np.array_equal(a, b), (n, force, heat)
    assert np.array_equal(pair.diag_history(), single.diag_history())
    pair.close()
    single.close()
