"""Double distribution, D2Q9: two steps per launch (lattices large enough for it) against the
one-step kernel, which calls of one step take: the same arithmetic with the state between the
steps rounded to float32 either way, so the populations agree bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

NEQ = dict(u=((-0.05, 0.0), (0.05, 0.0)), T=(0.8, 1.0))
OPTIONS = {
    "plain": {},
    "sources": dict(force=(1e-5, 2e-6), heat_source=1e-6),
    "transport": dict(prandtl=0.71, eta_over_mu=1.0),
    "vdw": dict(vdw=(0.27, 0.2)),
    "nophi": dict(phi=0),
}


def _lattice(nx, ny, option, walls, **kw):
    from paper_2609_28679_amd import binding
    rng = np.random.default_rng(0)
    y, x = np.mgrid[0:ny, 0:nx]
    u = 0.03 * np.stack([np.sin(2 * np.pi * y / ny), np.cos(2 * np.pi * x / nx)])
    u += 1e-3 * rng.standard_normal(u.shape)
    T = (1.4 if option == "vdw" else 0.9) + 0.01 * np.cos(2 * np.pi * x / nx)
    rho = np.ones_like(T) if option == "vdw" else 1.0 / T
    kw.update(OPTIONS[option])
    return binding.Lattice(rho, u, T, model="ddf", tau=0.6, wall_y=walls == "bounce",
                           neq_walls=NEQ if walls == "neq" else None, **kw)


# one column of workgroups and one column more than it, narrow and tall, wide and low, windows cut
# by the last row
@pytest.mark.parametrize("nx,ny", [(250, 2801), (251, 2803), (20, 35001), (35003, 21), (1100, 701)])
@pytest.mark.parametrize("walls", ["periodic", "bounce", "neq"])
def test_pair_equals_single_steps(nx, ny, walls):
    for option in OPTIONS:
        if walls == "neq" and option in ("sources", "vdw"):
            continue
        pair, single = _lattice(nx, ny, option, walls), _lattice(nx, ny, option, walls)
        pair.step(4)
        for _ in range(4):
            single.step(1)
        for a, b in zip(pair.populations(), single.populations()):
            assert np.array_equal(a, b), (option, float(np.abs(a - b).max()))
        pair.close()
        single.close()


def test_pair_around_diagnostics():
    pair = _lattice(1024, 700, "plain", "bounce", diag_every=5)
    single = _lattice(1024, 700, "plain", "bounce", diag_every=5)
    pair.step(13)
    for _ in range(13):
        single.step(1)
    assert np.array_equal(pair.diag_history(), single.diag_history())
    assert np.array_equal(pair.populations()[0], single.populations()[0])
    pair.close()
    single.close()
