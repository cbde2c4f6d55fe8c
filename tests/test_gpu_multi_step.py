"""Several steps per launch (isothermal D2Q9, float32 / float64 storage) against the one-step
kernels: `streaming="one"` keeps one buffer and so one step per launch. Both round every step to
the storage type after the same arithmetic, so the populations agree bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _fields(nx, ny, seed=0):
    rng = np.random.default_rng(seed)
    return 1.0 + 0.01 * rng.standard_normal((ny, nx)), 0.03 * rng.standard_normal((2, ny, nx))


# widths around the 54, 58 and 62 owned columns of six, four and two steps; heights below the
# halo, around the largest tiles (20, 24 rows) and over several tiles
SHAPES = [(1, 1), (2, 7), (53, 3), (54, 24), (55, 25), (64, 64), (58, 20), (63, 21), (109, 130),
          (300, 41), (1030, 50)]


@pytest.mark.parametrize("storage", ["fp32", "fp64"])
@pytest.mark.parametrize("walls", [False, True])
@pytest.mark.parametrize("force", [None, (2e-5, -1e-5)])
def test_multi_step_equals_single_steps(storage, walls, force):
    from paper_2609_28679_amd import binding
    for nx, ny in SHAPES:
        rho, u = _fields(nx, ny)
        kw = dict(storage=storage, wall_y=walls, force=force, tau=0.8, diag_every=25)
        many = binding.Lattice(rho, u, **kw)
        single = binding.Lattice(rho, u, streaming="one", **kw)
        # 13 = 6 + 6 + 1 (odd state of the one-buffer layout), then 1 + 6, 2, 4 and, across a
        # diagnostics entry at t = 25, 6 + 4 + 1 around it
        for n in (13, 7, 2, 11):
            many.step(n)
            single.step(n)
            a, b = many.populations()[0], single.populations()[0]
            assert np.array_equal(a, b), (nx, ny, n, float(np.abs(a - b).max()))
        for p, q in zip(many.moments(), single.moments()):
            assert p is None or np.array_equal(p, q), (nx, ny)
        assert np.array_equal(many.diag_history(), single.diag_history()), (nx, ny)
        many.close()
        single.close()


def test_multi_step_two_buffers():
    from paper_2609_28679_amd import binding
    rho, u = _fields(70, 33)
    for walls in (False, True):
        many = binding.Lattice(rho, u, wall_y=walls, tau=0.6, streaming="two")
        single = binding.Lattice(rho, u, wall_y=walls, tau=0.6, streaming="one")
        for n in (6, 5, 9):
            many.step(n)
            single.step(n)
            assert np.array_equal(many.populations()[0], single.populations()[0])
        many.close()
        single.close()


# rows around the 9 owned ones of a tile and below its halo, columns around 64, few and odd planes
@pytest.mark.parametrize("nx,ny,nz", [(1, 1, 1), (2, 3, 1), (63, 9, 5), (64, 10, 12), (65, 19, 3),
                                      (130, 28, 7), (37, 20, 130)])
def test_d3q27_two_steps_equal_single_steps(nx, ny, nz):
    from paper_2609_28679_amd import binding
    rng = np.random.default_rng(3)
    rho = 1.0 + 0.01 * rng.standard_normal((nz, ny, nx))
    u = 0.03 * rng.standard_normal((3, nz, ny, nx))
    kw = dict(lattice="D3Q27", tau=0.6, streaming="two", diag_every=7)
    many, single = binding.Lattice(rho, u, **kw), binding.Lattice(rho, u, **kw)
    for n in (4, 9):  # pairs, then pairs and single steps around the entry at t = 7
        many.step(n)
        for _ in range(n):
            single.step(1)
        assert np.array_equal(many.populations()[0], single.populations()[0]), n
    assert np.array_equal(many.diag_history(), single.diag_history())
    many.set_force((1e-5, 0.0, 0.0))  # one step per launch from here on
    single.set_force((1e-5, 0.0, 0.0))
    many.step(2)
    for _ in range(2):
        single.step(1)
    assert np.array_equal(many.populations()[0], single.populations()[0])
    many.close()
    single.close()
