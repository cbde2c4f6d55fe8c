"""Several steps per launch on the tiles that large lattices get (20 to 24 rows, 16 wavefronts, up to
138 KB of LDS), cut by the last row and column, and with totals recorded every few steps."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _pair(nx, ny, **kw):
    from paper_2609_28679_amd import binding
    rng = np.random.default_rng(nx)
    rho, u = 1.0 + 0.01 * rng.standard_normal((ny, nx)), 0.03 * rng.standard_normal((2, ny, nx))
    return binding.Lattice(rho, u, tau=0.7, **kw), binding.Lattice(rho, u, tau=0.7, streaming="one", **kw)


# rows per tile at six steps per launch: 20 (float32 and float64) and 24 / 20
@pytest.mark.parametrize("nx,ny", [(1001, 515), (2999, 1501)])
@pytest.mark.parametrize("storage", ["fp32", "fp64"])
@pytest.mark.parametrize("walls", [False, True])
@pytest.mark.parametrize("force", [None, (2e-5, -1e-5)])
def test_tall_tiles_equal_single_steps(nx, ny, storage, walls, force):
    many, single = _pair(nx, ny, storage=storage, wall_y=walls, force=force)
    for n in (12, 8, 4, 13):  # launches of six, four and two steps, then 6 + 6 and a single one
        many.step(n)
        single.step(n)
        assert np.array_equal(many.populations()[0], single.populations()[0]), n
    many.close()
    single.close()


@pytest.mark.parametrize("every", [1, 2, 3, 4, 5, 6])
@pytest.mark.parametrize("streaming", ["auto", "two"])
def test_totals_every_few_steps(every, streaming):
    from paper_2609_28679_amd import binding
    rng = np.random.default_rng(every)
    rho, u = 1.0 + 0.01 * rng.standard_normal((41, 130)), 0.03 * rng.standard_normal((2, 41, 130))
    kw = dict(tau=0.7, diag_every=every)
    many = binding.Lattice(rho, u, streaming=streaming, **kw)
    single = binding.Lattice(rho, u, streaming=streaming, **kw)
    for n in (7, 6, 12, 1, 14):
        many.step(n)
        for _ in range(n):
            single.step(1)
        assert np.array_equal(many.populations()[0], single.populations()[0]), n
    assert np.array_equal(many.diag_history(), single.diag_history())
    assert len(many.diag_history()) == 40 // every
    many.close()
    single.close()
