"""Double distribution, D2Q9: windows chosen by the lattice's size."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage,phi", [("fp32", 1), ("fp32", 2), ("fp16", 1), ("fp64", 1)])
@pytest.mark.parametrize("nx,ny", [(64, 64), (253, 600), (700, 511), (1500, 1500)])
def test_small_lattice_windows_keep_the_totals(nx, ny, storage, phi):
    """Windows chosen to fill the chip: every workgroup's diagnostics record is summed once (mass
    and energy of a periodic run stay; float32 rounds the state to 6e-8 a step, unbiased)."""
    from paper_2609_28679_amd import binding
    y, x = np.mgrid[0:ny, 0:nx]
    u = np.stack([0.02 * np.sin(2 * np.pi * y / ny) + 0.05, 0.02 * np.cos(2 * np.pi * x / nx) + 0.04])
    T = 0.9 + 0.01 * np.cos(2 * np.pi * x / nx)
    lat = binding.Lattice(1.0 / T, u, T, model="ddf", tau=0.6, storage=storage, phi=phi, diag_every=1)
    lat.step(4)
    h = lat.diag_history()
    mass = (1.0 / T).sum()
    energy = (5.0 / 6.0 + 0.5 * (u ** 2).sum(0) / T).sum()
    assert h.shape[0] == 4
    assert np.abs(h[:, 1] / mass - 1.0).max() < 1e-6
    assert np.abs(h[:, 5] / energy - 1.0).max() < 1e-6
    lat.close()
