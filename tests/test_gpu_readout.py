"""Read-outs of every staging shape (plain copy, small, medium and large chunks): the fields of
the initial equilibrium come back node for node, so a chunk out of place would show."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


# bytes of the read-out (3 float64 fields): 3 MB, 4.3 MB, 17 MB + a remainder, 300 MB + a remainder
@pytest.mark.parametrize("nx,ny", [(400, 312), (601, 300), (1013, 701), (4099, 3051)])
def test_moments_of_the_initial_state(nx, ny):
    from paper_2609_28679_amd import binding
    rng = np.random.default_rng(nx)
    rho = 1.0 + 0.05 * rng.standard_normal((ny, nx))
    u = 0.02 * rng.standard_normal((2, ny, nx))
    lat = binding.Lattice(rho, u, storage="fp64")
    for _ in range(2):  # the second call finds the staging memory
        r, v, _, totals = lat.moments()
        # float64 sums of nine populations of order one: a few ulp
        assert np.abs(r - rho).max() < 1e-14
        assert np.abs(v - u).max() < 1e-14
        assert abs(totals[0] - rho.sum()) < 1e-9 * rho.size ** 0.5
    f, _ = lat.populations()
    assert np.abs(f.sum(0) - rho).max() < 1e-14
    lat.close()


def test_readout_on_another_stream_and_thread():
    import threading

    import torch
    from paper_2609_28679_amd import binding
    rng = np.random.default_rng(1)
    rho = 1.0 + 0.05 * rng.standard_normal((2, 900, 1000))
    u = 0.02 * rng.standard_normal((2, 2, 900, 1000))
    out = [None, None]

    def work(k):
        with torch.cuda.stream(torch.cuda.Stream()):
            lat = binding.Lattice(rho[k], u[k], storage="fp64")
            out[k] = [lat.moments()[0] for _ in range(3)]
            lat.close()

    th = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    for t in th:
        t.start()
    for t in th:
        t.join()
    for k in range(2):
        for r in out[k]:
            assert np.abs(r - rho[k]).max() < 1e-14
