"""lbm_step captured into a graph: every replay takes the state on by the steps of the call."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

CASES = {
    "d2q9": ((300, 130), {}),
    "d2q9_two": ((300, 130), dict(streaming="two", wall_y=True)),
    "d3q27_two": ((20, 100, 100), dict(lattice="D3Q27", streaming="two")),
    "ddf": ((700, 1024), dict(model="ddf", tau=0.6)),
    "ddf_small": ((90, 130), dict(model="ddf", tau=0.6, phi=2)),
}


def _lattice(name):
    from paper_2609_28679_amd import binding
    shape, kw = CASES[name]
    rng = np.random.default_rng(len(name))
    rho = 1.0 + 0.01 * rng.standard_normal(shape)
    u = 0.02 * rng.standard_normal((len(shape),) + shape)
    return binding.Lattice(rho, u, 1.0 / rho if kw.get("model") else None, **kw)


@pytest.mark.parametrize("name", sorted(CASES))
@pytest.mark.parametrize("n", [2, 6, 16])
def test_replays_advance_the_state(name, n):
    import torch
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        lat, ref = _lattice(name), _lattice(name)
        lat.step(2)
        ref.step(2)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            lat.step(n)
        for k in range(4):
            g.replay()
            ref.step(n)
            work = torch.ones(1 << 16, device="cuda").cumsum(0)  # the program's own, in between
            torch.cuda.synchronize()
            assert np.array_equal(lat.populations()[0], ref.populations()[0]), k
            assert work[-1].item() == 1 << 16
        lat.close()
        ref.close()
