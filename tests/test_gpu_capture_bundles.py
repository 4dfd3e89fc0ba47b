"""rt_build_bundles under stream capture: refused, with nothing recorded, where a field has a set at its first step;
recorded where none has."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1110_4894_amd import rt

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rt.load()


def test_bundles_under_capture():
    c, n, radius = rt.cosmology(), 64, 1e-6
    chi = rt.rt_comoving_distance(c, 0.5)
    theta = torch.from_numpy(np.random.default_rng(0).uniform(-1e-3, 1e-3, (2, n))).cuda()
    xyzm = torch.tensor([[0.0], [0.0], [500.0], [1e14]], dtype=torch.float64, device="cuda")

    def table(step_set):
        return rt.FieldTable([dict(sets=[dict(xyzm=xyzm, softening=0.1)], z_nodes=[0.0, chi], step_set=[step_set],
                                   bundle_offset=0, n_bundles=n)])

    rays, eager = (torch.zeros((8, 9 * n), dtype=torch.float64, device="cuda") for _ in range(2))
    rt.rt_build_bundles(c, table(-1), n, theta, radius, eager)
    torch.cuda.synchronize()
    graph, s = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    with torch.cuda.graph(graph, stream=s):
        with pytest.raises(rt.RTError) as err:
            rt.rt_build_bundles(c, table(0), n, theta, radius, rays, s)
        assert err.value.status == -6 and "captured" in str(err.value)
        rt.rt_build_bundles(c, table(-1), n, theta, radius, rays, s)
    for _ in range(3):
        rays.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(rays, eager)
    rt.rt_build_bundles(c, table(0), n, theta, radius, rays)   # and outside a capture as ever
    torch.cuda.synchronize()
    assert not torch.equal(rays, eager)
