"""The mesh build's rounding does not depend on the unit of length: every quantity of every grid to a few units in
the last place of its own largest value, from spacings of 1e-5 to 1e3 Mpc and softenings below and above the grid.

Tolerance: a transform of N points in u = 2^-53 arithmetic is off by about 0.6 u sqrt(log2 N) in the root mean square,
relative to its result's; the masses', the kernel's and the way back add up in squares (N = 64^3: 4.4 u), and the largest of
some thousand errors is about four times that: 18 u, doubled."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import pm as opm
from paper_1110_4894_amd import rt

pytestmark = pytest.mark.gpu
U = 2.0 ** -53


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rt.load()


def _build(xyz, m, n, h, origin, eps, periodic):
    xyzm = torch.from_numpy(np.ascontiguousarray(np.concatenate([xyz.T, m[None]]))).cuda()
    grid = rt.pm_grid(n, origin, h, periodic)
    size = rt.rt_pm_workspace_bytes(grid)
    fields = torch.empty(8 * n ** 3, dtype=torch.float64, device="cuda")
    rt.rt_pm_build(rt.make_particle_set(xyzm, softening=eps), grid, fields,
                   torch.empty(size, dtype=torch.uint8, device="cuda"), size)
    torch.cuda.synchronize()
    return fields.reshape(8, n, n, n).cpu().numpy()[:4]


@pytest.mark.parametrize("soft", [0.0, 0.3, 5.0, 300.0])
@pytest.mark.parametrize("h", [1e-5, 1e-3, 0.03, 20.0, 1e3])
def test_isolated(h, soft):
    n = 32
    rng = np.random.default_rng(11)
    nodes = np.unique(rng.integers(0, n, (40, 3)), axis=0)
    m = rng.uniform(0.5, 1.5, len(nodes)) * 1e10
    got = _build(h * nodes, m, n, h, np.zeros(3), soft * h, False)
    # the direct sum over the node masses in extended precision, in units of the spacing
    g = np.arange(n, dtype=np.longdouble)
    want = np.zeros((4, n, n, n), np.longdouble)
    for (a, b, c), w in zip(nodes, m):
        dx, dy, dz = (g - a)[:, None, None], (g - b)[None, :, None], (g - c)[None, None, :]
        r2 = dx ** 2 + dy ** 2 + dz ** 2 + np.longdouble(soft) ** 2
        k1 = np.where(r2 > 0, 1 / np.sqrt(np.where(r2 > 0, r2, 1)), 0)
        k3 = w * k1 ** 3
        want[0] -= w * k1
        want[1] += dx * k3
        want[2] += dy * k3
        want[3] += dz * k3
    for q in range(4):
        scale = np.abs(want[q]).max()
        # (G is one factor of all results: taken from the two largest values)
        at = np.unravel_index(np.abs(want[q]).argmax(), want[q].shape)
        diff = got[q] * (want[q][at] / np.longdouble(got[q][at])) - want[q]
        assert np.abs(diff).max() <= 2 * 36 * U * scale, q


@pytest.mark.parametrize("h", [1e-5, 0.03, 1e3])
def test_periodic(h):
    n = 32
    rng = np.random.default_rng(12)
    nodes = np.unique(rng.integers(0, n, (400, 3)), axis=0)
    m = rng.uniform(0.5, 1.5, len(nodes)) * 1e10
    got = _build(h * nodes, m, n, h, np.zeros(3), 0.0, True)
    want = opm.periodic_field(opm.cic_deposit_periodic(h * nodes, m, np.zeros(3), h, n), h)
    for q in range(4):   # the oracle's transforms round too
        assert np.abs(got[q] - want[q]).max() <= 2 * 36 * U * np.abs(want[q]).max(), q
