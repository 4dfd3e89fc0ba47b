"""Many values for few targets: histograms of one or a few bins, masses of a great many particles on a grid of a
few nodes.  Right, and no slower than the same values on more targets (medians of events, compared within the test)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle as orc
from oracle import pm as opm
from paper_1110_4894_amd import rt

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rt.load()


def _us(call, burst=50):
    out = []
    for _ in range(9):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(burst):
            call()
        b.record()
        torch.cuda.synchronize()
        out.append(a.elapsed_time(b) * 1e3 / burst)
    return float(np.median(out[2:]))


def _mu_histogram(mu, bins):
    d = torch.from_numpy(mu).cuda()
    pdf = torch.empty(bins, dtype=torch.float64, device="cuda")
    mom = torch.empty(6, dtype=torch.float64, device="cuda")
    call = lambda: rt.rt_mu_histogram_noalloc(len(mu), d, bins, -0.1, 0.3, pdf, mom)
    call()
    torch.cuda.synchronize()
    return call, pdf.cpu().numpy(), mom.cpu().numpy()


@pytest.mark.parametrize("kind", ["one value", "two bins", "three bins", "four bins", "spread"])
@pytest.mark.parametrize("n", [64, 1000, 16385])
def test_values_that_share_bins(n, kind):
    rng = np.random.default_rng(n)
    k = {"one value": 1, "two bins": 2, "three bins": 3, "four bins": 4, "spread": 150}[kind]
    mu = 10.0 ** (-0.1 + 0.4 * (rng.integers(0, k, n) + 0.5) / 200)
    _, pdf, mom = _mu_histogram(mu, 200)
    want = orc.mu_histogram(mu, 200, -0.1, 0.3)
    # sums of n positive terms in another order, and a bin's width (the difference of two powers of ten)
    rtol = 2.0 * n * 2.0 ** -53 + 1e-13 + 8.0 * 2.0 ** -53 / (1.0 - 10.0 ** (-0.4 / 200))
    assert np.allclose(pdf, want[0], rtol=rtol, atol=0)
    # (the spread about the mean has its own tests: of equal values it is nothing but the mean's rounding)
    assert np.allclose(np.delete(mom, 2), np.delete(want[1], 2), rtol=1e-12, atol=1e-15)


def test_one_bin_costs_what_many_do():
    """A wavefront's values of one bin meet in six exchanges (one after the other they were 64: twice the time)."""
    mu = np.exp(np.random.default_rng(1).normal(0, 0.1, 1000))
    one, many = _us(_mu_histogram(mu, 1)[0]), _us(_mu_histogram(mu, 200)[0])
    print("1 bin %.1f us, 200 bins %.1f us" % (one, many))
    assert one <= 1.5 * many


def _deposit(n, periodic, m):
    rng = np.random.default_rng(n)
    h, origin = 0.03, np.array([-0.4, 0.2, 5.0])
    xyz = origin + h * rng.uniform(*((-0.5, n + 0.5) if periodic else (-1.5, n + 0.5)), (m, 3))
    mass = rng.uniform(0.5, 1.5, m) * 1e10
    xyzm = torch.from_numpy(np.ascontiguousarray(np.concatenate([xyz.T, mass[None]]))).cuda()
    grid = rt.pm_grid(n, origin, h, periodic)
    size = rt.rt_pm_workspace_bytes(grid)
    fields = torch.empty(8 * n ** 3, dtype=torch.float64, device="cuda")
    ws, ps = torch.empty(size, dtype=torch.uint8, device="cuda"), rt.make_particle_set(xyzm, softening=0.01)
    call = lambda: rt.rt_pm_build(ps, grid, fields, ws, size)
    call()
    torch.cuda.synchronize()
    return call, fields.reshape(8, n, n, n).cpu().numpy(), (xyz, mass, origin, h)


@pytest.mark.parametrize("periodic", [False, True])
@pytest.mark.parametrize("n", [4, 8])
@pytest.mark.parametrize("m", [1, 255, 257, 16384, 40001])
def test_many_particles_on_few_nodes(n, periodic, m):
    _, got, (xyz, mass, origin, h) = _deposit(n, periodic, m)
    if periodic:
        want = opm.periodic_field(opm.cic_deposit_periodic(xyz, mass, origin, h, n), h)
    else:
        want = opm.isolated_field(opm.cic_deposit(xyz, mass, origin, h, n), h, 0.01)
    for q in range(4):   # the tolerance of the builds at every line length
        assert np.max(np.abs(got[q] - want[q])) <= 1e-11 * np.abs(want[q]).max(), q


@pytest.mark.parametrize("periodic", [False, True])
def test_few_nodes_cost_what_more_do(periodic):
    """10^5 particles: a grid of 4^3 nodes takes no longer than one of 16^3 whose cache lines they share less (half as
    much again is allowed; with every addition at the same four lines it took five times as long)."""
    few, more = _us(_deposit(4, periodic, 100000)[0], 5), _us(_deposit(16, periodic, 100000)[0], 5)
    print("4^3 nodes %.0f us, 16^3 nodes %.0f us" % (few, more))
    assert few <= 1.5 * more


@pytest.mark.parametrize("bins", [1, 7, 1024, 1025])
def test_shear_that_is_no_number_counts_in_the_first_bin(bins):
    """mu and the Jacobian are independent arrays: a weight with no value has a bin all the same, on both ways."""
    n = 777
    rng = np.random.default_rng(bins)
    mu, jac = np.exp(rng.normal(0, 0.1, n)), rng.normal(0, 0.02, (4, n))
    lost = rng.random(n) < 0.1
    jac[1, lost] = np.nan
    pdf, mom = torch.empty(bins, dtype=torch.float64, device="cuda"), torch.empty(6, dtype=torch.float64, device="cuda")
    rt.rt_shear_histogram(n, torch.from_numpy(mu).cuda(), torch.from_numpy(jac).cuda(), bins, 0.0, 0.1, pdf, mom)
    torch.cuda.synchronize()
    jac[1:3, lost] = 0.0   # a value in the first bin
    want = orc.shear_histogram(mu, jac, bins, 0.0, 0.1)
    got = mom.cpu().numpy()
    assert np.allclose(pdf.cpu().numpy(), want[0], rtol=1e-12, atol=0)
    assert np.isclose(got[0], want[1][0], rtol=1e-12) and np.isnan(got[1]) and np.isnan(got[2])
    assert np.array_equal(got[3:], want[1][3:])
