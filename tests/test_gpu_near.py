"""FP32 sums with more near pairs than a wavefront's list holds: right, and not summed more often or walked further
than the pairs ask for.  The set is a filament along the line of sight, so that every plane of the trace has near pairs."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1110_4894_amd import rt

pytestmark = pytest.mark.gpu
FP64, FP32K = rt.RT_FP64, rt.RT_FP32_KAHAN
Z, ZS, WIDTH, LIST = 800.0, 1.0, 0.02, 62


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rt.load()
    yield
    rt.rt_force_plan(FP32K, -1)
    rt.rt_enable_timing(False)
    rt.rt_release_caches()


def _filament(n, order, heavy=0.0):
    rng = np.random.default_rng(n)
    xyz = np.stack([rng.normal(0, WIDTH, n), rng.normal(0, WIDTH, n), rng.uniform(Z - 2, Z + 2, n)], 1)
    if order == "sorted":
        xyz = xyz[np.argsort(xyz[:, 2])]
    m = np.ones(n)
    if heavy:
        xyz[-1], m[-1] = (0.5, 0.0, Z), heavy
    return xyz, m


class Case:
    def __init__(self, xyz, m, n_bundles, delta, eps, steps):
        self.c, self.nb = rt.cosmology(), n_bundles
        chi = rt.rt_comoving_distance(self.c, ZS)
        xyzm = torch.from_numpy(np.ascontiguousarray(np.concatenate([xyz, m[:, None]], 1).T)).cuda()
        self.nodes = np.concatenate([[0.0], np.linspace(Z - 1.8, Z + 1.8, steps + 1), [chi]])
        ss = np.zeros(steps + 2, np.int32)
        ss[0] = ss[-1] = -1
        self.steps = steps
        self.table = rt.FieldTable([dict(sets=[dict(xyzm=xyzm, softening=eps)], z_nodes=self.nodes, step_set=ss,
                                         bundle_offset=0, n_bundles=n_bundles)])
        theta = torch.from_numpy(np.random.default_rng(3).normal(0, WIDTH / Z, (2, n_bundles))).cuda()
        self.rays = torch.empty((8, 9 * n_bundles), dtype=torch.float64, device="cuda")
        rt.rt_build_bundles(self.c, self.table, n_bundles, theta, delta / Z, self.rays)
        rt.rt_trace(self.c, ZS, self.table, FP64, 0, 1, n_bundles, self.rays)
        self.first = self.rays.clone()

    def trace(self, precision):
        self.rays.copy_(self.first)
        rt.rt_trace(self.c, ZS, self.table, precision, 1, 1 + self.steps, self.nb, self.rays)
        torch.cuda.synchronize()
        return self.rays.cpu().numpy()

    def ms(self):
        rt.rt_enable_timing(True)
        times = []
        for _ in range(4):
            self.trace(FP32K)
            times.append(rt.rt_last_trace_info()["kernel_ms"])
        rt.rt_enable_timing(False)
        return min(times)


@pytest.mark.parametrize("order", ["random", "sorted"])
@pytest.mark.parametrize("n,delta,full", [(700, 1e-5, False), (3000, 1e-5, False), (40000, 1e-5, True), (9001, 3e-5, True)])
def test_lists_that_hold_the_near_pairs_and_lists_that_do_not(n, delta, full, order):
    """Every ray against the FP64 sums of the same launch.  full: some wavefront meets more near particles at some plane
    than its list holds (counted here from the positions, for a wavefront of seven bundles that sees the whole set)."""
    xyz, m = _filament(n, order)
    case = Case(xyz, 1e9 * m, 28, delta, 0.0005, 6)
    start = case.first.cpu().numpy()
    counts = []
    for group in range(4):
        near = np.zeros(n, bool)
        for b in range(7 * group, 7 * group + 7):
            at = start[1:3, 9 * b] * (Z / start[3, 9 * b])
            r2 = ((xyz[:, :2] - at) ** 2).sum(1)[None, :] + (xyz[:, 2][None, :] - case.nodes[1:-1, None]) ** 2
            near |= (r2[3] + 0.0005 ** 2) < (1024 * delta) ** 2
        counts.append(int(near.sum()))
    assert max(counts) > LIST if full else 0 < max(counts) <= LIST - 9, counts
    want = case.trace(FP64)
    for plan in range(rt.rt_plan_count(FP32K)):
        rt.rt_force_plan(FP32K, plan)
        got = case.trace(FP32K)
        for k in (5, 6):
            turn = np.abs(want[k] - start[k]).max()
            assert np.abs(got[k] - want[k]).max() <= 1e-5 * turn, plan
            # ring against anchor
            w, g = want[k].reshape(-1, 9), got[k].reshape(-1, 9)
            s = start[k].reshape(-1, 9)
            dw, dg = (w - s) - (w - s)[:, :1], (g - s) - (g - s)[:, :1]
            assert np.abs(dg - dw).max() <= 2e-4 * np.abs(dw).max(), plan
    rt.rt_force_plan(FP32K, -1)


def test_full_lists_cost_a_second_look_at_their_tiles():
    """Against the same launch without near pairs: the nearness test and a look at every tile for the particles that did
    not fit take a moment sum and a half; twice that is the limit (walked by every lane and with no plane
    kept, they took eleven)."""
    xyz, m = _filament(50000, "random")
    rt.rt_force_plan(FP32K, 0)
    free = Case(xyz, m, 14336, 1e-5, 0.05, 6).ms()
    full = Case(xyz, m, 14336, 1e-5, 0.0005, 6).ms()
    rt.rt_force_plan(FP32K, -1)
    print("no near pairs %.2f ms, full lists %.2f ms" % (free, full))
    assert full <= 3.0 * free


def test_rays_that_leave_the_expansion_points():
    """A heavy particle beside the filament moves the rays by hundreds of radii between the two visits of a middle
    plane: the second sum is about their own points, with no more near pairs than the first, and costs what a sum at every
    stage does, at most twice the launch whose planes are kept (half as much again is allowed; about the points that the
    rays had left it was more than four times)."""
    rt.rt_force_plan(FP32K, 0)
    xyz, m = _filament(50000, "random")
    kept = Case(xyz, m, 14336, 1e-6, 0.05, 5).ms()
    xyz, m = _filament(50000, "random", heavy=4e16)
    moved = Case(xyz, m, 14336, 1e-6, 0.0005, 5).ms()
    rt.rt_force_plan(FP32K, -1)
    print("planes kept %.2f ms, rays moved %.2f ms" % (kept, moved))
    assert moved <= 3.0 * kept


@pytest.mark.parametrize("order", ["random", "sorted"])
def test_full_lists_give_the_rays_of_one_run(order):
    """Step windows of any width give the same bits as one launch: a second visit's walk through the tiles repeats the
    first's, and a visit that cannot reuse the plane sums what a launch that starts there would."""
    xyz, m = _filament(9001, order, heavy=1e6)
    case = Case(xyz, 1e9 * m, 28, 3e-5, 0.0005, 6)
    for plan in range(rt.rt_plan_count(FP32K)):
        rt.rt_force_plan(FP32K, plan)
        whole = case.trace(FP32K)
        for width in (1, 4):
            case.rays.copy_(case.first)
            for s in range(1, 7, width):
                rt.rt_trace(case.c, ZS, case.table, FP32K, s, min(s + width, 7), case.nb, case.rays)
            torch.cuda.synchronize()
            assert np.array_equal(case.rays.cpu().numpy(), whole), (plan, width)
    rt.rt_force_plan(FP32K, -1)
