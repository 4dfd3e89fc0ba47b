"""The ways a mesh's field is taken at a ray: a window shared by its bundle, or its own nodes where the bundle is wide;
and what those cost that the general case should not pay for.

Times are medians of events on one stream, compared within the test only."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1110_4894_amd import rt

pytestmark = pytest.mark.gpu
N, ZS = 64, 1.0


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rt.load()


class Mesh:
    def __init__(self, periodic, h, origin):
        self.c = rt.cosmology()
        self.chi = rt.rt_comoving_distance(self.c, ZS)
        rng = np.random.default_rng(5)
        xyz = np.asarray(origin) + rng.uniform(0, N * h, (4000, 3))
        xyzm = torch.from_numpy(np.ascontiguousarray(np.concatenate([xyz.T, np.full((1, 4000), 1e12)]))).cuda()
        self.grid = rt.pm_grid(N, origin, h, periodic)
        size = rt.rt_pm_workspace_bytes(self.grid)
        self.fields = torch.empty(8 * N ** 3, dtype=torch.float64, device="cuda")
        rt.rt_pm_build(rt.make_particle_set(xyzm, softening=h), self.grid, self.fields,
                       torch.empty(size, dtype=torch.uint8, device="cuda"), size)
        torch.cuda.synchronize()

    def bundles(self, n, radius, half, seed=1):
        theta = torch.from_numpy(np.random.default_rng(seed).uniform(-half, half, (2, n))).cuda()
        rays = torch.empty((8, 9 * n), dtype=torch.float64, device="cuda")
        rt.rt_build_bundles(self.c, rt.FieldTable([]), n, theta, radius, rays)
        return rays

    def z(self, rays, n_int, steps=40, begin=0, end=None, field=True, nodes=None):
        nodes = np.linspace(0, self.chi, steps + 1) if nodes is None else nodes
        rt.rt_trace_pm(self.c, ZS, self.grid, self.fields, n_int, nodes, begin, steps if end is None else end,
                       rays.shape[1] // 9, rays, None, None if field else np.full(len(nodes) - 1, -1, np.int32))
        return rays

    def lam(self, rays, n_int, steps=40):
        rt.rt_trace_pm_lambda(self.c, ZS, self.grid, self.fields, n_int, self.chi / self.grid.h / steps, 2 * steps,
                              rays.shape[1] // 9, rays, None, None)
        return rays


def _ms(call, prepare):
    out = []
    for _ in range(7):
        x = prepare()
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        call(x)
        b.record()
        torch.cuda.synchronize()
        out.append(a.elapsed_time(b))
    return float(np.median(out[2:]))


@pytest.mark.parametrize("n_int", [1, 2, 3, 4])
@pytest.mark.parametrize("periodic", [False, True])
@pytest.mark.parametrize("radius", [1e-9, 2e-6, 2e-5, 4e-5, 3e-4, 8e-3])
def test_wide_bundles_give_each_ray_what_it_gets_alone(periodic, n_int, radius):
    """A ray's field depends on the ray: in z, bit by bit, whether its bundle is narrow, straddles cells or is wider than
    many; a bundle of nine copies of the ray is as narrow as can be.  (In the affine parameter a bundle's values along x^3 are
    one value and slope where the difference is below their rounding.)"""
    m = Mesh(periodic, 1.0, (-32.0, -32.0, 300.0))
    rays = m.bundles(31, radius, 2e-2)
    alone = rays.repeat_interleave(9, dim=1).contiguous()   # ray i as bundle i
    whole = m.z(rays.clone(), n_int)
    assert torch.equal(whole, m.z(alone.clone(), n_int)[:, ::9])
    parts = rays.clone()
    for s in range(0, 40, 13):
        m.z(parts, n_int, begin=s, end=min(s + 13, 40))
    assert torch.equal(whole, parts)
    a, b = m.lam(rays.clone(), n_int), m.lam(alone.clone(), n_int)[:, ::9]
    # some 200 stages of rounding, each below 2^-52 of the largest term
    assert ((a - b).abs() <= 1e-12 * b.abs().amax(dim=1, keepdim=True)).all()


@pytest.mark.parametrize("n_int", [2, 3, 4])
def test_wide_bundles_cost_a_load_of_each_rays_nodes(n_int):
    """Nine rays with windows of their own, on a grid that their way crosses for a fifth: at most two and a half times
    the launch whose bundles share one (a round of fetching for each took up to five times)."""
    m = Mesh(False, 4.0, (-128.0, -128.0, 100.0))
    narrow, wide = m.bundles(4096, 5e-9, 2e-2), m.bundles(4096, 9e-3, 2e-2)
    t = [_ms(lambda r: m.lam(r, n_int), lambda: x.clone()) for x in (narrow, wide)]
    print("n_int %d: narrow %.3f ms, wide %.3f ms" % (n_int, *t))
    assert t[1] <= 2.5 * t[0]


def test_points_with_large_windows_cost_their_nodes():
    """Points in cell order: eight nodes a side are four times the nodes of four a side, and half as much again is
    allowed (with each load waiting for the one before they took eleven to thirty times)."""
    m = Mesh(False, 1.0, (0.0, 0.0, 100.0))
    rng = np.random.default_rng(2)
    p = rng.uniform(0, N - 1, (3, 1000000))
    p = p[:, np.lexsort(np.floor(p))] + np.array([[0.0], [0.0], [100.0]])
    pts = torch.from_numpy(np.ascontiguousarray(p)).cuda()
    phi, grad = torch.empty(1000000, dtype=torch.float64, device="cuda"), torch.empty((3, 1000000), dtype=torch.float64, device="cuda")
    t = [_ms(lambda _: rt.rt_pm_eval(m.grid, m.fields, k, 1000000, pts, phi, grad), lambda: None) for k in (2, 4)]
    print("4 a side %.3f ms, 8 a side %.3f ms" % tuple(t))
    assert t[1] <= 6.0 * t[0]
