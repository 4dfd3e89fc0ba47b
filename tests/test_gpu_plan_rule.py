"""The plan that a launch gets without tuning against all others, at sizes between those that the rule's figures were
taken at: within a quarter of the best (its own claim is 8%; kernel times, least of four)."""
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
    yield
    for prec in (rt.RT_FP64, rt.RT_FP32_KAHAN):
        rt.rt_force_plan(prec, -1)
    rt.rt_enable_timing(False)
    rt.rt_release_caches()


@pytest.mark.parametrize("precision,bundles,n", [(rt.RT_FP32_KAHAN, 2700, 750), (rt.RT_FP32_KAHAN, 3300, 12000),
                                                 (rt.RT_FP32_KAHAN, 4000, 7700), (rt.RT_FP32_KAHAN, 4700, 5000),
                                                 (rt.RT_FP32_KAHAN, 6500, 8000), (rt.RT_FP32_KAHAN, 17000, 7000),
                                                 (rt.RT_FP64, 3300, 70)])
def test_the_rule_picks_a_good_plan(precision, bundles, n):
    rng = np.random.default_rng(n)
    c, zs, z = rt.cosmology(), 1.0, 1200.0
    chi = rt.rt_comoving_distance(c, zs)
    xyz = rng.uniform(-30, 30, (3, n)) + np.array([[0.0], [0.0], [z]])
    xyzm = torch.from_numpy(np.ascontiguousarray(np.concatenate([xyz, np.full((1, n), 1e10)]))).cuda()
    nodes = np.concatenate([[0.0], np.linspace(z - 0.25, z + 0.25, 5), [chi]])
    table = rt.FieldTable([dict(sets=[dict(xyzm=xyzm, softening=0.07)], z_nodes=nodes, step_set=[-1, 0, 0, 0, 0, -1],
                                bundle_offset=0, n_bundles=bundles)])
    theta = torch.from_numpy(rng.uniform(-0.02, 0.02, (2, bundles))).cuda()
    first = torch.empty((8, 9 * bundles), dtype=torch.float64, device="cuda")
    rt.rt_build_bundles(c, table, bundles, theta, 5e-9, first)
    rt.rt_trace(c, zs, table, precision, 0, 1, bundles, first)
    rays = torch.empty_like(first)

    def ms(plan):
        rt.rt_force_plan(precision, plan)
        out = []
        for _ in range(5):
            rays.copy_(first)
            rt.rt_enable_timing(True)
            rt.rt_trace(c, zs, table, precision, 1, 5, bundles, rays)
            out.append(rt.rt_last_trace_info()["kernel_ms"])
        return min(out[1:])

    times = {p: ms(p) for p in range(rt.rt_plan_count(precision))}
    ms(-1)
    # its own time in the sweep: launches after an idle or slow one run up to 14% slower than the same plan amid others
    chosen = rt.rt_last_trace_info()["plan_id"]
    best = min(times, key=times.get)
    print("%d bundles, %d particles: plan %d %.3f ms, best plan %d %.3f" % (bundles, n, chosen, times[chosen], best, times[best]))
    assert times[chosen] <= 1.25 * times[best]
