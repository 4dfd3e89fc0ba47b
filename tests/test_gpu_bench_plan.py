"""The launch that bench.py times by default, on the plans beside the one of a wavefront to a group of seven bundles: four
wavefronts to a group, which its autotuner picks on some cards (within 3% of it), and two.  Seeded bundles of the band against the oracle
traced through the window's first steps: positions and directions, each relative to its change from the straight ray."""
import dataclasses

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle as orc
from paper_1110_4894_amd import rt
from paper_1110_4894_amd import workloads as wl
from tests.oracle_run import oracle_run

pytestmark = pytest.mark.gpu
FP32K = rt.RT_FP32_KAHAN


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rt.load()
    yield
    rt.rt_force_plan(FP32K, -1)


@pytest.mark.parametrize("waves_per_group,tile", [(4, 576), (2, 1152)])
def test_band_through_the_first_steps(waves_per_group, tile):
    from paper_1110_4894_amd.runner import GpuRun
    w = wl.box(n_part_log2=20, n_side=512)
    f, band, window = w.fields[0], 28672, 10
    plan = [i for i in range(rt.rt_plan_count(FP32K))
            if [rt.rt_plan_describe(FP32K, i)[k] for k in ("waves_per_block", "waves_per_group", "tile", "waves_per_simd")]
            == [8, waves_per_group, tile, 4]]
    assert len(plan) == 1
    rt.rt_force_plan(FP32K, plan[0])
    g = GpuRun(dataclasses.replace(w, fields=[dataclasses.replace(f, theta=f.theta[:, :band])]))
    g.build_bundles()
    g.trace(FP32K, 0, window)
    torch.cuda.synchronize()
    info = rt.rt_last_trace_info()
    assert info["plan_id"] == plan[0] and info["grid_blocks"] == 512
    assert not g.flags.cpu().numpy().any()
    idx = np.sort(np.random.default_rng(2812).choice(band, 6, replace=False))
    got = g.rays.cpu().numpy()[:, (9 * idx[:, None] + np.arange(9)).ravel()]
    ws = dataclasses.replace(w, fields=[dataclasses.replace(f, theta=np.ascontiguousarray(f.theta[:, idx]))])
    o = oracle_run(ws, step_begin=0, step_end=window)
    r0 = orc.build_bundles(o["cosmo"], o["fields"], o["theta"], w.bundle_radius)
    want = o["rays"]
    assert np.allclose(got[3], want[3], rtol=1e-13, atol=0)
    for comp, kc in ((1, 5), (2, 6)):
        straight = r0[kc] / r0[7] * want[3]
        assert np.all(np.abs(got[comp] - want[comp]) <= 1e-4 * np.abs(want[comp] - straight) + 1e-13)
        bend = want[kc] / want[7] - r0[kc] / r0[7]
        assert np.all(np.abs(got[kc] / got[7] - want[kc] / want[7]) <= 1e-4 * np.abs(bend) + 1e-16)
