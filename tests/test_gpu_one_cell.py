"""The partition of one cell: counts, ownership and bounds against the oracle, bit for bit."""
import numpy as np
import pytest

import oracle
from paper_2406_11836_amd import raster, scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 63, 64, 257, 5000, 300_001])
@pytest.mark.parametrize("kind", ["normal", "sorted", "odd"])
@pytest.mark.parametrize("rule", [0, 1])
def test_one_cell(n, kind, rule):
    rng = np.random.default_rng(n)
    p = scenes.scene_uniform(n, seed=n, D=0, mu_s=-3.0)
    m = rng.normal(size=(3, n)).astype(np.float32) * 50
    if kind == "sorted":
        m = np.sort(m, axis=1)
    p["means"] = np.ascontiguousarray(m)
    if kind == "odd" and n >= 257:
        p["means"][0, :9], p["means"][1, 20:30] = np.inf, -np.inf
        p["log_scales"][1, 100:120] = 80.0
        p["log_scales"][2, 150:200] = -np.inf
    r = raster.Rasterizer()
    kd = r.kd_partition(raster.to_device(p), 0, rule=rule)
    o = oracle.kd_partition(p["means"], p["log_scales"], 0, 3.0, rule=rule)
    assert np.array_equal(kd.center_cell.cpu().numpy(), np.zeros(n, np.int32))
    assert kd.counts.cpu().tolist() == [n]
    assert np.array_equal(kd.own_mask.cpu().numpy().view(np.uint32).reshape(o["own_mask"].shape), o["own_mask"])
    smax = np.exp(p["log_scales"].astype(np.float64)).astype(np.float32).max()
    b = kd.cell_bounds_host[:, 0]
    assert np.array_equal(b[0:3], p["means"].min(1)) and np.array_equal(b[3:6], p["means"].max(1))
    assert b[6] == smax and b[7] == 0
    none = r.kd_partition(raster.to_device(p), 0, own_mask=False, rule=rule)
    assert np.array_equal(none.cell_bounds_host, kd.cell_bounds_host)
