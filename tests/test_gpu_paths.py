"""The kernels' own edges: tile remainders, the smallest and largest of a
path's range, each against plain torch or the oracle."""
import numpy as np
import pytest
import torch

from paper_2406_11836_amd import raster, scenes, train

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rast():
    return raster.Rasterizer()


@pytest.mark.parametrize("n,D", [(1, 0), (255, 1), (256, 2), (257, 3), (4097, 3)])
def test_regrouped_rows_are_the_permuted_rows(rast, n, D):
    """Staged 16-row groups (14, 23, 38 and 59 rows: full and partial last
    groups) and the row-major permute move every row exactly."""
    p = raster.to_device(scenes.scene_uniform(n, seed=n, D=D))
    kd = rast.kd_partition(p, 3)
    g, perm = rast.group_by_cell(p, kd)
    at = perm.long()
    assert torch.equal(torch.sort(at).values, torch.arange(n, device="cuda"))
    q = train.permute(rast.lib, p, perm)
    for k in raster.PARAM_KEYS:
        assert torch.equal(g[k], p[k][..., at]), k
        assert torch.equal(q[k], p[k][..., at]), k
    assert torch.all(torch.diff(kd.center_cell[at]) >= 0)


@pytest.mark.parametrize("D", [0, 3])
def test_sparse_projection_equals_direct(rast, D):
    """Large scenes seen by one or two views project survivors compacted per
    block; three views take the direct kernels.  The same view gives the same
    records, image and gradients bit for bit (views with a zero image gradient
    add exact zeros), with cell culling or without."""
    n = 2_000_137
    p = scenes.scene_city_device(n, seed=7, D=D, half=400.0, n_boxes=500)
    p, _ = rast.group_by_cell(p, rast.kd_partition(p, 4))
    kd = rast.kd_partition(p, 4)
    cams = [scenes.aerial_camera(np.random.default_rng(k), 401, 273, 300.0, 90.0, -50.0) for k in (3, 4, 5)]
    a = rast.forward(p, kd, cams[:1], 5e-5)
    b = rast.forward(p, kd, cams, 5e-5)
    c = rast.forward(p, kd, cams[:1], 5e-5, cull=True)
    na, px = n, 401 * 273
    kept = a.proj["count"][:na] != 0
    assert 0.001 < kept.float().mean().item() < 0.5
    assert torch.equal(a.proj["count"][:na], b.proj["count"][:na])
    assert torch.equal(a.proj["count"][:na], c.proj["count"][:na])
    for key, w in (("rec", 16), ("bin", 8)):
        x = a.proj[key][: na * w].view(na, w)[kept].view(torch.int32)
        assert torch.equal(x, b.proj[key][: na * w].view(na, w)[kept].view(torch.int32)), key
        assert torch.equal(x, c.proj[key][: na * w].view(na, w)[kept].view(torch.int32)), key
    assert torch.equal(a.image, b.image[: 3 * px]) and torch.equal(a.image, c.image)
    d = torch.randn(3 * px, device="cuda", generator=torch.Generator("cuda").manual_seed(1))
    ga = rast.backward(a, p, d)
    gb = rast.backward(b, p, torch.cat([d, torch.zeros(6 * px, device="cuda")]))
    for k in raster.PARAM_KEYS:
        assert torch.equal(ga[k], gb[k]), k
        assert torch.count_nonzero(ga[k]) > 0, k
