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
