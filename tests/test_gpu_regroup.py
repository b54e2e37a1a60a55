"""Regrouping and permuting: the way rows are moved depends on whether neighbours come
from neighbours and on the size, the rows do not."""
import ctypes as C

import pytest
import torch

from paper_2406_11836_amd import _lib as L
from paper_2406_11836_amd import raster, train

pytestmark = pytest.mark.gpu


def _scene(n, D, seed=1):
    f = dict(device="cuda", generator=torch.Generator("cuda").manual_seed(seed))
    return dict(means=torch.randn((3, n), **f), log_scales=torch.randn((3, n), **f) * 0.5 - 5,
                quats=torch.randn((4, n), **f), opacity=torch.randn((n,), **f),
                sh=torch.randn((3 * (D + 1) ** 2, n), **f), sh_degree=D)


@pytest.mark.parametrize("n,D", [(131_072, 1), (131_073, 0), (131_073, 3), (400_001, 2), (2_000_003, 0)])
def test_group_by_cell_again(n, D):
    """A scattered scene (rows staged beyond 131072 Gaussians), the grouped one (rows
    moved directly) and one of which a part is scattered again."""
    r = raster.Rasterizer()
    p = _scene(n, D)
    for turn in range(3):
        kd = r.kd_partition(p, 3)
        g, perm = r.group_by_cell(p, kd)
        at = perm.long()
        assert torch.equal(torch.sort(at).values, torch.arange(n, device="cuda"))
        assert torch.all(torch.diff(kd.center_cell[at]) >= 0)
        for k in raster.PARAM_KEYS:
            assert torch.equal(g[k], p[k][..., at]), (turn, k)
        p = g
        if turn == 1:  # a tenth of it moves anywhere
            some = torch.randperm(n, device="cuda", generator=torch.Generator("cuda").manual_seed(2))[: n // 10]
            for k in raster.PARAM_KEYS:
                p[k][..., some] = p[k][..., some.roll(7)]


@pytest.mark.parametrize("n,kind", [(n, kind) for n in (1, 2, 255, 262_143, 262_144, 1_000_003)
                                    for kind in ("identity", "swaps", "random", "backwards", "out of range")]
                         + [(8_000_001, "swaps"), (8_000_001, "random")])  # (longer tiles)
def test_permute(n, kind):
    """Every row of out[j] = in[perm[j]]; entries outside [0, n) leave the row as it was."""
    r = raster.Rasterizer()
    p = _scene(n, 0 if n > 1_000_003 else 2)
    g = torch.Generator("cuda").manual_seed(3)
    perm = torch.arange(n, device="cuda", dtype=torch.int32)
    if kind == "swaps":  # near: places up to 1000 apart
        perm = (perm + torch.randint(-500, 500, (n,), device="cuda", generator=g)).clamp(0, n - 1).int()
    elif kind == "random":
        perm = torch.randperm(n, device="cuda", generator=g).int()
    elif kind == "backwards":
        perm = perm.flip(0).contiguous()
    elif kind == "out of range":
        perm[::3] = -1
        perm[1::5] = n
        perm[2::7] = 2 ** 31 - 1
    ok = (perm >= 0) & (perm < n)
    at = perm.long().clamp(0, n - 1)
    if ok.all():
        q = train.permute(r.lib, p, perm)
        for k in raster.PARAM_KEYS:
            assert torch.equal(q[k], p[k][..., at]), k
    out = {k: torch.full_like(p[k], 7.0) for k in raster.PARAM_KEYS}
    gi = raster.gaussians_struct(p)
    go = L.GaussiansGrad(*[out[k].data_ptr() for k in raster.PARAM_KEYS])
    L.check("rgs_permute_gaussians", r.lib.rgs_permute_gaussians(C.byref(gi), perm.data_ptr(), C.byref(go), raster._stream()))
    for k in raster.PARAM_KEYS:
        assert torch.equal(out[k], torch.where(ok, p[k][..., at], torch.full_like(p[k], 7.0))), k
