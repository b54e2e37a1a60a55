"""The instance sort from 32M keys on, where digits are counted per sixteen tiles."""
import pytest
import torch

from paper_2406_11836_amd import raster, scenes

pytestmark = pytest.mark.gpu
WIDE, TILE, UNIT = 32_000_000, 2048, 16 * 2048


@pytest.mark.parametrize("n,W,H,L,views,sync", [
    (6500, 1600, 1060, 0, 1, True),    # 13 key bits: digits of 7 and 6
    (1000, 1600, 1060, 3, 1, False),   # 16 bits, the count left on the device
    (48, 3840, 2160, 5, 1, True),      # 20 bits, three passes: the emission writes to the alt buffers
    (3300, 1600, 1060, 0, 2, True),    # two views
])
def test_more_than_32m_instances(n, W, H, L, views, sync):
    """Keys in order, ties in emission order, positions a permutation, each with its
    pair's source, every pair's tiles distinct and inside its rectangle; slots the runs of equal keys."""
    r = raster.Rasterizer()
    p = raster.to_device(scenes.scene_uniform(n, seed=n, D=0, mu_s=0.3))
    kd = r.kd_partition(p, L)
    cams = [scenes.orbit_camera(3.0, 0.3 + v, 0.3, W, H) for v in range(views)]
    st = r.forward(p, kd, cams, 5e-5)
    if not sync:
        st = r.forward(p, kd, cams, 5e-5, no_sync=True)
        assert st.overflow() == 0 and st.bins_struct.n_instances < 0
    b = st.bins
    npair, ninst, nslot = (int(x) for x in b["counters"][:3])
    assert ninst >= WIDE and ninst % TILE and (ninst + TILE - 1) // TILE % 16  # partial last tile and unit
    keys = b["keys"][:ninst]
    j = (b["vals"][:ninst] & 0xFFFFFFFF)
    src = b["vals"][:ninst] >> 32
    assert torch.all((keys[1:] > keys[:-1]) | ((keys[1:] == keys[:-1]) & (j[1:] > j[:-1])))
    seen = torch.zeros(ninst, dtype=torch.bool, device="cuda")
    seen[j] = True
    assert seen.all()
    del seen
    off = b["pair_off"][: npair + 1].long()
    assert off[0] == 0 and off[-1] == ninst
    assert torch.equal(off.diff(), st.proj["count"][b["pair_src"][:npair].long()].long())
    pair = torch.searchsorted(off, j, right=True) - 1
    assert torch.equal(b["pair_src"][:npair].long()[pair], src)
    per_view = st.total_tiles // views
    tile, view = keys.long() >> L, src // n
    tx_n = (W + 15) // 16
    t = tile - view * per_view
    assert torch.all((t >= 0) & (t < per_view))
    rect = st.proj["bin"].view(-1, 8)[:, :2].contiguous().view(torch.int16).view(-1, 4)[src].long() >> 4
    tx, ty = t % tx_n, t // tx_n
    assert torch.all((tx >= rect[:, 0]) & (tx <= rect[:, 1]) & (ty >= rect[:, 2]) & (ty <= rect[:, 3]))
    del rect, tx, ty, t
    one = (pair * (st.total_tiles << L) + keys.long()).sort().values
    assert torch.all(one[1:] > one[:-1])
    start = torch.cat([torch.zeros(1, dtype=torch.long, device="cuda"), (keys.diff() != 0).nonzero()[:, 0] + 1])
    assert nslot == start.numel()
    rng = b["slot_range"][: 2 * nslot].view(nslot, 2).long()
    assert torch.equal(rng[:, 0], start) and torch.equal(rng[:-1, 1], start[1:]) and int(rng[-1, 1]) == ninst
