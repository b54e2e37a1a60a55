"""The longest tiles' four-block walk against the others' walk, where they could part."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2406_11836_amd import _lib, raster, scenes

pytestmark = pytest.mark.gpu
SPLIT = 256  # tiles of a launch that are split


@pytest.fixture(scope="module")
def rast():
    return raster.Rasterizer()


def _first_view_equal(alone, batch, px):
    m = int(alone.bins["counters"][2])
    assert torch.equal(alone.bins["slot_key"][:m], batch.bins["slot_key"][:m])
    for a, b, w in ((alone.image, batch.image, 3 * px), (alone.T_final, batch.T_final, px),
                    (alone.parts["C"], batch.parts["C"], 768 * m), (alone.parts["T"], batch.parts["T"], 256 * m),
                    (alone.parts["last"], batch.parts["last"], 256 * m)):
        assert torch.equal(a.view(-1)[:w].view(torch.int32), b.view(-1)[:w].view(torch.int32))


def _whole(batch, n_tiles):
    """Tiles 0 .. n_tiles - 1 of the first view that are not split."""
    order = batch.bins["tile_order"][: batch.total_tiles].cpu().numpy()
    assert order.size > SPLIT
    at = np.empty(order.size, np.int64)
    at[order] = np.arange(order.size)
    return at[:n_tiles] >= SPLIT


def test_a_pixel_at_the_stop_threshold(rast):
    """eps_T chosen so that a pixel ends a slot at exactly T = eps_T / P: it has not stopped,
    but its product P T is rounded to just below eps_T, and the next slot's threshold to
    above 1.  It takes one contribution there, in a split tile as in a whole one."""
    W, H, L = 256, 240, 2
    p = raster.to_device(scenes.scene_uniform(3000, seed=11, D=1, mu_s=-3.0))
    kd = rast.kd_partition(p, L)
    cam = scenes.orbit_camera(1.8, 0.3, 0.3, W, H)
    far = [scenes.orbit_camera(3.0, 0.3 + 0.4 * v, 0.3, W, H) for v in range(15)]  # longer lists
    tiles = ((W + 15) // 16) * ((H + 15) // 16)
    assert tiles <= SPLIT
    whole = _whole(rast.forward(p, kd, [cam] + far, 0.0), tiles)
    st = rast.forward(p, kd, [cam], 0.0)
    S = int(st.bins["counters"][2])
    T = st.parts["T"][: 256 * S].view(S, 256).cpu().numpy()
    last = st.parts["last"][: 256 * S].view(S, 256).cpu().numpy()
    tile = st.bins["slot_key"][:S].cpu().numpy() >> L
    found = []
    for s in range(S - 1):
        if s == 0 or tile[s] != tile[s - 1]:
            P = np.ones(256, np.float32)
        Pn = P * T[s]
        eps = np.nextafter(Pn, np.float32(np.inf))
        if tile[s + 1] == tile[s] and whole[tile[s]]:
            hit = (eps / P == T[s]) & (Pn < eps) & (last[s + 1] > 0) & (last[s] > 0) & (eps < 1)
            found += [(s, int(k), float(eps[k])) for k in np.nonzero(hit)[0][:2]]
        P = Pn
    assert len(found) >= 4
    for s, k, eps in found[:: max(len(found) // 6, 1)][:6]:
        alone = rast.forward(p, kd, [cam], eps)
        batch = rast.forward(p, kd, [cam] + far, eps)
        assert int(batch.parts["last"][256 * (s + 1) + k]) > 0
        _first_view_equal(alone, batch, W * H)


def test_a_slot_table_of_some_cells(rast):
    """A caller that renders some of the cells passes a table of their slots, whose
    instances do not follow each other: the same partials as in the whole table
    (without early termination no cell depends on another)."""
    W, H, L = 250, 150, 3
    p = raster.to_device(scenes.scene_uniform(4000, seed=12, D=1, mu_s=-3.4))
    kd = rast.kd_partition(p, L)
    cam = scenes.orbit_camera(3.0, 0.3, 0.3, W, H)
    st = rast.forward(p, kd, [cam], 0.0)
    S = int(st.bins["counters"][2])
    key = st.bins["slot_key"][:S].cpu().numpy()
    tiles = st.total_tiles
    assert tiles <= SPLIT and st.T_final.min().item() > 2.0 ** -90
    sel = np.nonzero(np.isin(key & ((1 << L) - 1), (0, 2, 5, 7)))[0]
    assert (np.bincount(key[sel] >> L) > 1).sum() > 50
    idx = torch.from_numpy(sel).cuda()
    bs = st.bins_struct
    sk = torch.zeros(st.slot_capacity, dtype=torch.int32, device="cuda")
    sr = torch.zeros(2 * st.slot_capacity, dtype=torch.int32, device="cuda")
    sk[: sel.size] = st.bins["slot_key"][idx]
    sr[: 2 * sel.size] = st.bins["slot_range"][: 2 * S].view(S, 2)[idx].reshape(-1)
    ts = torch.from_numpy(np.searchsorted(key[sel] >> L, np.arange(tiles + 1)).astype(np.int32)).cuda()
    own = {k: torch.zeros_like(st.parts[k]) for k in ("C", "T", "last")}
    pt = _lib.Partials(*[own[k].data_ptr() for k in ("C", "T", "last")])
    saved = (bs.slot_key, bs.slot_range, bs.tile_slot)
    bs.slot_key, bs.slot_range, bs.tile_slot = sk.data_ptr(), sr.data_ptr(), ts.data_ptr()
    try:
        ps, ks = st.proj_struct(), kd.struct()
        _lib.check("rgs_render_partial", rast.lib.rgs_render_partial(
            C.byref(ps), st.n, C.byref(bs), st.cam_arr, 1, st.views.data_ptr(), C.byref(ks), 0.0, C.byref(pt), None,
            torch.cuda.current_stream().cuda_stream))
    finally:
        bs.slot_key, bs.slot_range, bs.tile_slot = saved
    for k, w in (("C", 768), ("T", 256), ("last", 256)):
        assert torch.equal(own[k][: w * sel.size].view(-1, w), st.parts[k][: w * S].view(S, w)[idx]), k


@pytest.mark.parametrize("n", [1, 2, 3, 5])
def test_short_lists_split_and_whole(rast, n):
    """Lists of fewer instances than a group of four, in a split tile and in a whole one."""
    W, H = 96, 96
    p = raster.to_device(scenes.scene_uniform(n, seed=n, D=1, mu_s=-0.5))
    kd = rast.kd_partition(p, 1)
    cams = [scenes.orbit_camera(3.0, 0.3, 0.3, W, H)] * 16
    batch = rast.forward(p, kd, cams, 5e-5)
    alone = rast.forward(p, kd, cams[:1], 5e-5)
    m = int(alone.bins["counters"][2])
    held = np.unique(alone.bins["slot_key"][:m].cpu().numpy() >> 1)
    longest = (alone.bins["slot_range"][: 2 * m].view(m, 2).diff(dim=1)).max().item()
    assert longest <= n and m > 0
    order = batch.bins["tile_order"][:SPLIT].cpu().numpy()
    views = [v for v in range(16) if not np.isin(held + 36 * v, order).all()]
    assert views  # some view has such a list in a whole tile
    keys, total = batch.bins["slot_key"], int(batch.bins["counters"][2])
    assert total == 16 * m
    for v in views:
        for k, w in (("C", 768), ("T", 256), ("last", 256)):
            assert torch.equal(alone.parts[k][: w * m], batch.parts[k][w * m * v: w * m * (v + 1)]), (k, v)
        assert torch.equal(keys[m * v: m * (v + 1)] - 72 * v, alone.bins["slot_key"][:m])
        assert torch.equal(alone.image, batch.image[3 * W * H * v: 3 * W * H * (v + 1)])
