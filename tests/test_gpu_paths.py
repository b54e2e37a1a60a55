"""The kernels' own edges: tile remainders, the smallest and largest of a
path's range, each against plain torch or the oracle."""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import grad_close
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


@pytest.mark.parametrize("n,W,H,L,mu,views,sync", [
    (1, 40, 24, 0, -1.0, 1, True),          # one pair, a single 6-bit pass (odd: the emission writes to the alt buffers)
    (300, 16, 16, 0, -3.0, 1, True),        # one tile: no key bit at all
    (5000, 256, 256, 2, -4.0, 1, False),    # 512-key tiles, emission of 256 instances per block
    (30000, 256, 256, 2, -3.6, 1, True),    # beyond 64K instances: 2048-key tiles, still folded
    (30000, 320, 200, 3, -3.0, 1, False),   # around the fold's 262144 instances
    (40000, 333, 201, 3, -3.0, 1, True),    # beyond it
    (20000, 3840, 2160, 5, -3.4, 1, True),  # 20 key bits, three passes; rectangles without a descriptor
    (20000, 333, 201, 2, -4.0, 3, True),    # a fifth, view pass in the depth order
    (64, 1600, 1060, 3, 0.0, 1, True),      # a few Gaussians of thousands of tiles each
])
def test_instance_lists_are_the_sorted_emission(n, W, H, L, mu, views, sync):
    """Pairs in (view, depth, gid) order, offsets their running sum, instances a
    stable sort by key of the emission, each pair's instances the tiles of its
    rectangle times the ranks of its cells, without repetition."""
    r = raster.Rasterizer()
    p = raster.to_device(scenes.scene_uniform(n, seed=n, D=0, mu_s=mu))
    kd = r.kd_partition(p, L)
    cams = [scenes.orbit_camera(3.0, 0.3 + v, 0.3, W, H) for v in range(views)]
    st = r.forward(p, kd, cams, 5e-5)
    if not sync:
        st = r.forward(p, kd, cams, 5e-5, no_sync=True)
        assert st.overflow() == 0
    b, V = st.bins, views
    npair, ninst, nslot = (int(x) for x in b["counters"][:3].cpu())
    count = st.proj["count"][: V * n].cpu().numpy().view(np.uint32).astype(np.int64)
    depth = st.proj["depth"][: V * n].cpu().numpy()
    vis = np.nonzero(count)[0]
    order = vis[np.lexsort((vis, depth[vis], vis // n))]
    assert npair == len(vis) and ninst == count.sum()
    assert np.array_equal(b["pair_src"][:npair].cpu().numpy().view(np.uint32), order)
    off = np.concatenate([[0], np.cumsum(count[order])])
    assert np.array_equal(b["pair_off"][: npair + 1].cpu().numpy().view(np.uint32), off)
    assert np.array_equal(b["pair_rank"].cpu().numpy()[order], np.arange(npair))
    keys = b["keys"][:ninst].cpu().numpy().view(np.uint32).astype(np.int64)
    vals = b["vals"][:ninst].cpu().numpy().view(np.uint64)
    j, src = (vals & np.uint64(0xFFFFFFFF)).astype(np.int64), (vals >> np.uint64(32)).astype(np.int64)
    assert np.array_equal(np.lexsort((j, keys)), np.arange(ninst))  # sorted by key, ties in emission order
    assert np.array_equal(np.sort(j), np.arange(ninst))
    pair = np.searchsorted(off, j, side="right") - 1
    assert np.array_equal(order[pair], src)
    # every pair's keys are distinct, its tiles inside its rectangle, its ranks those of its cells
    K = 1 << L
    assert len(np.unique(pair * (1 << 32) + keys)) == ninst
    rec = st.proj["bin"][: 8 * V * n].view(V * n, 8).cpu().numpy().view(np.uint32)
    rect = np.ascontiguousarray(rec[:, :2]).view(np.int16).astype(np.int64)
    mask = np.ascontiguousarray(rec[:, 4:6]).view(np.uint64)[:, 0]
    ranks = r.cell_ranks(kd, cams)
    tx_n = (W + 15) // 16
    per_view = tx_n * ((H + 15) // 16)
    v = src // n
    t = keys // K - v * per_view
    assert np.all((t >= 0) & (t < per_view))
    tx, ty = t % tx_n, t // tx_n
    q = rect[src]
    assert np.all((tx >= q[:, 0] >> 4) & (tx <= q[:, 1] >> 4) & (ty >= q[:, 2] >> 4) & (ty <= q[:, 3] >> 4))
    cell = np.argsort(ranks, 1)[v, keys % K]
    assert np.all((mask[src] >> cell.astype(np.uint64)) & np.uint64(1))
    # slots: the runs of equal keys
    start = np.nonzero(np.concatenate([[True], np.diff(keys) != 0]))[0]
    assert nslot == len(start)
    assert np.array_equal(b["slot_range"][: 2 * nslot].cpu().numpy().reshape(-1, 2),
                          np.stack([start, np.append(start[1:], ninst)], 1))


@pytest.mark.parametrize("n,W,H,L,mu,eps,stats,hot", [
    (20000, 256, 256, 0, -3.4, 5e-5, False, False),   # one slot per tile, 256 tiles: all split
    (20000, 250, 150, 3, -3.4, 5e-5, False, False),   # several slots, ragged edges
    (6000, 250, 150, 2, -2.2, 1e-2, True, False),     # long lists that stop early; the counters
    (6000, 130, 70, 2, -2.2, 0.0, False, False),      # never stop
    (20000, 250, 150, 3, -3.4, 5e-5, False, True),    # colours that are not finite
    (3, 16, 16, 1, -1.0, 5e-5, False, False),         # fewer instances than a wave's group of four
])
def test_split_tiles_equal_whole_tiles(n, W, H, L, mu, eps, stats, hot):
    """The tiles of the longest lists are walked by four blocks of 4x4-pixel waves, the
    others by one: a view alone (at most 256 tiles, all split) has the bits that it
    has in a batch, where most tiles are whole."""
    r = raster.Rasterizer()
    p = scenes.scene_uniform(n, seed=n + W, D=1, mu_s=mu)
    if hot:
        p["sh"][:, ::100] = float("inf")
    p = raster.to_device(p)
    kd = r.kd_partition(p, L)
    per_view = ((W + 15) // 16) * ((H + 15) // 16)
    V = min(1024 // per_view + 2, 16)
    cams = [scenes.orbit_camera(3.0, 0.3 + 0.5 * v, 0.3, W, H) for v in range(V)]
    pairs = [torch.zeros(2, dtype=torch.int64, device="cuda") if stats else None for _ in range(2)]
    batch = r.forward(p, kd, cams, eps, stats=pairs[0])
    keep = [t.clone() for t in (batch.image, batch.T_final, batch.parts["C"], batch.parts["T"], batch.parts["last"])]
    keys, nslot = batch.bins["slot_key"].clone(), int(batch.bins["counters"][2])
    at = 0
    for v, cam in enumerate(cams):
        st = r.forward(p, kd, [cam], eps, stats=pairs[1])
        m = int(st.bins["counters"][2])
        assert torch.equal(keys[at: at + m].long() - v * per_view * (1 << L), st.bins["slot_key"][:m].long())
        for kept, own, w, first in ((keep[0], st.image, 3 * W * H, 3 * v * W * H),
                                    (keep[1], st.T_final, W * H, v * W * H),
                                    (keep[2], st.parts["C"], 768 * m, 768 * at),
                                    (keep[3], st.parts["T"], 256 * m, 256 * at),
                                    (keep[4], st.parts["last"], 256 * m, 256 * at)):
            a, b = kept.view(-1)[first: first + w], own.view(-1)[:w]
            a, b = a.view(torch.int32), b.view(torch.int32)
            nan = (a & 0x7FFFFFFF) > 0x7F800000  # any NaN for a NaN
            assert torch.equal(nan, (b & 0x7FFFFFFF) > 0x7F800000)
            assert torch.equal(a[~nan], b[~nan])
        at += m
    assert at == nslot
    assert not stats or torch.equal(pairs[0], pairs[1])


@pytest.mark.parametrize("H,W", [
    (1500, 1888),    # 16 full strips
    (2003, 1405),    # a partial last strip and segment
    (131, 20901),    # short segments: 118 columns, 32 rows and 3
    (20901, 131),    # too narrow for strips: tiles
])
def test_large_view_loss(rast, H, W):
    """The one-pass SSIM of large views: against the oracle, and a value that is not
    finite changes the gradient within ten pixels of it only."""
    rng = np.random.default_rng(H)
    x = rng.uniform(size=(3, H, W)).astype(np.float32)
    y = rng.uniform(size=(3, H, W)).astype(np.float32)
    xd, yd = torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda()
    lv, d = rast.loss(xd, yd, 0.2)
    ol, od = oracle.loss(x.astype(np.float64), y.astype(np.float64), 0.2)
    assert abs(lv.item() - ol) <= 1e-5 * abs(ol)
    ok, info = grad_close(d.cpu().numpy(), od, 1e-3, "dimage %dx%d" % (W, H))
    assert ok, info
    far = torch.ones_like(xd, dtype=torch.bool)
    for c, py, px, v in ((0, 0, 0, float("nan")), (1, H // 2, W // 2, float("inf")), (2, H - 1, W - 1, float("nan"))):
        xd[c, py, px] = v
        far[c, max(py - 10, 0): py + 11, max(px - 10, 0): px + 11] = False
    _, e = rast.loss(xd, yd, 0.2)
    assert torch.equal(d[far], e[far])
    assert not torch.isfinite(e[~far]).all()


@pytest.mark.parametrize("reuse", [False, True])
def test_one_allocation_per_stage_equals_separate_buffers(monkeypatch, reuse):
    """Buffers carved from one allocation, and one by one (large passes): the same
    pass, the same names, and a replaced buffer is the one the backward reads."""
    p = raster.to_device(scenes.scene_uniform(3000, seed=5, D=1, mu_s=-3.0))
    cams = [scenes.orbit_camera(3.0, 0.3 + v, 0.3, 150, 90) for v in range(2)]
    d = torch.randn(3 * 2 * 150 * 90, device="cuda", generator=torch.Generator("cuda").manual_seed(1))
    got = []
    for limit in (raster.ARENA_BYTES, 0):
        monkeypatch.setattr(raster, "ARENA_BYTES", limit)
        r = raster.Rasterizer(reuse=reuse)
        kd = r.kd_partition(p, 2)
        for _ in range(2):  # the second pass knows its capacity
            st = r.forward(p, kd, cams, 5e-5)
        assert type(st.parts) is (raster.Carved if limit else dict)
        m = int(st.bins["counters"][2])
        g = r.backward(st, p, d)
        got.append([st.image, st.T_final, st.parts["C"][: 768 * m], st.bins["slot_key"][:m]] +
                   [g[k] for k in raster.PARAM_KEYS])
        names = [{k: (v.numel(), v.dtype) for k, v in x.items()} for x in (st.proj, st.bins, st.parts)]
        got[-1].append(names)
        assert all(len(x) == len(y) and all(k in x for k in y) and list(x) == list(y)
                   for x, y in zip((st.proj, st.bins, st.parts), names))
        st.parts["T"] = torch.zeros_like(st.parts["T"])
        assert st.parts_struct().T == st.parts["T"].data_ptr()
    for a, b in zip(*got):
        assert torch.equal(a, b) if isinstance(a, torch.Tensor) else a == b


@pytest.mark.parametrize("n,Ld,kind", [
    (1, 1, "normal"), (2, 6, "normal"), (85, 2, "normal"), (700, 3, "normal"),   # no room for the list; empty nodes
    (5000, 4, "equal"),          # every member matches every prefix
    (9000, 6, "grid"),           # few distinct values, both zeros
    (300000, 5, "narrow"),       # blocks with more 16-bit matches than the list takes
    (300000, 6, "normal"),       # the list; 64 cells, two mask words
    (70000, 3, "odd"),           # centres and scales that are not finite
])
@pytest.mark.parametrize("rule", [0, 1])
def test_partition_at_its_edges(rast, n, Ld, kind, rule):
    """Splits, leaves, counts, ownership and bounds against the oracle, bit for bit."""
    rng = np.random.default_rng(n + Ld)
    p = scenes.scene_uniform(n, seed=n, D=0, mu_s=-3.0)
    m = rng.normal(size=(3, n)).astype(np.float32) * 50
    if kind == "equal":
        m[:] = 1.25
    elif kind == "grid":
        m = np.round(m / 20) * 20 * np.where(rng.uniform(size=m.shape) < 0.5, 1, -1)
    elif kind == "narrow":
        m = 1000 + rng.uniform(size=m.shape) * 3
    p["means"] = np.ascontiguousarray(m, np.float32)
    if kind == "odd":
        p["means"][0, :40], p["means"][1, 40:80] = np.inf, -np.inf
        p["log_scales"][1, 100:200] = 200.0
        p["log_scales"][2, 150:300] = -np.inf
    kd = rast.kd_partition(raster.to_device(p), Ld, rule=rule)
    o = oracle.kd_partition(p["means"], p["log_scales"], Ld, 3.0, rule=rule)
    K = 1 << Ld
    assert np.array_equal(kd.split.cpu().numpy()[: K - 1].view(np.uint32), o["split"].view(np.uint32))
    assert np.array_equal(kd.center_cell.cpu().numpy(), o["center_cell"])
    assert np.array_equal(kd.counts.cpu().numpy(), o["counts"])
    own = kd.own_mask.cpu().numpy().view(np.uint32).reshape(o["own_mask"].shape)
    assert np.array_equal(own, o["own_mask"])
    b = kd.cell_bounds_host
    smax = np.exp(p["log_scales"].astype(np.float64)).astype(np.float32).max(0)
    for k in range(K):
        sel = o["center_cell"] == k
        lo, hi, sc = ((p["means"][:, sel].min(1), p["means"][:, sel].max(1), smax[sel].max()) if sel.any()
                      else (np.inf, -np.inf, 0.0))
        assert np.array_equal(b[0:3, k], np.broadcast_to(lo, 3)) and np.array_equal(b[3:6, k], np.broadcast_to(hi, 3))
        assert b[6, k] == sc


@pytest.mark.parametrize("n", [1, 63, 4095, 4096, 4097, 70001])
def test_kept_pairs_in_index_order(rast, n):
    """The compaction's bit words at tile and word edges: the pairs of a pass are the
    kept Gaussians, by depth, ties in index order."""
    p = scenes.scene_uniform(n, seed=n, D=0, mu_s=-4.0)
    p["means"][2] = np.round(p["means"][2] * 4) / 4  # many equal depths
    cam = scenes.orbit_camera(3.0, 0.3, 0.0, 96, 64)
    p = raster.to_device(p)
    st = rast.forward(p, rast.kd_partition(p, 1), [cam], 5e-5)
    count, depth = st.proj["count"][:n].cpu().numpy(), st.proj["depth"][:n].cpu().numpy()
    kept = np.nonzero(count)[0]
    m = int(st.bins["counters"][0])
    assert m == len(kept)
    assert np.array_equal(st.bins["pair_src"][:m].cpu().numpy(), kept[np.argsort(depth[kept], kind="stable")])


def test_many_slots_launch_order(rast):
    """From 65536 slots on the launch order's tables take more slots per block: the
    first view has the gradients it has alone (the other views' image gradients are
    zero; a later view's instances lie elsewhere in the waves of the pair sums)."""
    W, H, L = 640, 480, 6
    p = raster.to_device(scenes.scene_uniform(40000, seed=3, D=1, mu_s=-3.0))
    kd = rast.kd_partition(p, L)
    cams = [scenes.orbit_camera(3.0, 0.3 + 0.4 * v, 0.3, W, H) for v in range(16)]
    d = torch.randn(3 * W * H, device="cuda", generator=torch.Generator("cuda").manual_seed(1))
    r = raster.Rasterizer()
    a = r.forward(p, kd, cams[:1], 5e-5)
    ga = r.backward(a, p, d)
    b = r.forward(p, kd, cams, 5e-5)
    assert int(a.bins["counters"][2]) < 65536 <= int(b.bins["counters"][2])
    z = torch.zeros(16, 3 * W * H, device="cuda")
    z[0] = d
    gb = r.backward(b, p, z.view(-1))
    for k in raster.PARAM_KEYS:
        assert torch.equal(ga[k], gb[k]) and torch.count_nonzero(ga[k]) > 0, k


@pytest.mark.parametrize("n,mu,W,H", [(50, 0.0, 640, 480), (3000, -2.0, 333, 201), (40000, -3.5, 333, 201), (1, -1.0, 40, 24)])
def test_pair_sums_of_the_records(monkeypatch, n, mu, W, H):
    """Pairs inside a wave, spanning waves, and waves without a record: the sums of the
    backward's records, against a float64 sum of those in the workspace."""
    r = raster.Rasterizer()
    p = raster.to_device(scenes.scene_uniform(n, seed=n, D=0, mu_s=mu))
    st = r.forward(p, r.kd_partition(p, 3), [scenes.orbit_camera(3.0, 0.3, 0.3, W, H)], 1e-2)
    spaces = []
    empty = raster.Rasterizer._empty

    def kept(self, size, dtype):
        t = empty(self, size, dtype)
        if dtype == torch.uint8:
            spaces.append(t)
        return t
    monkeypatch.setattr(raster.Rasterizer, "_empty", kept)
    g = r.backward(st, p, torch.randn(3 * W * H, device="cuda", generator=torch.Generator("cuda").manual_seed(2)))
    ws, cap = spaces[-1], st.bins_struct.capacity
    up = lambda x: (x + 255) & ~255
    nw = (cap + 63) // 64
    at = up(cap * 36) + up(cap * 48) + up(nw * 96) + up(nw * 4)
    npair, ninst = (int(x) for x in st.bins["counters"][:2].cpu())
    words = ws[at: at + 8 * ((ninst + 63) // 64)].cpu().numpy()
    has = np.unpackbits(words, bitorder="little")[:ninst].astype(bool)
    rec = ws[: 36 * ninst].view(torch.float32).view(ninst, 9).cpu().numpy().astype(np.float64)
    rec[~has] = 0.0
    off = st.bins["pair_off"][: npair + 1].cpu().numpy().view(np.uint32).astype(np.int64)
    src = st.bins["pair_src"][:npair].cpu().numpy()
    want, mag = np.zeros((n, 9)), np.zeros((n, 9))
    for q in range(npair):
        want[src[q]] = rec[off[q]: off[q + 1]].sum(0)
        mag[src[q]] = np.abs(rec[off[q]: off[q + 1]]).sum(0) * (64 + (off[q + 1] - off[q]) // 64)
    got = g["_dproj"][: 9 * n].view(9, n).cpu().numpy().T.astype(np.float64)
    assert has.any() and np.all(np.abs(got - want) <= 2.0 ** -24 * mag)
