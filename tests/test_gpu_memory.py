"""What a pass asks for and holds on the device."""
import pytest
import torch

from paper_2406_11836_amd import raster, scenes

pytestmark = pytest.mark.gpu


def _scene(n, mu, D=1):
    return raster.to_device(scenes.scene_uniform(n, seed=n, D=D, mu_s=mu))


def test_memory_of_a_pass_with_a_large_capacity():
    """Between the passes: the instance lists (12 bytes per instance of capacity), not
    the sort's workspace; in the backward: a 36-byte record and the sums of 64
    instances (about 2 more), not bytes per instance for what there is per pair and per slot."""
    r = raster.Rasterizer()
    p = _scene(2000, -3.0)
    kd = r.kd_partition(p, 2)
    cam = scenes.orbit_camera(3.0, 0.3, 0.3, 160, 96)
    cap = r.capacity_hint = 20_000_000
    torch.cuda.synchronize()
    before = torch.cuda.memory_allocated()
    st = r.forward(p, kd, [cam], 5e-5)
    held = torch.cuda.memory_allocated() - before
    assert st.bins_struct.capacity == cap
    assert 12 * cap <= held <= 13 * cap
    torch.cuda.reset_peak_memory_stats()
    before = torch.cuda.memory_allocated()
    r.backward(st, p, torch.ones(3 * 160 * 96, device="cuda"))
    peak = torch.cuda.max_memory_allocated() - before
    assert 36 * cap <= peak <= 40 * cap


@pytest.mark.parametrize("n,mu,W,H,views,L,out", [
    (1, -1.0, 40, 24, 1, 0, False),         # one pair
    (40000, -5.0, 96, 64, 2, 0, False),     # more pairs than four per slot: the flags outgrow the slots' words
    (50, 0.0, 640, 480, 1, 3, False),       # few pairs, many slots, pairs that span waves
    (3000, -2.0, 333, 201, 3, 4, False),
    (500, -3.0, 64, 48, 1, 2, True),        # no instance at all
])
def test_gradients_with_either_workspace(monkeypatch, n, mu, W, H, views, L, out):
    """The workspace by slots and pairs gives the bits of the one by the capacity alone."""
    p = _scene(n, mu)
    cams = [scenes.orbit_camera(3.0, 0.3 + v, 0.3, W, H) for v in range(views)]
    if out:
        p["means"][2] += 1000.0
    d = torch.randn(3 * views * W * H, device="cuda", generator=torch.Generator("cuda").manual_seed(1))
    got, asked = [], []
    empty = raster.Rasterizer._empty

    def kept(self, size, dtype):
        if dtype == torch.uint8:
            asked[-1].append(int(size))
        return empty(self, size, dtype)
    monkeypatch.setattr(raster.Rasterizer, "_empty", kept)
    for limit in (raster.ARENA_BYTES, 0):
        monkeypatch.setattr(raster, "ARENA_BYTES", limit)
        asked.append([])
        r = raster.Rasterizer()
        kd = r.kd_partition(p, L)
        st = r.forward(p, kd, cams, 5e-5)
        g = r.backward(st, p, d)
        got.append([g[k] for k in raster.PARAM_KEYS] + [g["_dproj"]])
    cap = st.bins_struct.capacity
    assert asked[0][-1] == r.lib.rgs_render_bwd_workspace(cap)
    assert asked[1][-1] == r.lib.rgs_render_bwd_workspace_for(cap, st.slot_capacity, views * n) <= asked[0][-1]
    for a, b in zip(*got):
        assert torch.equal(a, b)
        assert out or n == 1 or torch.count_nonzero(a) > 0


def test_stream_handle(monkeypatch):
    """The current stream's handle, also where torch lacks the direct way to it."""
    side = torch.cuda.Stream()
    for names in ({}, {"_RAW_STREAM": None}, {"_DEVICE": None}):
        with monkeypatch.context() as m:
            for k, v in names.items():
                m.setattr(raster, k, v)
            assert raster._stream() == torch.cuda.current_stream().cuda_stream
            with torch.cuda.stream(side):
                assert raster._stream() == side.cuda_stream != torch.cuda.default_stream().cuda_stream


@pytest.mark.parametrize("backward", [True, False])
def test_autograd_passes_free_their_buffers(backward):
    """A pass through torch's autograd leaves nothing on the device once its outputs are
    dropped, whether it was differentiated or not."""
    r = raster.Rasterizer()
    p = _scene(3000, -3.0)
    for k in raster.PARAM_KEYS:
        p[k].requires_grad_(True)
    kd = r.kd_partition(p, 2)
    cam = scenes.orbit_camera(3.0, 0.3, 0.3, 96, 64)
    sizes = []
    for _ in range(8):
        for k in raster.PARAM_KEYS:
            p[k].grad = None
        image, T = raster.rasterize(p, [cam], kd, r)
        if backward:
            (image.sum() + T.sum()).backward()
            assert all(p[k].grad is not None for k in raster.PARAM_KEYS)
        del image, T
        sizes.append(torch.cuda.memory_allocated())
    assert sizes[-1] <= sizes[2]
