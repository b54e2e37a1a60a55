"""The loss of large views of unusual shapes: the way it is computed depends on the shape,
its values do not."""
import pytest
import torch

from paper_2406_11836_amd import raster

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W", [
    (100, 60000),    # one segment per strip, one round of blocks
    (100, 20500),    # short segments, of which too few: tiles
    (300, 7000),     # just not worth the marching pass
    (600, 3400),     # just worth it
    (20000, 236),    # two strips
    (6000, 354),     # three, full
])
def test_gradient_of_a_crop(H, W):
    """Away from a crop's cut edges the gradient is that of the whole, scaled by the
    number of values (the crops take tiles: they are small)."""
    r = raster.Rasterizer()
    g = torch.Generator("cuda").manual_seed(H + W)
    x = torch.rand((3, H, W), generator=g, device="cuda")
    y = (x + 0.2 * torch.randn((3, H, W), generator=g, device="cuda")).clamp_(0, 1)
    lv, d = r.loss(x, y, 0.2)
    d = d.double() * x.numel()
    assert torch.isfinite(d).all()
    ch, cw = min(H, 700), min(W, 700)
    for y0, x0 in ((0, 0), (H - ch, W - cw), ((H - ch) // 2, (W - cw) // 2), (0, W - cw)):
        cx, cy = (t[:, y0: y0 + ch, x0: x0 + cw].contiguous() for t in (x, y))
        _, e = r.loss(cx, cy, 0.2)
        e = e.double() * cx.numel()
        top, left = (0 if y0 == 0 else 10), (0 if x0 == 0 else 10)
        bottom, right = (ch if y0 + ch == H else ch - 10), (cw if x0 + cw == W else cw - 10)
        a = d[:, y0 + top: y0 + bottom, x0 + left: x0 + right]
        b = e[:, top:bottom, left:right]
        # the scale is rounded once more per side; the sums are the same
        assert ((a - b).abs() <= 1e-5 * (1 + b.abs())).all()
    # the loss itself, in double
    l1 = (x.double() - y.double()).abs().mean()
    assert lv.item() > l1.item()
