"""First bins of device-built plans (found and checked on the device).

The adjoint reads a pixel's bins from its first bin and its entry count, so it
equals the host-built plan's bit for bit where the matrices do: radius units,
bounding boxes or whole pixels. Sizes around the kernel's blocks of pixels,
pixels without entries (clipped ranges), pixels over many bins.
"""
import pytest
import torch

from tests.helpers import azint

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h,w,cy,cx,npt,split,rng", [
    (1, 1, 0.5, 0.5, 3, "bbox", None),
    (1, 255, 0.5, 9.0, 40, "bbox", None),
    (16, 16, 8.0, 8.0, 500, "bbox", None),             # many bins a pixel
    (1, 257, 0.5, 100.25, 64, "none", None),
    (61, 67, 30.0, 33.0, 50, "bbox", (1e-3, 2e-3)),    # pixels without entries
    (61, 67, 30.0, 33.0, 50, "none", (1e-3, 2e-3)),
], ids=str)
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
def test_adjoint_of_device_plan(h, w, cy, cx, npt, split, rng, dtype, dev):
    az = azint()
    kw = dict(center=(cy, cx), split=split, range=rng, dtype=dtype)
    dp = az.Plan.on_device(h, w, npt, device=dev, **kw)
    hp = az.Plan(h, w, npt, layout="band", band=4, **kw)
    hp.upload(dev)
    gen = torch.Generator().manual_seed(h * 1000 + w)
    U = (torch.rand(npt, generator=gen, dtype=torch.float64) + 0.5).to(dtype).to(dev)
    g = torch.randn(npt, generator=gen, dtype=torch.float64).to(dtype).to(dev)
    want = hp.backward(U, g)
    assert torch.equal(dp.backward(U, g), want)
    for layout in ("run", "band", "pixel"):   # leaves the builder's buffers
        dp.set_layout(layout)
        hp.set_layout(layout)
        assert torch.equal(dp.backward(U, g), hp.backward(U, g))
