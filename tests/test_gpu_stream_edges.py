"""The stream encoding's kernels where their special branches meet the edges
of what a caller may hand over."""
import sys

import numpy as np
import pytest
import torch

from tests.helpers import azint

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
def test_gradient_towards_raw_of_masked_pixels(dtype, dev):
    """A norm of zero, of an infinity or below zero, on pixels that feed bins,
    on pixels that feed none, and on whole tiles that feed none: the values and
    signs of the adjoint over the pixel-major entries."""
    say("masked gradient", dtype)
    az = azint()
    h, w, npt = 200, 260, 37
    kw = dict(range=(5e-4, 2e-3), dtype=dtype, device=dev)
    stream, entries = az.Plan(h, w, npt, **kw), az.Plan(h, w, npt, layout="pixel", **kw)
    gen = np.random.default_rng(21)
    flat = gen.uniform(0.9, 1.1, h * w)
    mask = gen.random(h * w) < 0.2
    flat[mask] = gen.choice([0.0, -0.0, -1.5, np.inf, -np.inf, np.nan], mask.sum())
    flat = torch.from_numpy(flat).to(dtype).to(dev)
    x = torch.from_numpy(gen.uniform(0, 1, h * w)).to(dtype).to(dev)
    U = stream.integrate(x)[2]
    g = torch.from_numpy(gen.standard_normal((2, npt))).to(dtype).to(dev)
    out = []
    for p in (stream, entries):
        p.set_corrections(flat=flat)
        out.append(p.backward(U, g[0].contiguous(), g[1].contiguous(), wrt_raw=True))
    a, b = out
    torch.cuda.synchronize()
    assert torch.equal(torch.isnan(a), torch.isnan(b))
    keep = ~torch.isnan(b)
    assert torch.equal(a[keep], b[keep])
    assert torch.equal(torch.signbit(a[keep]), torch.signbit(b[keep]))
    assert bool(torch.isnan(a).any())
