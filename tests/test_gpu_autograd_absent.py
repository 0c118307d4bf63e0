"""Integrate1d with outputs that no loss uses: their gradients stay absent and
count as zeros; and the default stream handle follows the current stream."""
import pytest
import torch

import paper_1412_6367_amd as az

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h,w,npt", [(1, 3, 2), (37, 53, 61), (130, 141, 100)])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
def test_absent_gradients_count_as_zeros(h, w, npt, dtype, dev):
    plan = az.Plan(h, w, npt, dtype=dtype, device=dev)
    gen = torch.Generator().manual_seed(h)
    x = torch.rand(h, w, generator=gen, dtype=torch.float64).to(dtype).to(dev).requires_grad_()
    gI = torch.randn(npt, generator=gen, dtype=torch.float64).to(dtype).to(dev)
    gW = torch.randn(npt, generator=gen, dtype=torch.float64).to(dtype).to(dev)
    zero = torch.zeros_like(gI)
    for use in ((gI, None), (None, gW), (gI, gW)):
        I, W, U = az.Integrate1d.apply(x, plan, 0.0)
        pairs = [(o, g) for o, g in zip((I, W), use) if g is not None]
        (gx,) = torch.autograd.grad([o for o, _ in pairs], x, [g for _, g in pairs])
        full = [zero if g is None else g for g in use]
        assert torch.equal(gx.reshape(-1), plan.backward(U, *full))
        assert not U.requires_grad


def test_outputs_keep_their_own_storage_and_stream(dev):
    plan = az.Plan(37, 53, 61, device=dev)
    x = torch.rand(37 * 53, dtype=torch.float64, device=dev)
    outs = plan.integrate(x)
    assert len({o.untyped_storage().data_ptr() for o in outs}) == 3
    version = outs[2]._version
    outs[0].mul_(2.0)
    assert outs[2]._version == version
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        assert az._stream() == side.cuda_stream == az._stream(side)
    assert az._stream() == torch.cuda.current_stream().cuda_stream
