"""The binding's call path: workspace sizes it keeps follow the handle's
options, and outputs are contiguous whatever the strides of the input."""
import pytest
import torch

from paper_2609_01864_amd import autograd as A
from paper_2609_01864_amd import credit as C

pytestmark = pytest.mark.gpu


def test_kept_sizes_follow_the_options(lib_built):
    h = C.Handle(0)
    try:
        x = torch.randn(512, 4096, device="cuda")
        dy = torch.randn_like(x)
        g = torch.rand(4096, device="cuda") + 0.5
        mean, rstd = x.mean(1), torch.rsqrt(x.var(1, correction=0) + 1e-5)
        p = C.plan("resident")
        h.set_option(C.OPT_MAX_GROUPS, 1)
        small = h._call_ws(C.LAYERNORM, C.BWD, C.F32, 512, 4096, p, h._stream()).numel()
        one = C.layernorm_bwd(x, dy, g, mean, rstd, p=p, h=h)
        h.set_option(C.OPT_MAX_GROUPS, 0)
        many = C.layernorm_bwd(x, dy, g, mean, rstd, p=p, h=h)  # more partial rows: a larger workspace
        torch.cuda.synchronize()
        assert h._ws[h._stream()].numel() >= h.workspace_size(C.LAYERNORM, C.BWD, C.F32, 512, 4096, p) > small // 2
        # sums of 512 FP32 terms in another order
        for a, b in ((one[0], many[0]), (one[2], many[2]), (one[3], many[3])):
            assert torch.allclose(a, b, rtol=0, atol=512 * 2.0 ** -24 * 8)
    finally:
        h.close()


@pytest.mark.parametrize("shape", [(3, 40), (2, 3, 40), (40,)])
def test_autograd_shapes_and_strides(gpu_handle, shape):
    base = torch.randn(*shape[:-1], 2 * shape[-1], device="cuda")
    x = base[..., ::2].detach().requires_grad_(True)  # strided: made contiguous
    g, b = (torch.rand(shape[-1], device="cuda").requires_grad_(True) for _ in range(2))
    y = A.layer_norm(x, g, b)
    dy = torch.randn(shape, device="cuda")
    got = torch.autograd.grad(y, (x, g, b), dy)
    xd, gd, bd = (t.detach().double().requires_grad_(True) for t in (x, g, b))
    yd = torch.nn.functional.layer_norm(xd, shape[-1:], gd, bd, 1e-5)
    ref = torch.autograd.grad(yd, (xd, gd, bd), dy.double())
    assert y.shape == x.shape and y.is_contiguous() and got[0].shape == x.shape
    for a, r in zip((y, *got), (yd, *ref)):
        assert torch.max(torch.abs(a.double() - r)).item() <= 1e-5 * max(1.0, r.abs().max().item())
    s = A.softmax(x)
    assert s.shape == x.shape and torch.allclose(s.double(), torch.softmax(x.detach().double(), -1), atol=2e-6)
