"""The adjoint's vector kernel on rows of any width, stride and alignment:
stacks large enough to take it, bit for bit against single frames (scalar
tiles)."""
import numpy as np
import pytest

import paper_2209_08241_amd as bn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("alpha", [1, 2, 3, 4])
@pytest.mark.parametrize("H,W,pad,shift", [(97, 131, 0, 0), (112, 118, 3, 1), (33, 389, 0, 2),
                                           (17, 1030, 5, 3), (260, 57, 0, 0), (2600, 5, 1, 1),
                                           (64, 225, 7, 1), (129, 228, 0, 1), (9, 1537, 0, 0),
                                           (40, 448, 0, 0)])
def test_ragged_stacks_equal_single_frames(H, W, pad, shift, alpha):
    import torch
    n = 64   # every size reaches the vector kernel for alpha <= 2, most for 3 and 4
    gen = torch.Generator(device="cuda")
    gen.manual_seed(H * W + alpha)
    stride = W + pad
    # the last row ends the buffer: nothing behind it may be read into a result
    flat = torch.empty(shift + n * H * stride - pad, device="cuda")
    d = torch.as_strided(flat, (n, H, W), (H * stride, stride, 1), shift)
    flat.fill_(float("nan"))
    v = 1.5 + 0.3 * torch.rand((n, H, W), device="cuda", generator=gen)
    v[torch.rand((n, H, W), device="cuda", generator=gen) < 0.03] = 0.0
    d.copy_(v)
    g = torch.randn((n, H, W, 3), device="cuda", generator=gen)
    out = torch.full((n * H * W + 2 * shift,), 5.0, device="cuda")
    gd = out[shift:shift + n * H * W].view(n, H, W)
    intr = [(150.0 + k, 160.0, (W - 1) / 2, (H - 1) / 2) for k in range(n)]
    bn.normals_vjp_stack(d, intr, g, alpha, "rel", 1.1, grad_depth=gd)
    torch.cuda.synchronize()
    if shift:
        assert bool((out[:shift] == 5.0).all()) and bool((out[-shift:] == 5.0).all())
    for k in (0, 1, n // 2, n - 1):
        one = bn.normals_vjp(d[k], *intr[k], g[k], alpha, "rel", 1.1)
        assert np.array_equal(gd[k].cpu().numpy().view(np.uint32), one.cpu().numpy().view(np.uint32))
