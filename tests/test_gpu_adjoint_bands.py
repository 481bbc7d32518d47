"""The adjoint's bands of 4 and of 8 wavefronts: stacks on both sides of
the rule's line, bit for bit against single frames (scalar tiles)."""
import numpy as np
import pytest

import paper_2209_08241_amd as bn

pytestmark = pytest.mark.gpu


# 320x240 is 2 strips of 8 (alpha 3: 5) bands of 8 wavefronts: 512 workgroups
# from 32 (52) frames on; alpha 4 always takes 4 wavefronts
@pytest.mark.parametrize("alpha", [1, 2, 3, 4])
@pytest.mark.parametrize("n", [31, 32, 43, 51, 52])
@pytest.mark.parametrize("W", [320, 319])
def test_stacks_equal_single_frames(n, W, alpha):
    import torch
    H = 240
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n * W + alpha)
    d = 1.5 + 0.3 * torch.rand((n, H, W), device="cuda", generator=gen)
    d[torch.rand((n, H, W), device="cuda", generator=gen) < 0.03] = 0.0
    g = torch.randn((n, H, W, 3), device="cuda", generator=gen)
    intr = [(150.0 + k, 160.0, (W - 1) / 2, (H - 1) / 2) for k in range(n)]
    gd = torch.full((n, H, W), 5.0, device="cuda")
    bn.normals_vjp_stack(d, intr, g, alpha, "rel", 1.1, grad_depth=gd)
    for k in (0, n // 2, n - 1):
        one = bn.normals_vjp(d[k], *intr[k], g[k], alpha, "rel", 1.1)
        assert np.array_equal(gd[k].cpu().numpy().view(np.uint32), one.cpu().numpy().view(np.uint32))
