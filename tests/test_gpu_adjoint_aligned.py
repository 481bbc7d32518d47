"""The adjoint's vector kernel on aligned rows of few columns or few rows:
stacks large enough to take it, every frame bit for bit against the
single-frame call (few pixels: scalar tiles) and one against the oracle."""
import numpy as np
import pytest

import oracle
import paper_2209_08241_amd as bn
from test_gpu_adjoint import vjp_tol
from test_gpu_adjoint_ragged import test_ragged_stacks_equal_single_frames as check_ragged

pytestmark = pytest.mark.gpu

N = 64   # frames: the vector kernel serves more than 3 * 2^17 (alpha 3, 4: 3 * 2^18) pixels


# widths on and off the strips of 224 columns, heights on and off the bands of
# 16, 24 and 32 rows (4 wavefronts) and of 32 and 48 (8, from 512 workgroups on)
@pytest.mark.parametrize("H,W", [(3100, 4), (1541, 8), (1057, 12), (60, 224), (57, 228), (49, 252),
                                 (31, 448), (33, 452), (13, 996), (9, 1992), (3, 4480),
                                 (17, 1200), (1, 12320)])
@pytest.mark.parametrize("alpha", [1, 2, 3, 4])
def test_aligned_stacks_equal_single_frames(H, W, alpha):
    import torch
    line = (3 << 17) if alpha <= 2 else (3 << 18)
    assert N * H * W > line >= H * W
    gen = torch.Generator(device="cuda")
    gen.manual_seed(H * W + alpha)
    d = 1.0 + 0.3 * torch.rand((N, H, W), device="cuda", generator=gen)
    d[torch.rand((N, H, W), device="cuda", generator=gen) < 0.02] = 0.0
    g = torch.randn((N, H, W, 3), device="cuda", generator=gen)
    intr = [(150.0 + k, 160.0, (W - 1) / 2, (H - 1) / 2) for k in range(N)]
    gd = torch.full((N, H, W), 5.0, device="cuda")
    bn.normals_vjp_stack(d, intr, g, alpha, "rel", 1.1, grad_depth=gd)
    for k in range(0, N, 7):
        one = bn.normals_vjp(d[k], *intr[k], g[k], alpha, "rel", 1.1)
        assert torch.equal(gd[k].view(torch.int32), one.view(torch.int32)), k
    k = N - 1
    o = oracle.default()
    dk = d[k].cpu().numpy()
    codes = o.normals_f32(dk, *intr[k], alpha, "rel", 1.1)["mask"]
    ref = o.normals_vjp_f64(dk, *intr[k], alpha, codes, g[k].cpu().numpy().astype(np.float64))
    assert np.all(np.abs(gd[k].cpu().numpy() - ref) <= vjp_tol(ref))


@pytest.mark.parametrize("alpha", [1, 4])
@pytest.mark.parametrize("H,W,pad,shift", [(130, 131, 0, 0), (141, 118, 3, 1), (49, 389, 0, 2),
                                           (300, 57, 0, 0), (3400, 5, 1, 1), (75, 225, 7, 1),
                                           (12, 1537, 0, 0), (1, 16389, 0, 3)])
def test_ragged_stacks_above_their_line(H, W, pad, shift, alpha):
    """Ragged rows take the vector kernel from 2^20 pixels (alpha 1) and 7 * 2^17
    (alpha 4) on."""
    assert N * H * W > 1 << 20
    check_ragged(H, W, pad, shift, alpha)
