"""The angle error of a map against itself is exactly zero, as the difference
of two equal angles is."""
import math

import pytest

import paper_2209_08241_amd as bn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W", [(1, 1), (37, 53), (480, 640)])
@pytest.mark.parametrize("scale", [1.0, 3e-20, 7e18])
def test_equal_maps(H, W, scale):
    import torch
    gen = torch.Generator(device="cuda")
    gen.manual_seed(H)
    a = torch.randn((H, W, 3), device="cuda", generator=gen) * scale
    m = (torch.rand((H, W), device="cuda", generator=gen) < 0.3).to(torch.uint8)
    assert bn.angle_mse(a, m, a.clone(), m) == (0.0, 0.0, int((m == 0).sum()))


def test_equal_special_vectors():
    import torch
    v = [0.0, -0.0, 1.0, -1.0, 1e-40, math.inf, -math.inf]
    a = torch.tensor([[[x, y, z] for z in v] for x in v for y in v], device="cuda")
    m = torch.zeros(a.shape[:2], dtype=torch.uint8, device="cuda")
    assert bn.angle_mse(a, m, a.clone(), m) == (0.0, 0.0, m.numel())
