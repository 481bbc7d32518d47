"""The fused cosine loss and its gradient against 64-bit tensor operations:
tile remainders, unaligned maps, masks, special values, and the calls that
keep going through tensor operations (second derivatives, transforms)."""
import math

import pytest

import paper_2209_08241_amd as bn

pytestmark = pytest.mark.gpu


def maps(shape, seed, offset=0):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    px = math.prod(shape)

    def rows(n, dtype):
        # `offset` elements into a larger buffer: any alignment of the element type
        flat = torch.empty(n + offset, dtype=dtype, device="cuda")
        return flat[offset:]

    n, t = rows(3 * px, torch.float32), rows(3 * px, torch.float32)
    for v in (n, t):
        v.copy_(torch.nn.functional.normalize(torch.randn((px, 3), device="cuda", generator=g),
                                              dim=-1).reshape(-1))
    m, tm = rows(px, torch.uint8), rows(px, torch.uint8)
    for v in (m, tm):
        v.copy_(torch.randint(0, 4, (px,), device="cuda", generator=g).clamp(min=1) - 1)
    return (n.view(*shape, 3), t.view(*shape, 3), m.view(shape), tm.view(shape))


def reference(n, t, m, tm):
    import torch
    x = n.detach().double().requires_grad_(True)
    U = (m == 0) & (tm == 0)
    cos = (x * t.double()).sum(-1)
    loss = torch.where(U, 1.0 - cos, torch.zeros_like(cos)).sum() / U.sum().clamp(min=1)
    loss.backward()
    return loss.detach(), x.grad


@pytest.mark.parametrize("shape", [(1,), (3,), (1, 4), (5, 51), (2, 1023), (2048,), (2049,),
                                   (4, 4097), (3, 480, 641), (16, 480, 640)])
@pytest.mark.parametrize("offset", [0, 1, 4])
def test_loss_and_gradient(shape, offset):
    import torch
    n, t, m, tm = maps(shape, sum(shape) + offset, offset)
    x = n.detach().requires_grad_(True)
    loss = bn.cosine_loss(x, t, m, tm)
    (2.5 * loss).backward()
    rl, rg = reference(n, t, m, tm)
    assert loss.shape == () and loss.dtype == torch.float32
    # the terms are rounded to binary32 (a few 2^-24 of values up to 2) and
    # averaged in 64 bits; the gradient is one quotient and one product
    assert abs(float(loss.detach()) - float(rl)) <= 8 * 2.0 ** -24 * 2
    assert float((x.grad.double() - 2.5 * rg).abs().max()) <= 4 * 2.0 ** -24 * float(
        (2.5 * rg).abs().max())
    with torch.no_grad():
        assert torch.equal(bn.cosine_loss(n, t, m, tm), loss.detach())


def test_special_values_and_an_empty_mask():
    import torch
    n, t, m, tm = maps((7, 64), 1)
    n[0, 0] = float("nan")
    t[1, 1] = float("inf")
    m[0, 0] = 2
    m[1, 1] = 1                       # masked: neither reaches the loss
    x = n.detach().requires_grad_(True)
    loss = bn.cosine_loss(x, t, m, tm)
    loss.backward()
    U = (m == 0) & (tm == 0)
    w = torch.where(U, -1.0 / U.sum(), 0.0)
    want = w[..., None] * t           # 0 times a special target, as tensor operations give it
    assert math.isfinite(float(loss))
    assert torch.allclose(x.grad, want, rtol=1e-6, atol=0, equal_nan=True)
    n[2, 2] = float("nan")
    m[2, 2] = tm[2, 2] = 0
    assert math.isnan(float(bn.cosine_loss(n, t, m, tm)))
    m.fill_(1)
    assert float(bn.cosine_loss(n, t, m, tm)) == 0.0


def test_mask_buffers_may_be_reused_before_the_backward_pass():
    import torch
    n, t, m, tm = maps((5, 333), 4)
    x = n.detach().requires_grad_(True)
    _, rg = reference(n, t, m, tm)
    loss = bn.cosine_loss(x, t, m, tm)
    m.fill_(2)
    tm.fill_(2)
    loss.backward()
    assert float((x.grad.double() - rg).abs().max()) <= 4 * 2.0 ** -24 * float(rg.abs().max())


def test_calls_that_stay_tensor_operations():
    import torch
    n, t, m, tm = maps((6, 40), 9)
    rl, rg = reference(n, t, m, tm)
    # double precision, a target that wants a gradient, an empty map
    assert abs(float(bn.cosine_loss(n.double(), t.double(), m, tm)) - float(rl)) < 1e-12
    tt = t.detach().requires_grad_(True)
    bn.cosine_loss(n, tt, m, tm).backward()
    assert tt.grad is not None
    assert float(bn.cosine_loss(n[:0], t[:0], m[:0], tm[:0])) == 0.0
    # a second derivative with respect to the incoming gradient
    x = n.detach().requires_grad_(True)
    s = torch.ones((), device="cuda", requires_grad=True)
    g, = torch.autograd.grad(s * bn.cosine_loss(x, t, m, tm), x, create_graph=True)
    (g * t).sum().backward()
    assert abs(float(s.grad) - float((rg * t.double()).sum())) < 1e-5
    # batched gradients, vmap, forward mode
    two, = torch.autograd.grad(bn.cosine_loss(x, t, m, tm), x,
                               torch.tensor([1.0, -2.0], device="cuda"), is_grads_batched=True)
    assert torch.allclose(two[1].double(), -2.0 * rg, atol=1e-6)
    per = torch.vmap(bn.cosine_loss)(n, t, m, tm)
    assert per.shape == (6,)
    with torch.autograd.forward_ad.dual_level():
        d = torch.autograd.forward_ad.make_dual(n, t)
        out = torch.autograd.forward_ad.unpack_dual(bn.cosine_loss(d, t, m, tm))
        assert abs(float(out.tangent) - float((rg * t.double()).sum())) < 1e-5
    # saved tensors on the host in between
    x.grad = None
    with torch.autograd.graph.save_on_cpu():
        loss = bn.cosine_loss(x, t, m, tm)
    loss.backward()
    assert float((x.grad.double() - rg).abs().max()) <= 4 * 2.0 ** -24 * float(rg.abs().max())
