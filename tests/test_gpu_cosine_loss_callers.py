"""The fused cosine loss under callers that hand its gradient on lazily or
compile it."""
import pytest

import paper_2209_08241_amd as bn
from test_gpu_cosine_loss import maps, reference

pytestmark = pytest.mark.gpu


def close(got, want):
    # one quotient and one product in binary32
    return float((got.double() - want).abs().max()) <= 4 * 2.0 ** -24 * float(want.abs().max())


def test_an_incoming_gradient_that_is_negated_lazily():
    """The imaginary part of a conjugate is a view with the negative bit set:
    its memory holds the opposite sign."""
    import torch
    n, t, m, tm = maps((5, 333), 11)
    _, rg = reference(n, t, m, tm)
    x = n.detach().requires_grad_(True)
    lazy = torch.tensor(1.0 + 2.0j, device="cuda").conj().imag
    assert lazy.is_neg()
    bn.cosine_loss(x, t, m, tm).backward(lazy)
    assert close(x.grad, -2.0 * rg)
    # the same through complex arithmetic on the loss
    x.grad = None
    z = torch.complex(torch.ones((), device="cuda"), bn.cosine_loss(x, t, m, tm)).conj()
    torch.view_as_real(z.resolve_conj())[1].backward()
    assert close(x.grad, -rg)


@pytest.mark.parametrize("grad", [False, True])
def test_a_compiled_loss(grad):
    import torch
    n, t, m, tm = maps((6, 40), 9)
    rl, rg = reference(n, t, m, tm)
    x = n.detach().requires_grad_(grad)
    torch._dynamo.reset()
    loss = torch.compile(bn.cosine_loss, backend="aot_eager", fullgraph=True)(x, t, m, tm)
    # 240 terms of up to 2, summed in binary32
    assert abs(float(loss.detach()) - float(rl)) <= 240 * 2.0 ** -24 * 2
    if grad:
        loss.backward()
        assert close(x.grad, rg)
