"""The backward's two routes: through BitRev.apply where it can be recorded or
transformed, the kernel itself otherwise."""
import pytest

import paper_1708_01873_amd as br
from paper_1708_01873_amd.autograd import BitRev, bitrev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    br.lib()


def _rev(k):
    r = torch.zeros(1, dtype=torch.int64, device="cuda")
    for _ in range(k):
        r = torch.cat([2 * r, 2 * r + 1])
    return r


@pytest.mark.parametrize("shape", [(1 << 9,), (3, 1 << 5), (2, 5, 1 << 11)])
def test_first_and_second_order(shape):
    idx = _rev(shape[-1].bit_length() - 1)
    x = torch.randn(*shape, device="cuda", dtype=torch.float64, requires_grad=True)
    w = torch.randn(*shape, device="cuda", dtype=torch.float64, requires_grad=True)
    y = bitrev(x)
    assert torch.equal(y, x[..., idx])
    (g,) = torch.autograd.grad(y, x, w, retain_graph=True)
    assert not g.requires_grad and torch.equal(g, w[..., idx])
    (g,) = torch.autograd.grad(y, x, w, create_graph=True)
    assert g.requires_grad and torch.equal(g, w[..., idx])
    v = torch.randn_like(w)
    (h,) = torch.autograd.grad(g, w, v)  # d<g, v>/dw = rev(v)
    assert torch.equal(h, v[..., idx])


def test_a_gradient_that_is_not_contiguous():
    x = torch.randn(4, 256, device="cuda", requires_grad=True)
    bitrev(x).sum().backward()  # an expanded gradient
    assert torch.equal(x.grad, torch.ones_like(x))
    g = torch.randn(256, 4, device="cuda").t()
    (gx,) = torch.autograd.grad(bitrev(x), x, g)
    assert torch.equal(gx, g[:, _rev(8)])


def test_hooks_and_streams_see_the_backward():
    x = torch.randn(2, 128, device="cuda", requires_grad=True)
    seen = []
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):  # the backward runs on the forward's stream
        y = BitRev.apply(x)
    torch.cuda.current_stream().wait_stream(side)
    y.register_hook(lambda g: seen.append("out"))
    x.register_hook(lambda g: seen.append("in"))
    y.backward(torch.ones_like(y))
    torch.cuda.synchronize()
    assert seen == ["out", "in"] and torch.equal(x.grad, torch.ones_like(x))


def test_batched_gradients_stay_refused():
    x = torch.randn(2, 64, device="cuda", requires_grad=True)
    y = bitrev(x)
    with pytest.raises(RuntimeError):
        torch.autograd.grad(y, x, torch.ones(3, 2, 64, device="cuda"), is_grads_batched=True)


def test_a_dual_gradient_stays_refused():
    """Forward mode over the backward: BitRev has no jvp, and a direct call
    would drop the tangent."""
    import torch.autograd.forward_ad as fw
    x = torch.randn(2, 64, device="cuda", requires_grad=True)
    y = bitrev(x)
    with fw.dual_level():
        w = fw.make_dual(torch.ones_like(y), torch.randn_like(y))
        with pytest.raises((NotImplementedError, RuntimeError)):
            torch.autograd.grad(y, x, w)
