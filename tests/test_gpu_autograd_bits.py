"""Tensors that torch negates or conjugates only when they are read (its conj
and neg bits) through the differentiable form: the forward of such an input,
the gradient that arrives as one (the adjoint of conj() is a conj()), on both
routes of the backward, against a gather."""
import pytest

import paper_1708_01873_amd as br
from paper_1708_01873_amd.autograd import bitrev

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


@pytest.mark.parametrize("dtype", (torch.complex64, torch.complex128))
def test_forward_of_a_lazy_conjugate(dtype):
    z = torch.randn(3, 1 << 7, dtype=dtype, device="cuda")
    x = z.conj()
    assert x.is_conj() and x.is_contiguous()
    assert torch.equal(bitrev(x), x.resolve_conj()[..., _rev(7)])
    assert x.is_conj()


def test_forward_of_a_lazy_negative():
    x = torch._neg_view(torch.randn(2, 1 << 6, device="cuda"))
    assert x.is_neg() and x.is_contiguous()
    assert torch.equal(bitrev(x), x.resolve_neg()[..., _rev(6)])


@pytest.mark.parametrize("create_graph", (False, True))
@pytest.mark.parametrize("dtype", (torch.complex64, torch.complex128))
def test_gradient_that_arrives_conjugated(dtype, create_graph):
    idx = _rev(8)
    z = torch.randn(2, 1 << 8, dtype=dtype, device="cuda", requires_grad=True)
    w = torch.randn(2, 1 << 8, dtype=dtype, device="cuda")
    seen = []
    y = bitrev(z)
    y.register_hook(lambda g: seen.append(g.is_conj()))
    (got,) = torch.autograd.grad(y.conj(), z, w, create_graph=create_graph)
    (want,) = torch.autograd.grad(z[..., idx].conj(), z, w)
    assert seen == [True]
    assert torch.equal(got, want)
