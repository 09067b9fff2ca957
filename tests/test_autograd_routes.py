"""Which route the backward takes (CPU: the routes themselves need the GPU):
through the Function wherever grad mode, a functorch transform, a forward-mode
level or a trace sees it, and wherever torch does not say."""
import pytest

torch = pytest.importorskip("torch")

from paper_1708_01873_amd import autograd  # noqa: E402


def test_nothing_records():
    with torch.no_grad():
        assert not autograd._recorded()
    assert autograd._recorded()


def test_a_trace_records():
    seen = []

    def f(x):
        with torch.no_grad():
            seen.append(autograd._recorded())
        return x + 1
    torch.jit.trace(f, torch.zeros(3), check_trace=False)
    assert seen == [True]


def test_a_transform_records():
    seen = []

    def f(x):
        with torch.no_grad():
            seen.append(autograd._recorded())
        return x + 1
    torch.func.vmap(f)(torch.zeros(2, 3))
    with torch.no_grad():
        with torch.autograd.forward_ad.dual_level():
            seen.append(autograd._recorded())
    assert seen == [True, True]


@pytest.mark.parametrize("holder,name", [
    (torch._C, "_are_functorch_transforms_active"), (torch._C, "_get_tracing_state"),
    (torch.autograd.forward_ad, "_current_level")])
def test_a_torch_that_does_not_say_records(monkeypatch, holder, name):
    monkeypatch.delattr(holder, name)
    with torch.no_grad():
        assert autograd._recorded()
