"""The network under torch's scripting and tracing tools, and on empty volumes, on the CPU: what torch's
own operators take."""
import pytest

torch = pytest.importorskip("torch")
N = pytest.importorskip("paper_2201_02309_amd.network")


@pytest.fixture
def net():
    torch.manual_seed(2)
    return N.SubNet(channels=4, blocks=2)


X = (1, 1, 3, 5, 6)


def test_script(net):
    x = torch.randn(X)
    s = torch.jit.script(net)
    for shape in (X, (2, 1, 1, 7, 4)):
        v = torch.randn(shape)
        assert torch.equal(s(v), net(v))
    for a, b in zip(torch.autograd.grad(s(x).square().sum(), tuple(s.parameters())),
                    torch.autograd.grad(net(x).square().sum(), tuple(net.parameters()))):
        assert torch.allclose(a, b, rtol=1e-5, atol=1e-5)


@pytest.mark.parametrize("grad", [True, False])
def test_symbolic_trace(net, grad):
    x = torch.randn(X)
    with torch.set_grad_enabled(grad):
        traced = torch.fx.symbolic_trace(net)
        assert torch.equal(traced(x), net(x))


@pytest.mark.parametrize("shape", [(1, 1, 0, 5, 6), (0, 1, 3, 5, 6)])
def test_empty_volumes(net, shape):
    x = torch.randn(shape, requires_grad=True)
    y = net(x)
    assert y.shape == shape
    y.sum().backward()
    assert x.grad.shape == shape and all(bool((p.grad == 0).all()) for p in net.parameters())


def test_frozen_layer_keeps_no_input(monkeypatch):
    """The input's gradient needs the weights alone, so the input may change before the backward: the
    layer's own function with the kernels' part done by torch."""
    def stack(x):
        B, C, D, H, W = x.shape
        xp = torch.nn.functional.pad(x, (0, 0, 0, 0, 1, 1))
        return torch.cat([xp[:, :, k:k + D] for k in range(3)], 1).permute(0, 2, 1, 3, 4).reshape(B * D, 3 * C, H, W)
    m = N.Conv3x3x3(2, 3).requires_grad_(False)
    x = torch.randn(1, 2, 3, 5, 6, requires_grad=True)
    want = torch.autograd.grad(m(x).sum(), x)[0]
    gate = iter([True, False])                    # the forward's decision, the backward's
    monkeypatch.setattr(N, "_native_conv", lambda *a: next(gate))
    monkeypatch.setattr(N._K, "stack3", stack)
    h = x * 1
    y = m(h)
    assert type(y.grad_fn).__name__ == "_Conv3FnBackward"
    h.add_(1)
    assert torch.allclose(torch.autograd.grad(y.sum(), x)[0], want, rtol=1e-5, atol=1e-6)
