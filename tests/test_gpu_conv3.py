"""The network's 3x3x3 convolution on the library's matrix-core kernels against the same
convolution in float64: outputs and gradients over channel counts, tile edges and layouts, and the
ways of calling it that keep torch's operators; and PReLU's gradients."""
import pytest

torch = pytest.importorskip("torch")
N = pytest.importorskip("paper_2201_02309_amd.network")

pytestmark = pytest.mark.gpu


def _conv(cin, cout, seed=0):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.manual_seed(seed)
    return N.Conv3x3x3(cin, cout).cuda()


# channels; batch, depth, height, width (tiles of 8 x 32, depth ranges of 4 and more)
@pytest.mark.parametrize("cin,cout", [(1, 16), (16, 16), (16, 1), (8, 8), (3, 5), (12, 9), (1, 1)])
@pytest.mark.parametrize("shape", [(1, 1, 1, 1), (2, 3, 7, 31), (1, 9, 8, 32), (1, 4, 17, 65), (2, 5, 9, 33)])
def test_matches_float64(cin, cout, shape):
    m = _conv(cin, cout)
    B, D, H, W = shape
    print(f"[case] {cin} -> {cout}, {shape}", flush=True)
    x = torch.randn(B, cin, D, H, W, device="cuda", requires_grad=True)
    assert N._native_conv(x, m.weight, m.bias)
    with torch.no_grad():
        y = m(x)
    g = torch.randn_like(y)
    got = torch.autograd.grad(m(x), (x, m.weight, m.bias), g)
    conv = torch.nn.functional.conv3d

    def ref(x, w, b, g):
        x, w, b = (t.detach().double().cpu().requires_grad_() for t in (x, w, b))
        y = conv(x, w, b, padding=1)
        return (y, *torch.autograd.grad(y, (x, w, b), g.double().cpu()))
    want = ref(x, m.weight, m.bias, g)
    size = ref(x.abs(), m.weight.abs(), m.bias.abs(), g.abs())     # sums of the terms' magnitudes
    terms = (27 * cin + 1, 27 * cout, B * D * H * W, B * D * H * W)
    for v, r, s, n in zip((y, *got), want, size, terms):
        # rounding of n products and sums in float32, and of the result
        bound = (n + 2) * 2.0 ** -24 * s.detach()
        assert bool(((v.detach().double().cpu() - r.detach()).abs() <= bound + 1e-30).all())


def test_layouts_and_repeats():
    m = _conv(16, 16)
    x = torch.randn(2, 16, 6, 20, 40, device="cuda")
    with torch.no_grad():
        ref = m(x)
    assert ref.stride() == N._conv3x3x3(x, m.weight, m.bias).stride()
    for v in (x.permute(0, 2, 1, 3, 4).contiguous().permute(0, 2, 1, 3, 4),
              x.transpose(3, 4).contiguous().transpose(3, 4),
              x.to(memory_format=torch.channels_last_3d), torch.cat([x, x], 2)[:, :, :6],
              torch.cat([x, x], 4)[..., :40]):
        with torch.no_grad():
            assert torch.equal(m(v), ref)
    xg = x.clone().requires_grad_()
    y = m(xg)
    a, b = (torch.autograd.grad(y, (xg, m.weight, m.bias), torch.ones(1, device="cuda").expand_as(y),
                                retain_graph=True) for _ in range(2))
    assert all(torch.equal(p, q) for p, q in zip(a, b))


def test_second_derivatives_transforms_autocast_and_in_place():
    m = _conv(3, 4)
    x = torch.randn(1, 3, 3, 5, 6, device="cuda", requires_grad=True)
    p = dict(m.named_parameters())

    def grads(f):
        gx, gw = torch.autograd.grad((f(x) ** 2).sum(), (x, m.weight), create_graph=True)
        return torch.autograd.grad((gx ** 2).sum() + (gw ** 3).sum(), (x, m.weight, m.bias))
    for a, b in zip(grads(m), grads(lambda v: N._conv3x3x3(v, m.weight, m.bias))):
        assert torch.allclose(a, b, rtol=1e-4, atol=1e-3 * float(b.abs().max()))
    # batched gradients, function transforms, forward mode
    y = m(x)
    eye = torch.randn(3, *y.shape, device="cuda")
    each = [torch.autograd.grad(y, x, e, retain_graph=True)[0] for e in eye]
    many = torch.autograd.grad(y, x, eye, retain_graph=True, is_grads_batched=True)[0]
    assert torch.allclose(many, torch.stack(each), atol=1e-5)
    xs = torch.randn(4, 1, 3, 3, 5, 6, device="cuda")
    out = torch.func.vmap(lambda v: torch.func.functional_call(m, p, (v,)))(xs)
    assert torch.allclose(out, torch.stack([m(v) for v in xs]), atol=1e-5)
    t = torch.randn_like(x)
    _, jvp = torch.func.jvp(lambda v: torch.func.functional_call(m, p, (v,)), (x.detach(),), (t,))
    assert torch.allclose(jvp, m(t) - m(torch.zeros_like(t)), atol=1e-5)
    with torch.autocast("cuda", dtype=torch.bfloat16):
        assert m(x).dtype == torch.bfloat16
    # the input and the weights may change before the backward
    z = x.detach().clone()
    y = m(z)
    want = torch.autograd.grad(y.sum(), m.weight, retain_graph=True)[0]
    z.mul_(2.0)
    with torch.no_grad():
        m.weight.mul_(0.5)
    assert torch.equal(torch.autograd.grad(y.sum(), m.weight)[0], want)


@pytest.mark.parametrize("shape", [(1, 1, 1, 1, 1), (2, 5, 3, 7, 31), (1, 16, 4, 64, 128), (1, 3, 2, 91, 91)])
def test_prelu_gradients(shape):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    C = shape[1]
    print(f"[case] PReLU {shape}", flush=True)
    torch.manual_seed(1)
    m = N.PReLU(C).cuda()
    with torch.no_grad():
        m.weight.copy_(torch.randn(C))
    x = torch.randn(shape, device="cuda")
    x.view(-1)[::5] = 0.0
    B, _, D, H, W = shape
    for v in (x, x.permute(0, 2, 1, 3, 4).contiguous().permute(0, 2, 1, 3, 4), x.transpose(3, 4).contiguous().transpose(3, 4)):
        v = v.detach().requires_grad_()
        y = m(v)
        assert type(y.grad_fn).__name__ == "_PReLUFnBackward"
        g = torch.randn_like(y)
        gx, gw = torch.autograd.grad(y, (v, m.weight), g, retain_graph=True)
        xd, wd = v.detach().double().requires_grad_(), m.weight.detach().double().requires_grad_()
        rx, rw = torch.autograd.grad(torch.nn.functional.prelu(xd, wd), (xd, wd), g.double())
        assert torch.equal(gx, rx.float())                       # one rounding each
        size = (v.detach() * g).double().abs().sum(dim=(0, 2, 3, 4))
        # summed in float64, rounded once
        assert bool(((gw.double() - rw).abs() <= 2.0 ** -24 * rw.abs() + 1e-12 * size + 1e-30).all())
        assert torch.equal(gw, torch.autograd.grad(y, m.weight, g)[0])
    # second derivatives go through torch
    v = x.detach().requires_grad_()
    gx = torch.autograd.grad((m(v) ** 2).sum(), v, create_graph=True)[0]
    assert torch.isfinite(torch.autograd.grad(gx.sum(), v)[0]).all()


# planes of whole vectors, of a remainder, one sample; unaligned; strided as the layers store them
@pytest.mark.parametrize("shape", [(2, 3, 1, 4, 4), (1, 16, 2, 8, 32), (2, 5, 7, 65, 31), (1, 1, 1, 1, 1),
                                   (3, 4, 5, 130, 66)])
@pytest.mark.parametrize("layout", ["dense", "depth first", "shifted"])
def test_depth_copies(shape, layout):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    B, C, D, H, W = shape
    if layout == "depth first":
        x = torch.randn(B, D, C, H, W, device="cuda").permute(0, 2, 1, 3, 4)
    else:
        off = 1 if layout == "shifted" else 0
        x = torch.randn(B * C * D * H * W + off, device="cuda")[off:].view(shape)
    x[0, 0, 0, 0, 0] = float("nan")
    xp = torch.nn.functional.pad(x, (0, 0, 0, 0, 1, 1))
    want = torch.stack([xp[:, :, k:k + D] for k in range(3)], 1).permute(0, 3, 1, 2, 4, 5).reshape(B * D, 3 * C, H, W)
    got = N._K.stack3(x)
    assert torch.equal(got.view(torch.int32), want.contiguous().view(torch.int32))


@pytest.mark.parametrize("cout,shape", [(1, (1, 10, 256, 256)), (16, (2, 9, 64, 96))])
def test_bias_gradient_that_cancels(cout, shape):
    """The sum of a cotangent of either sign is far smaller than its terms: float64 sums, whose
    errors are 2^-50 of the magnitudes, and one rounding to float32."""
    m = _conv(2, cout)
    B, D, H, W = shape
    for seed in range(4):
        torch.manual_seed(seed)
        x = torch.randn(B, 2, D, H, W, device="cuda")
        g = torch.randn(B, cout, D, H, W, device="cuda")
        g -= g.double().mean(dim=(0, 2, 3, 4), keepdim=True).float()
        got = torch.autograd.grad(m(x), m.bias, g)[0].double()
        want, size = g.double().sum(dim=(0, 2, 3, 4)), g.double().abs().sum(dim=(0, 2, 3, 4))
        assert bool(((got - want).abs() <= 2.0 ** -24 * want.abs() + 2.0 ** -50 * size).all()), (got - want)


def test_launch_limits():
    """Volumes whose launches would pass 2^32 threads along x stay with torch."""
    one = torch.empty(1)
    assert N._native_volume(one.expand(4, 16, 1 << 17, 1, 1), 16)
    assert not N._native_volume(one.expand(8, 16, 1 << 17, 1, 1), 16)
