"""Values that are not finite in the network layers' gradients: each reaches the sums that contain
it and no other, as in torch's operators in float64."""
import pytest

torch = pytest.importorskip("torch")
N = pytest.importorskip("paper_2201_02309_amd.network")

pytestmark = pytest.mark.gpu

INF, NAN = float("inf"), float("nan")


def _same(got, want):
    """Equal NaNs and infinities; the finite ones to float32's rounding of small whole numbers."""
    got, want = got.detach().double().cpu(), want.detach().double().cpu()
    assert torch.equal(torch.isnan(got), torch.isnan(want)), (got, want)
    assert torch.equal(torch.nan_to_num(got), torch.nan_to_num(want)), (got, want)


# a vector of samples and a remainder; x, cotangent
@pytest.mark.parametrize("W", [4, 5])
@pytest.mark.parametrize("xv,gv", [(2.0, INF), (2.0, NAN), (INF, -INF), (-1.0, INF), (-INF, 1.0),
                                   (0.0, INF), (NAN, 1.0)])
def test_prelu(W, xv, gv):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    m = N.PReLU(2).cuda()
    x = torch.tensor([-3.0, 1.0, -2.0, 5.0, -1.0][:W]).repeat(2).view(1, 2, 1, 1, W)
    g = torch.ones(1, 2, 1, 1, W)
    x[0, 0, 0, 0, 1], g[0, 0, 0, 0, 1] = xv, gv
    v = x.cuda().requires_grad_()
    y = m(v)
    assert type(y.grad_fn).__name__ == "_PReLUFnBackward"
    got = torch.autograd.grad(y, (v, m.weight), g.cuda())
    xd, wd = x.double().requires_grad_(), m.weight.detach().cpu().double().requires_grad_()
    for a, b in zip(got, torch.autograd.grad(torch.nn.functional.prelu(xd, wd), (xd, wd), g.double())):
        _same(a, b)


# tiles of 8 x 32: whole ones, one row and one column past them, less than one
@pytest.mark.parametrize("H,W", [(8, 32), (9, 33), (7, 31), (17, 64), (16, 65), (3, 5)])
@pytest.mark.parametrize("bad", [INF, NAN])
def test_weight_gradient_at_the_edges(H, W, bad):
    """A sample that is not finite in the last row or column: the taps that meet it with a sample of
    the cotangent, and no others."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    m = N.Conv3x3x3(2, 3).cuda()
    for at in ((H - 1, 0), (0, W - 1), (H - 1, W - 1)):
        x, g = torch.ones(1, 2, 3, H, W), torch.ones(1, 3, 3, H, W)
        x[0, 1, 1, at[0], at[1]] = bad
        v = x.cuda().requires_grad_()
        y = m(v)
        assert type(y.grad_fn).__name__ == "_Conv3FnBackward"
        got = torch.autograd.grad(y, m.weight, g.cuda())[0]
        # one tap at a time: the products of the samples that both lie in the volume
        want = torch.zeros(3, 2, 3, 3, 3, dtype=torch.float64)
        for d in range(3):
            for h in range(3):
                for w in range(3):
                    here, there = [], []
                    for t, n in ((d, 3), (h, H), (w, W)):
                        here.append(slice(max(0, 1 - t), n - max(0, t - 1)))
                        there.append(slice(max(0, t - 1), n - max(0, 1 - t)))
                    xs, gs = x.double()[0][(slice(None), *there)], g.double()[0][(slice(None), *here)]
                    want[:, :, d, h, w] = (gs[:, None] * xs[None]).sum(dim=(2, 3, 4))
        print(f"[case] {H} x {W}, {bad} at {at}: {int((~torch.isfinite(want)).sum())} of 162", flush=True)
        _same(got, want)


# cotangents whose sums are infinite, not numbers, and pass float32's range on the way to one in it
@pytest.mark.parametrize("values", [(INF,), (-INF, 5.0), (INF, -INF), (NAN,), (3.0e38, 3.0e38, -3.0e38),
                                    (3.0e38, 3.0e38)])
def test_bias_gradient(values):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    m = N.Conv3x3x3(2, 3).cuda()
    x = torch.ones(1, 2, 3, 9, 33, device="cuda")
    g = torch.zeros(1, 3, 3, 9, 33)
    for i, v in enumerate(values):
        g[0, 1, 1, 4, 3 + 7 * i] = v
    got = torch.autograd.grad(m(x), m.bias, g.cuda())[0]
    _same(got, g.double().sum(dim=(0, 2, 3, 4)).float())
