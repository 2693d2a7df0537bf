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
