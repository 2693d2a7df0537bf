"""Dual-domain network of Sec. III: sinogram-domain subnetwork -> Katsevich reconstruction
as the domain-transfer layer -> image-domain subnetwork, trained on the loss of eq. loss
with Adam.

The domain-transfer layer is the library's differentiable reconstruction (KatsevichFn:
katsevich_recon forward, its exact adjoint katsevich_recon_backward backward) on a plan of
one pitch: the sinogram window that reconstructs that pitch's slices goes in, the slices
come out.  The gradients of the subnetworks' 3x3x3 convolutions and PReLUs, and the convolutions
of inference, run on the library's kernels (katsevich_conv3, katsevich_conv3_grad,
katsevich_prelu_grad: float32 matrix cores); a training step's forward, other types, devices,
channel counts and tracing or transforming callers take one PyTorch 2-D convolution over the three
depth-shifted copies of the input stacked as channels, with depth folded into the batch.
"""
from __future__ import annotations

import math

import torch
import torch.nn.functional as F
from torch import nn
from torch.overrides import _get_current_function_mode_stack
from torch.utils._device import DeviceContext

from . import katsevich as _K
from .katsevich import KatsevichFn, Plan


def _conv3x3x3(x, weight, bias):
    """The convolution as a 2-D convolution: output depth d sees input depths d-1, d, d+1 stacked
    as 3 cin channels.  Any type and device, every order of derivative."""
    B, C, D, H, W = x.shape
    xp = F.pad(x, (0, 0, 0, 0, 1, 1))
    stack = torch.cat([xp[:, :, k:k + D] for k in range(3)], dim=1)      # [B, 3C, D, H, W]
    stack = stack.permute(0, 2, 1, 3, 4).reshape(B * D, 3 * C, H, W)
    return _conv_stack(stack, B, D, weight, bias)


def _conv_stack(stack, B: int, D: int, weight, bias):
    """The 2-D convolution of [B D, 3 C, H, W] depth-shifted copies -> [B, cout, D, H, W]."""
    _, C3, H, W = stack.shape
    cout = weight.shape[0]
    w2 = weight.permute(0, 2, 1, 3, 4).reshape(cout, C3, 3, 3)
    y = F.conv2d(stack, w2, bias, padding=1)
    return y.reshape(B, D, cout, H, W).permute(0, 2, 1, 3, 4)


def _plain(*tensors):
    """Whether every tensor is a plain float32 one of the same GPU, and no autocast, tracing,
    compilation, forward-mode derivative, function transform, function or dispatch mode (other than
    a default device) is at work, which need torch's operators."""
    if torch.compiler.is_compiling():          # first: a compiler follows what comes after it
        return False
    for t in tensors:
        if type(t) not in (torch.Tensor, nn.Parameter) or t.dtype != torch.float32 or not t.is_cuda \
                or t.device != tensors[0].device or not torch._C._has_storage(t):
            return False
    return not (torch.is_autocast_enabled("cuda") or torch._C._is_tracing()
                or torch.autograd.forward_ad._current_level >= 0
                or torch._C._functorch.peek_interpreter_stack() is not None
                or torch._C._len_torch_dispatch_stack() > 0
                or torch._C._len_torch_function_stack() > 0 and any(
                    not isinstance(m, DeviceContext) for m in _get_current_function_mode_stack()))


def _native_volume(x, channels):
    """Whether x is a [B, channels, D, H, W] volume within the kernels' grids and 32-bit offsets."""
    if x.dim() != 5 or x.numel() == 0 or x.shape[1] != channels:
        return False
    B, C, D, H, W = x.shape
    return (B <= 65535 and D <= 4 * 65535 and (16 * D + 1) * H * W <= 1 << 30
            and B * D * C * ((H * W + 8191) // 8192) < 1 << 24       # workgroups of 256 along x
            and B * ((H + 7) // 8) * ((W + 31) // 32) < 1 << 31)


def _native_conv(x, weight, bias):
    """Whether the library's kernels take this convolution (at most 16 channels on either side)."""
    if not _plain(x, weight, bias) or x.dim() != 5:     # (a symbolic x has no dim() to compare)
        return False
    cin, cout = x.shape[1], weight.shape[0]
    return (1 <= cout <= 16 and cin <= 16 and weight.shape == (cout, cin, 3, 3, 3)
            and bias.shape == (cout,) and _native_volume(x, cin))


def _check_kept(gy, *kept):
    """Hooks on saved tensors may hand back others than were kept, which torch's operators refuse and
    the kernels would read out of range: every (tensor, shape) must have that shape and gy's type and
    device."""
    dtype, device = gy.dtype, gy.device
    for t, shape in kept:
        if t.shape != shape or t.dtype != dtype or t.device != device:
            raise RuntimeError(f"a saved tensor came back as {t.dtype} {tuple(t.shape)} on {t.device}: "
                               f"{gy.dtype} {tuple(shape)} on {gy.device} was kept")


class _Conv3Fn(torch.autograd.Function):
    """_conv3x3x3 with its gradients on the library's kernels; a derivative that is itself to be
    differentiated, or whose gradient the kernels do not take, goes through _conv3x3x3 again.  x and
    weight are kept as they are: the caller hands over tensors that nothing changes before the
    backward.  The forward of a training step stays torch's: PReLU's derivative jumps at 0, so
    another rounding of the activations would move a whole network's gradients by 1e-3."""

    @staticmethod
    def forward(ctx, x, weight, bias):
        # (x plays a part in the weight's gradient alone: a frozen layer's may change)
        ctx.save_for_backward(x if ctx.needs_input_grad[1] else None, weight)
        ctx.shape = x.shape
        stack = _K.stack3(x)
        return _conv_stack(stack, x.shape[0], x.shape[2], weight, bias)

    @staticmethod
    def backward(ctx, gy):
        x, weight = ctx.saved_tensors
        if x is None:
            x = weight.new_zeros(1, 1, 1, *ctx.shape[3:]).expand(ctx.shape)
        want = ctx.needs_input_grad
        again = torch.is_grad_enabled()
        _check_kept(gy, (x, ctx.shape), (weight, (gy.shape[1], ctx.shape[1], 3, 3, 3)))
        if again or not _plain(gy, x, weight) or not _native_volume(gy, gy.shape[1]):
            with torch.enable_grad():
                bias = weight.new_zeros(weight.shape[0], requires_grad=True)   # its value plays no part
                args = [t if t.requires_grad else t.detach().requires_grad_(n)
                        for t, n in zip((x, weight, bias), want)]
                grads = iter(torch.autograd.grad(_conv3x3x3(*args), [t for t, n in zip(args, want) if n],
                                                 gy, create_graph=again))
            return tuple(next(grads) if n else None for n in want)
        gy = _K.dense_volume(gy)
        gx = _K.conv3(gy, weight, transposed=True) if want[0] else None
        gw = gb = None
        if want[1] or want[2]:
            gw, gb = _K.conv3_grad(x, gy, tuple(weight.shape))
        return gx, gw if want[1] else None, gb if want[2] else None


class Conv3x3x3(nn.Module):
    """3-D convolution with a 3x3x3 kernel and zero padding 1 (as nn.Conv3d(cin, cout, 3,
    padding=1)).  Its input and parameters may be changed in place before the backward: it keeps
    copies of them (of the input only while `copy_input` holds; a network whose forward leaves a
    convolution's input alone clears it there)."""

    copy_input = True

    def __init__(self, cin: int, cout: int):
        super().__init__()
        ref = nn.Conv3d(cin, cout, 3, padding=1)           # same initialisation as Conv3d
        self.weight = nn.Parameter(ref.weight.detach().clone())
        self.bias = nn.Parameter(ref.bias.detach().clone())

    def forward(self, x):                                   # x [B, C, D, H, W]
        if torch.jit.is_scripting():                        # (a script compiles this branch alone)
            return _conv3x3x3(x, self.weight, self.bias)
        else:
            return self._eager(x)

    def _eager(self, x):
        w, b = self.weight, self.bias
        if not _native_conv(x, w, b):
            return _conv3x3x3(x, w, b)
        if torch.is_grad_enabled() and (x.requires_grad or w.requires_grad or b.requires_grad):
            return _Conv3Fn.apply(x.clone() if self.copy_input and w.requires_grad else x, w.clone(), b)
        return _K.conv3(x, w, b)


class _PReLUFn(torch.autograd.Function):
    """PReLU with one slope per channel, its gradients on the library's kernel; a derivative that is
    itself to be differentiated, or whose gradient the kernel does not take, goes through torch."""

    @staticmethod
    def forward(ctx, x, weight):
        ctx.save_for_backward(x, weight)
        return F.prelu(x, weight)

    @staticmethod
    def backward(ctx, gy):
        x, weight = ctx.saved_tensors
        want = ctx.needs_input_grad
        again = torch.is_grad_enabled()
        _check_kept(gy, (x, gy.shape), (weight, gy.shape[1:2]))
        if again or not _plain(gy, x, weight):
            with torch.enable_grad():
                args = [t if t.requires_grad else t.detach().requires_grad_(n) for t, n in zip((x, weight), want)]
                grads = iter(torch.autograd.grad(F.prelu(*args), [t for t, n in zip(args, want) if n], gy,
                                                 create_graph=again))
            return tuple(next(grads) if n else None for n in want)
        gx, gw = _K.prelu_grad(x, gy, weight)
        return gx if want[0] else None, gw if want[1] else None


class PReLU(nn.PReLU):
    """nn.PReLU whose gradients on float32 volumes of one GPU run on the library's kernel."""

    def forward(self, x):
        if torch.jit.is_scripting():                        # (as in Conv3x3x3)
            return F.prelu(x, self.weight)
        else:
            return self._eager(x)

    def _eager(self, x):
        w = self.weight
        if torch.is_grad_enabled() and _plain(x, w) and (x.requires_grad or w.requires_grad) \
                and _native_volume(x, w.numel()):
            return _PReLUFn.apply(x, w)
        return F.prelu(x, w)


class SubNet(nn.Module):
    """Subnetwork of Sec. III-A: `blocks` cascaded Conv3D(channels, 3x3x3) + PReLU blocks
    and one Conv3D(1, 3x3x3).  The output of every Conv3D+PReLU block is added to the last
    block's output before the final convolution, and the subnetwork's input is added to
    the final convolution's output (ResNet-style skips)."""

    def __init__(self, channels: int = 16, blocks: int = 7):
        super().__init__()
        self.convs = nn.ModuleList([Conv3x3x3(1 if i == 0 else channels, channels)
                                    for i in range(blocks)])
        self.acts = nn.ModuleList([PReLU(channels) for _ in range(blocks)])
        self.out = Conv3x3x3(channels, 1)
        for conv in (*self.convs[1:], self.out):
            conv.copy_input = False        # forward() makes these inputs and does not change them

    def forward(self, x):                          # x [B, 1, D, H, W]
        h = x
        outs = []
        for conv, act in zip(self.convs, self.acts):
            h = act(conv(h))
            outs.append(h)
        s = outs[-1]
        for o in outs[:-1]:
            s = s + o
        return x + self.out(s)


class DualDomainNet(nn.Module):
    """g (the window sinogram of one pitch, [B, views, rows, cols]) -> (denoised sinogram,
    denoised slices [B, nz, ny, nx])."""

    def __init__(self, plan: Plan, channels: int = 16, blocks: int = 7):
        super().__init__()
        self.plan = plan
        self.sino_net = SubNet(channels, blocks)
        self.image_net = SubNet(channels, blocks)

    def forward(self, g):
        gs = self.sino_net(g.unsqueeze(1)).squeeze(1)
        f0 = KatsevichFn.apply(gs.contiguous(), self.plan)
        f = self.image_net(f0.unsqueeze(1)).squeeze(1)
        return gs, f


def loss(g, f, g_gt, f_gt):
    """Eq. loss: squared L2 errors of the sinogram and of the image, averaged over the
    batch."""
    return ((g_gt - g) ** 2).sum(dim=(1, 2, 3)).mean() + ((f_gt - f) ** 2).sum(dim=(1, 2, 3)).mean()


def pitch_window_geometry(geom: dict, grid: dict):
    """(geometry of the views a pitch's slices use, index of its first view in geom): the
    scan restricted to the views the plan filters plus the derivative's neighbour on each
    side, at the same lambdas."""
    p = Plan(geom, grid, bind=False)
    a, b = int(p.info["first_view"]) - 1, int(p.info["last_view"]) + 1
    p.close()
    w = dict(geom)
    w["lambda_first"] = float(geom.get("lambda_first", 0.0)) + a * 2.0 * math.pi / int(
        geom["views_per_turn"])
    w["n_views"] = b - a + 1
    return w, a
