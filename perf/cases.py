"""Workloads whose speed matters to users of this framework, each one pass through its public
entry points, with the arithmetic of the same pass in float64.

Kinds of case:
  recon    sinogram -> volume on a kept plan (katsevich_recon)
  adjoint  volume cotangent -> sinogram cotangent on a kept plan (katsevich_recon_backward)
  train    the reconstruction as a network layer: KatsevichFn forward and backward
  cold     a new scan geometry: plan built on the GPU, then the reconstruction
  group    several requests on kept plans: filter each, one grouped backprojection
  data     sparse-detector data preparation: upsampling, maximum, noise
  metrics  RMSE and SSIM of a volume against a reference
  subnet   a subnetwork of the dual-domain network, training (gradients) or inference

Scans: R = 570 mm, D = 1040 mm, a detector whose fan covers the grid's corners and whose rows
cover the Tam-Danielsson window + 10 %, slices that repeat every pitch; the network scan is one
pitch window of the p = 7 pi workload.  Sinograms are line integrals of seeded ellipsoids.
"""
import math
import random

import torch

import paper_2201_02309_amd as K
from paper_2201_02309_amd import network as N

PI = math.pi


# ------------------------------------------------------------------------------- the cases
def _scan(kind, name=None, **kw):
    case = {"kind": kind, "nxy": 64, "nz": 64, "dxy": 1.0, "cols": 128, "rows": 16, "vpt": 360,
            "turns": 3, "feed": 24.0, "spp": 24, "batch": 1, "half": False, "det": False}
    case.update(kw)
    return case if name is None else dict(case, name=name)


CLINICAL = dict(nxy=512, nz=128, dxy=0.7, cols=736, rows=64, vpt=1160, turns=6, feed=76.8, spp=77)
SPARSE = dict(nxy=256, nz=64, dxy=1.4, cols=184, rows=64, vpt=1160, turns=6, feed=96.0, spp=48)


def listed():
    return [
        # a small volume of a short scan: launches and the length of the view loop count
        _scan("recon", "recon-64"),
        # the clinical high-pitch scan, whole volume: the framework's headline workload
        _scan("recon", "recon-clinical", **CLINICAL),
        # half-sample derivative on sizes that are multiples of nothing
        _scan("recon", "recon-half-ragged", nxy=301, nz=77, dxy=1.15, cols=511, rows=45, vpt=1000,
              turns=4, feed=61.0, spp=53, half=True),
        # the exact adjoint of the clinical reconstruction (iterative methods, training)
        _scan("adjoint", "adjoint-clinical", **CLINICAL),
        # training through the layer on the 4x sparse detector, a batch of two scans
        _scan("train", "train-sparse", batch=2, **SPARSE),
        # the layer of the dual-domain network: one pitch of 10 slices, 16-row window sinogram
        {"kind": "train", "name": "train-network-pitch", "net": True, "nxy": 512, "nz": 10,
         "batch": 1},
        # bit-reproducible gradients of a thin slab
        _scan("adjoint", "adjoint-reproducible", nxy=256, nz=32, dxy=1.4, cols=736, rows=64,
              vpt=1160, turns=3, feed=60.0, spp=60, det=True),
        # serving: a request with a geometry not seen before
        _scan("cold", "cold-request", nxy=256, nz=96, dxy=1.4, cols=736, rows=64, vpt=1160,
              turns=5, feed=64.0, spp=64),
        # serving: four requests of different sizes closed into one group
        {"kind": "group", "name": "serving-group", "requests": 4, "pick": 20},
        # data preparation of a sparse-detector training set (every 4th column kept)
        {"kind": "data", "name": "sparse-data", "views": 2320, "rows": 64, "cols": 736, "step": 4},
        # image quality of one clinical volume
        {"kind": "metrics", "name": "metrics-volume", "nz": 128, "ny": 512, "nx": 512},
        # a training step's forward and backward of the image subnetwork on one pitch's slices
        {"kind": "subnet", "name": "subnet-image-train", "depth": 10, "height": 512, "width": 512,
         "channels": 16, "blocks": 7, "train": True},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_scan(rng, kind, max_nxy=512, max_nz=128):
    nxy = _log_int(rng, 32, max_nxy)
    nz = _log_int(rng, 4, max_nz)
    feed = round(rng.uniform(24.0, 96.0), 3)
    spp = max(2, int(round(feed / rng.uniform(0.9, 2.2))))
    turns = int(math.ceil(nz / spp)) + rng.choice((2, 3))
    vpt = _log_int(rng, 360, 1160)
    return _scan(kind, nxy=nxy, nz=nz, dxy=round(rng.uniform(60.0, 358.0) / nxy, 4),
                 cols=_log_int(rng, 64, 736), rows=_log_int(rng, 16, 64), vpt=vpt, turns=turns,
                 feed=feed, spp=spp)


def draw(rng):
    kind = rng.choice(("recon", "recon", "adjoint", "train", "cold", "group", "data", "metrics",
                       "subnet"))
    if kind == "recon":
        return dict(_draw_scan(rng, kind), half=rng.random() < 0.3)
    if kind == "adjoint":
        return dict(_draw_scan(rng, kind, 320, 64), det=rng.random() < 0.3)
    if kind == "train":
        if rng.random() < 0.4:
            return {"kind": "train", "net": True, "nxy": _log_int(rng, 64, 512),
                    "nz": rng.randint(5, 10), "batch": rng.randint(1, 2)}
        return dict(_draw_scan(rng, kind, 256, 64), batch=rng.randint(1, 2))
    if kind == "cold":
        return _draw_scan(rng, kind, 384, 96)
    if kind == "group":
        return {"kind": "group", "requests": rng.randint(2, 5), "pick": rng.randint(0, 9999)}
    if kind == "data":
        return {"kind": "data", "views": _log_int(rng, 90, 2320), "rows": _log_int(rng, 8, 64),
                "cols": _log_int(rng, 64, 736), "step": rng.choice((2, 3, 4, 4, 5))}
    if kind == "metrics":
        return {"kind": "metrics", "nz": _log_int(rng, 4, 128), "ny": _log_int(rng, 33, 512),
                "nx": _log_int(rng, 33, 512)}
    return {"kind": "subnet", "depth": _log_int(rng, 4, 40), "height": _log_int(rng, 16, 192),
            "width": _log_int(rng, 48, 256), "channels": rng.choice((8, 16, 16)),
            "blocks": rng.randint(2, 7), "train": rng.random() < 0.5}


def _group(case):
    """Plain scans of the group's requests."""
    r = random.Random(case["pick"])
    out = []
    for _ in range(case["requests"]):
        nxy, nz, dxy = r.choice(((256, 32, 1.4), (256, 96, 1.4), (512, 64, 0.7)))
        feed = r.uniform(40.0, 96.0)
        spp = int(round(feed))
        out.append(_scan("recon", nxy=nxy, nz=nz, dxy=dxy, cols=r.choice((736, 184)), rows=64,
                         vpt=1160, turns=int(math.ceil(nz / spp)) + 2, feed=feed, spp=spp))
    return out


# --------------------------------------------------------------------- geometry and inputs
def _geometry(case):
    """(geometry, grid) dicts of a scan, as the framework takes them."""
    if case.get("net"):
        R, D, feed, vpt, cols, rows = 595.0, 1085.6, 7.0 * PI, 360, 627, 16
        dalpha, col_offset, turns, dxy = PI / 2880.0, 0.25, 4, 512.0 / case["nxy"]
        alpha_m, dz = (0.5 * (cols - 1) + col_offset) * dalpha, feed / case["nz"]
    else:
        R, D, feed, vpt, cols, rows = (570.0, 1040.0, case["feed"], case["vpt"], case["cols"],
                                       case["rows"])
        col_offset, turns, dxy, dz = 0.0, case["turns"], case["dxy"], feed / case["spp"]
        alpha_m = math.asin((math.hypot(0.5, 0.5) * (case["nxy"] - 1) * dxy + 0.05) / R)
        dalpha = 2.0 * alpha_m / (cols - 1)
    w_td = D * feed / (2.0 * PI * R) * (0.5 * PI + alpha_m) / math.cos(alpha_m)
    n_views = vpt * turns
    geom = dict(R=R, D=D, feed_per_turn=feed, views_per_turn=vpt, n_views=n_views, det_cols=cols,
                det_rows=rows, dalpha=dalpha, dw=2.2 * w_td / (rows - 1), lambda0=0.0, z0=0.0,
                lambda_first=0.0, col_offset=col_offset, row_offset=0.0)
    nxy, nz = case["nxy"], case["nz"]
    zmid = 0.5 * feed * (n_views - 1) / vpt
    grid = dict(nx=nxy, ny=nxy, nz=nz, dx=dxy, dy=dxy, dz=dz, x_first=-0.5 * (nxy - 1) * dxy,
                y_first=-0.5 * (nxy - 1) * dxy, z_first=zmid - 0.5 * (nz - 1) * dz)
    if case.get("net"):          # only the views that the pitch's slices use
        geom, _ = N.pitch_window_geometry(geom, grid)
    return geom, grid


def _sinogram(geom, grid, seed):
    """float32 [n_views, rows, cols]: closed-form line integrals of eight ellipsoids."""
    r = random.Random(seed)
    half = 0.5 * min(grid["nx"] * grid["dx"],
                     1.4 * geom["R"] * math.sin(0.5 * (geom["det_cols"] - 1) * geom["dalpha"]))
    zlo, zhi = grid["z_first"], grid["z_first"] + (grid["nz"] - 1) * grid["dz"]
    body = [(0.0, 0.0, 0.5 * (zlo + zhi), 0.85 * half, 0.7 * half, 0.6 * (zhi - zlo) + 0.8 * half, 1.0)]
    for _ in range(7):
        phi, rho = r.uniform(0, 2 * PI), 0.5 * half * math.sqrt(r.random())
        body.append((rho * math.cos(phi), rho * math.sin(phi), r.uniform(zlo, zhi),
                     *(half * r.uniform(0.06, 0.35) for _ in range(3)), r.uniform(-0.3, 0.6)))
    V, rows, cols = geom["n_views"], geom["det_rows"], geom["det_cols"]
    out = torch.empty(V, rows, cols, device="cuda")
    al = ((torch.arange(cols, device="cuda") - 0.5 * (cols - 1) + geom["col_offset"]) * geom["dalpha"])[None, None, :]
    w = ((torch.arange(rows, device="cuda") - 0.5 * (rows - 1) + geom["row_offset"]) * geom["dw"])[None, :, None]
    inv = 1.0 / torch.sqrt(geom["D"] ** 2 + w * w)
    dlam, h = 2.0 * PI / geom["views_per_turn"], geom["feed_per_turn"] / (2.0 * PI)
    for a in range(0, V, 128):
        lam = (geom["lambda_first"] + torch.arange(a, min(V, a + 128), device="cuda", dtype=torch.float64) * dlam)
        beta = torch.remainder(lam + geom["lambda0"], 2.0 * PI).float()[:, None, None]
        dirx, diry = -torch.cos(beta + al) * geom["D"] * inv, -torch.sin(beta + al) * geom["D"] * inv
        dirz = w * inv
        acc = 0.0
        for x, y, z, ax, ay, az, rho in body:
            sx, sy = (geom["R"] * torch.cos(beta) - x) / ax, (geom["R"] * torch.sin(beta) - y) / ay
            sz = ((geom["z0"] + h * lam - z) / az).float()[:, None, None]
            ex, ey, ez = dirx / ax, diry / ay, dirz / az
            q2 = ex * ex + ey * ey + ez * ez
            cx, cy, cz = sy * ez - sz * ey, sz * ex - sx * ez, sx * ey - sy * ex   # s x e
            acc = acc + (2.0 * rho) * torch.sqrt(torch.clamp(q2 - (cx * cx + cy * cy + cz * cz), min=0.0)) / q2
        out[a:a + 128] = acc
    return out


def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _cotangent(grid, seed, batch=None):
    shape = (grid["nz"], grid["ny"], grid["nx"])
    return torch.randn(shape if batch is None else (batch,) + shape, device="cuda",
                       generator=_generator(seed + 17))


def _scan_input(case, seed):
    geom, grid = _geometry(case)
    sino = [_sinogram(geom, grid, seed * 131 + b) for b in range(case["batch"])]
    return torch.stack(sino) if case["kind"] == "train" else sino[0]


def _weights(case, seed):
    """The subnetwork's parameters in the order of its parameters(): every convolution's weight
    and bias, every PReLU's slopes, the last convolution's weight and bias."""
    g = torch.Generator().manual_seed(seed + 5)
    C, blocks = case["channels"], case["blocks"]

    def conv(cin, cout):
        b = 1.0 / math.sqrt(27 * cin)
        return [(torch.rand(cout, cin, 3, 3, 3, generator=g) * 2 - 1) * b,
                (torch.rand(cout, generator=g) * 2 - 1) * b]
    convs = [conv(1 if i == 0 else C, C) for i in range(blocks)]
    acts = [torch.full((C,), 0.25) + 0.02 * torch.randn(C, generator=g) for _ in range(blocks)]
    return convs, acts, conv(C, 1)


def _image(case, seed):
    """[1, 1, depth, height, width]: smooth structure and noise, as a reconstruction has."""
    shape = (1, 1, case["depth"], case["height"], case["width"])
    z, y, x = (torch.linspace(-1, 1, n, device="cuda") for n in shape[2:])
    g = _generator(seed)
    img = torch.zeros(shape, device="cuda")
    for _ in range(6):
        p = torch.rand(5, generator=g, device="cuda").tolist()
        img += (p[4] - 0.3) * torch.sigmoid(40.0 * (0.05 + 0.4 * p[0] - (
            (z[:, None, None] * 0.3) ** 2 + (y[:, None] - 1.4 * p[1] + 0.7) ** 2 + (x - 1.4 * p[2] + 0.7) ** 2)))
    return img + 0.02 * torch.randn(shape, generator=g, device="cuda")


def _volumes(case, seed):
    g = _generator(seed)
    ref = torch.rand(case["nz"], case["ny"], case["nx"], device="cuda", generator=g)
    return ref + 0.05 * torch.randn(ref.shape, device="cuda", generator=g), ref


def _sparse_data(case, seed):
    """A sinogram of the kept columns, the framework's sparse-detector input."""
    scan = _scan("recon", nxy=256, nz=64, dxy=1.4, cols=case["cols"], rows=case["rows"], vpt=1160,
                 feed=96.0, spp=48, turns=1)
    geom, grid = _geometry(scan)
    geom["n_views"] = case["views"]
    return _sinogram(geom, grid, seed)[..., ::case["step"]].contiguous()


# ------------------------------------------------------------------------------- one pass
def prepare(case, seed):
    kind = case["kind"]
    if kind in ("recon", "adjoint", "train", "cold"):
        geom, grid = _geometry(case)
        s = {"kind": kind, "geom": geom, "grid": grid}
        if kind != "cold":
            s["plan"] = K.Plan(geom, grid, gpu_plan=True, half_sample=case.get("half", False),
                               deterministic_adjoint=case.get("det", False))
        if kind == "adjoint":
            s["grad"] = _cotangent(grid, seed)
            s["out"] = torch.empty(geom["n_views"], geom["det_rows"], geom["det_cols"], device="cuda")
            return s
        s["sino"] = _scan_input(case, seed)
        if kind == "train":
            s["sino"].requires_grad_(True)
            s["grad"] = _cotangent(grid, seed, case["batch"])
        else:
            s["out"] = torch.empty(grid["nz"], grid["ny"], grid["nx"], device="cuda")
        return s
    if kind == "group":
        s = {"kind": kind, "plans": [], "sinos": [], "gF": [], "vols": []}
        for i, c in enumerate(_group(case)):
            geom, grid = _geometry(c)
            p = K.Plan(geom, grid, gpu_plan=True)
            s["plans"].append(p)
            s["sinos"].append(_sinogram(geom, grid, seed * 131 + i))
            s["gF"].append(torch.empty(K.filtered_shape(p), device="cuda"))
            s["vols"].append(torch.empty(grid["nz"], grid["ny"], grid["nx"], device="cuda"))
        return s
    if kind == "data":
        return {"kind": kind, "sparse": _sparse_data(case, seed), "cols": case["cols"],
                "step": case["step"], "seed": seed}
    if kind == "metrics":
        f, ref = _volumes(case, seed)
        return {"kind": kind, "f": f, "ref": ref}
    net = N.SubNet(case["channels"], case["blocks"])
    convs, acts, last = _weights(case, seed)
    with torch.no_grad():
        for m, (w, b) in zip(list(net.convs) + [net.out], convs + [last]):
            m.weight.copy_(w)
            m.bias.copy_(b)
        for m, a in zip(net.acts, acts):
            m.weight.copy_(a)
    x = _image(case, seed)
    s = {"kind": kind, "net": net.cuda(), "x": x, "train": case["train"]}
    if case["train"]:
        x.requires_grad_(True)
        s["grad"] = torch.randn(x.shape, device="cuda", generator=_generator(seed + 3))
    return s


def run(s):
    kind = s["kind"]
    if kind == "recon":
        return K.recon(s["plan"], s["sino"], out=s["out"])
    if kind == "adjoint":
        return K.recon_backward(s["plan"], s["grad"], out=s["out"])
    if kind == "train":
        s["sino"].grad = None
        vol = K.KatsevichFn.apply(s["sino"], s["plan"])
        vol.backward(s["grad"])
        return vol.detach(), s["sino"].grad
    if kind == "cold":
        plan = K.Plan(s["geom"], s["grid"], gpu_plan=True)
        return K.recon(plan, s["sino"], out=s["out"])
    if kind == "group":
        for p, g, f in zip(s["plans"], s["sinos"], s["gF"]):
            K.filter_views(p, g, out=f)
        return K.backproject_batch(s["plans"], s["gF"], s["vols"])
    if kind == "data":
        full = K.sparse_upsample(s["sparse"], s["cols"], s["step"])
        return full, K.add_noise(full, 1e5, 0.5, s["seed"], d_max=K.max_value(full))
    if kind == "metrics":
        return K.rmse_ssim(s["f"], s["ref"])
    if not s["train"]:
        with torch.no_grad():
            return s["net"](s["x"])
    s["x"].grad = None
    s["net"].zero_grad(set_to_none=True)
    y = s["net"](s["x"])
    y.backward(s["grad"])
    return y.detach(), s["x"].grad, [p.grad for p in s["net"].parameters()]


# ------------------------------------------------------- what one pass cannot do without
def work(case):
    kind = case["kind"]
    if kind == "group":
        parts = [work(c) for c in _group(case)]
        return {k: sum(p[k] for p in parts) for k in ("bytes", "flops")}
    if kind in ("recon", "adjoint", "train", "cold"):
        if case.get("net"):
            vpt, rows, cols, fov = 360, 16, 627, 0.5
            views = 586
        else:
            vpt, rows, cols, fov = case["vpt"], case["rows"], case["cols"], 1.0
            views = min(vpt * case["turns"], int(vpt * (case["nz"] / case["spp"] + 0.8)))
        vox = case["nxy"] ** 2 * case["nz"]
        n = (2 if kind == "train" else 1) * case["batch"]
        # 20 operations for each (voxel, view) pair: about 0.55 turns of views per voxel
        return {"bytes": 4.0 * n * (views * rows * cols + vox), "flops": 20.0 * n * 0.55 * vpt * vox * fov}
    if kind == "data":
        n = case["views"] * case["rows"]
        full = n * case["cols"]
        return {"bytes": 4.0 * (full / case["step"] + 2 * full), "flops": 60.0 * full}
    if kind == "metrics":
        n = case["nz"] * case["ny"] * case["nx"]
        return {"bytes": 8.0 * n, "flops": 16.0 * n}
    n = case["depth"] * case["height"] * case["width"]
    C = case["channels"]
    flops = 2.0 * 27 * n * (2 * C + C * C * (case["blocks"] - 1))
    return {"bytes": 4.0 * n * (4 if case["train"] else 2), "flops": flops * (3 if case["train"] else 1)}


# ------------------------------------------------------------------- the same in float64
class _Scan64:
    """The discretised reconstruction in float64: filter as dense matrices per detector column,
    backprojection view by view over the whole grid."""

    def __init__(self, geom, grid, half=False, device="cuda"):
        self.dev, self.half, self.grid = device, half, grid
        g = dict(geom)
        self.dlam = 2.0 * PI / g["views_per_turn"]
        if half:                         # views and columns between those of the sinogram
            g.update(lambda_first=g["lambda_first"] + 0.5 * self.dlam, n_views=g["n_views"] - 1,
                     det_cols=g["det_cols"] - 1)
        self.g = g
        self.h = g["feed_per_turn"] / (2.0 * PI)
        cols, rows = g["det_cols"], g["det_rows"]
        f64 = dict(dtype=torch.float64, device=device)
        al = (torch.arange(cols, **f64) - 0.5 * (cols - 1) + g["col_offset"]) * g["dalpha"]
        w = (torch.arange(rows, **f64) - 0.5 * (rows - 1) + g["row_offset"]) * g["dw"]
        self.lw = g["D"] / torch.sqrt(g["D"] ** 2 + w * w)
        self.cos = torch.cos(al)
        a_m = float(al.abs().max())
        self.r_fov = g["R"] * math.sin(min(-float(al[0]), float(al[-1])))
        n_psi, psi_max = 2 * rows + 1, 0.5 * PI + a_m
        dpsi = 2.0 * psi_max / (n_psi - 1)
        psi = (torch.arange(n_psi, **f64) - 0.5 * (n_psi - 1)) * dpsi
        ks = g["D"] * self.h / g["R"]

        def wk(a, p):
            return ks * (p * torch.cos(a) + torch.where(p == 0, 1.0, p / torch.tan(p)) * torch.sin(a))

        def slope(a, p):
            return torch.cos(a) + torch.sin(a) * (1.0 / torch.tan(p) - p / torch.sin(p) ** 2)
        # forward rebinning: rows of w_kappa(alpha_c, psi_k)
        s = wk(al[None, :], psi[:, None]) / g["dw"] + 0.5 * (rows - 1) - g["row_offset"]
        r0 = torch.floor(s)
        t = s - r0
        F = torch.zeros(cols, n_psi, rows + 2, **f64)          # row r at r + 1, ends dropped
        i0 = (r0.clamp(-1, rows) + 1).long().t()[:, :, None]
        i1 = ((r0 + 1).clamp(-1, rows) + 1).long().t()[:, :, None]
        F.scatter_add_(2, i0, (1.0 - t).t()[:, :, None].contiguous())
        F.scatter_add_(2, i1, t.t()[:, :, None].contiguous())
        self.F = F[:, :, 1:-1].contiguous()
        # psi_hat: the root of w_kappa(alpha_c, .) = w_r on the branch through 0
        pm = torch.full_like(al, psi_max)
        turn = self._bisect(lambda p: -slope(al.abs(), p), torch.full_like(al, 1e-3), pm)
        end = torch.where(slope(al.abs(), pm) < 0, turn, pm)
        hi = torch.where(al > 0, end, pm)
        lo = torch.where(al < 0, -end, -pm)
        W, A = w[:, None].expand(rows, cols), al[None, :].expand(rows, cols)
        LO, HI = lo[None, :].expand(rows, cols), hi[None, :].expand(rows, cols)
        ph = self._bisect(lambda p: wk(A, p) - W, LO.clone(), HI.clone())
        ph = torch.where(W <= wk(A, LO), LO, torch.where(W >= wk(A, HI), HI, ph))
        q = (ph / dpsi + 0.5 * (n_psi - 1)).clamp(0, n_psi - 1)
        k0 = torch.floor(q).clamp(max=n_psi - 2)
        B = torch.zeros(cols, rows, n_psi, **f64)
        B.scatter_(2, k0.long().t()[:, :, None], (1.0 - (q - k0)).t()[:, :, None].contiguous())
        B.scatter_(2, k0.long().t()[:, :, None] + 1, (q - k0).t()[:, :, None].contiguous())
        self.B = B * self.cos[:, None, None]
        m = torch.arange(cols, device=device)[:, None] - torch.arange(cols, device=device)[None, :]
        self.T = torch.where(m % 2 != 0, 2.0 * g["dalpha"] / (PI * torch.sin(m.double() * g["dalpha"])), 0.0)
        self._pi_lines()

    @staticmethod
    def _bisect(f, lo, hi):
        for _ in range(70):
            mid = 0.5 * (lo + hi)
            up = f(mid) < 0
            lo, hi = torch.where(up, mid, lo), torch.where(up, hi, mid)
        return 0.5 * (lo + hi)

    def _pi_lines(self):
        """PI interval of every voxel in view units; the voxel lies on the chord of in-plane
        half-span gam at the signed fraction tau of its half-length."""
        g, gr, dev = self.g, self.grid, self.dev
        x, y, z = (gr[a + "_first"] + torch.arange(gr["n" + a], dtype=torch.float64, device=dev) * gr["d" + a]
                   for a in "xyz")
        self.x, self.y, self.z = x[None, :], y[:, None], z
        rho, phi = torch.hypot(self.x, self.y), torch.atan2(self.y, self.x)
        inside = rho * rho <= self.r_fov ** 2
        self.li = torch.empty(gr["nz"], gr["ny"], gr["nx"], dtype=torch.float64, device=dev)
        self.lo = torch.empty_like(self.li)

        def chord(th):
            gam = torch.acos(rho * torch.cos(th) / g["R"])
            return gam, rho * torch.sin(th) / (g["R"] * torch.sin(gam))
        views = []
        for j in range(gr["nz"]):
            zr = (float(z[j]) - g["z0"]) / self.h
            c = zr + g["lambda0"] - phi

            def f(th):
                gam, tau = chord(th)
                return th + c - gam * tau
            gam, tau = chord(self._bisect(f, -c - PI, -c + PI))
            li = (zr - gam * (1.0 + tau) - g["lambda_first"]) / self.dlam
            lo = (zr + gam * (1.0 - tau) - g["lambda_first"]) / self.dlam
            nf, nl = torch.floor(li - 0.5) + 1, torch.ceil(lo + 0.5) - 1
            ok = inside & (nf >= 1) & (nl <= g["n_views"] - 2)
            self.li[j] = torch.where(ok, li, 1e9)
            self.lo[j] = torch.where(ok, lo, -1e9)
            views.append((int(nf[ok].min()), int(nl[ok].max())) if bool(ok.any()) else (0, -1))
        self.views = views
        used = [v for v in views if v[0] <= v[1]]
        self.first = min(v[0] for v in used) if used else 1
        self.last = max(v[1] for v in used) if used else 0

    def _each_view(self):
        """(view, slice range, flat index of the first tap in the padded view, row and column
        weights, coverage weight over v*) for every filtered view."""
        g, gr = self.g, self.grid
        rows, cols = g["det_rows"], g["det_cols"]
        for n in range(self.first, self.last + 1):
            on = [j for j, (a, b) in enumerate(self.views) if a <= n <= b]
            if not on:
                continue
            sl = slice(on[0], on[-1] + 1)
            lam = g["lambda_first"] + n * self.dlam
            b = lam + g["lambda0"]
            u = -self.x * math.sin(b) + self.y * math.cos(b)
            v = g["R"] - self.x * math.cos(b) - self.y * math.sin(b)
            cc = torch.atan2(u, v) / g["dalpha"] + 0.5 * (cols - 1) - g["col_offset"]
            c0 = torch.floor(cc)
            q = g["D"] / (torch.hypot(u, v) * g["dw"])
            rr = q * (self.z[sl] - g["z0"] - self.h * lam)[:, None, None]
            rr += 0.5 * (rows - 1) - g["row_offset"]
            r0 = torch.floor(rr)
            tr = rr.sub_(r0)
            idx = r0.clamp_(-2, rows).add_(2).mul_(cols + 4).add_(c0.clamp(-2, cols) + 2).long()
            cov = torch.minimum(n + 0.5 - self.li[sl], self.lo[sl] - (n - 0.5)).clamp_(0.0, 1.0)
            yield n, sl, idx, tr, cc - c0, cov.div_(v)

    def _lambda_alpha(self, s):
        """g2 of the filtered views among consecutive sinogram views s (eqs. Deriv, LW)."""
        a, b = 1.0 / (2.0 * self.dlam), 1.0 / (2.0 * self.g["dalpha"])
        if self.half:
            d = s[1:] - s[:-1]
            e = s[:, :, 1:] - s[:, :, :-1]
            out = a * (d[:, :, 1:] + d[:, :, :-1]) + b * (e[1:] + e[:-1])
        else:
            p = torch.nn.functional.pad(s[1:-1], (1, 1))
            out = a * (s[2:] - s[:-2]) + b * (p[:, :, 2:] - p[:, :, :-2])
        return out * self.lw[None, :, None]

    def recon(self, sino):
        gr, cols = self.grid, self.g["det_cols"]
        vol = torch.zeros(gr["nz"], gr["ny"], gr["nx"], dtype=torch.float64, device=self.dev)
        gF, lo, width, pre = None, 0, self.g["det_cols"] + 4, 0 if self.half else 1
        for n, sl, idx, tr, tc, wgt in self._each_view():
            if gF is None or n >= lo + gF.shape[0]:
                lo, hi = n, min(self.last + 1, n + 128)
                g2 = self._lambda_alpha(sino[lo - pre:hi + 1].double())
                V = g2.shape[0]
                g3 = torch.bmm(self.F, g2.permute(2, 1, 0).contiguous())
                g4 = (self.T @ g3.reshape(cols, -1)).reshape(g3.shape)
                gF = torch.nn.functional.pad(torch.bmm(self.B, g4).permute(2, 1, 0), (2, 2, 2, 2)).reshape(V, -1)
            img = gF[n - lo]
            top = img[idx]
            top += tc * (img[idx + 1] - top)
            idx += width
            bot = img[idx]
            bot += tc * (img[idx + 1] - bot)
            vol[sl] += wgt * (top + tr * (bot - top))
        return vol * (self.dlam / (2.0 * PI))

    def adjoint(self, fbar):
        g, rows, cols = self.g, self.g["det_rows"], self.g["det_cols"]
        V = self.last - self.first + 1
        f = fbar.double() * (self.dlam / (2.0 * PI))
        gb = torch.zeros(max(V, 0), (rows + 4) * (cols + 4), dtype=torch.float64, device=self.dev)
        for n, sl, idx, tr, tc, wgt in self._each_view():
            a = wgt * f[sl]
            on = a != 0
            k, a, tr = idx[on], a[on], tr[on]
            tc = tc.expand(idx.shape)[on]
            img = gb[n - self.first]
            for step, p in ((0, (1 - tr) * (1 - tc)), (1, (1 - tr) * tc), (cols + 4, tr * (1 - tc)),
                            (cols + 5, tr * tc)):
                img.index_add_(0, k + step, a * p)
        n_s = g["n_views"] + (1 if self.half else 0)
        out = torch.zeros(n_s, rows, cols + (1 if self.half else 0), dtype=torch.float64, device=self.dev)
        a, b = 1.0 / (2.0 * self.dlam), 1.0 / (2.0 * g["dalpha"])
        for i in range(0, V, 128):
            gF = gb[i:i + 128].reshape(-1, rows + 4, cols + 4)[:, 2:-2, 2:-2]
            g4 = torch.bmm(self.B.transpose(1, 2).contiguous(), gF.permute(2, 1, 0).contiguous())
            g3 = (self.T.t() @ g4.reshape(cols, -1)).reshape(g4.shape)
            g2 = torch.bmm(self.F.transpose(1, 2).contiguous(), g3).permute(2, 1, 0) * self.lw[None, :, None]
            m, n = self.first + i, g2.shape[0]
            if self.half:
                for dv, dc, c in ((0, 0, -a - b), (0, 1, b - a), (1, 0, a - b), (1, 1, a + b)):
                    out[m + dv:m + dv + n, :, dc:dc + cols] += c * g2
            else:
                out[m + 1:m + 1 + n] += a * g2
                out[m - 1:m - 1 + n] -= a * g2
                out[m:m + n, :, 1:] += b * g2[:, :, :-1]
                out[m:m + n, :, :-1] -= b * g2[:, :, 1:]
        return out


def _mulhilo(a, b):
    """High and low words of the 128-bit products of 64-bit words held in int64 (a tensor and
    a Python integer)."""
    mask = 0xFFFFFFFF
    a0, a1 = a & mask, (a >> 32) & mask
    b0, b1 = b & mask, b >> 32
    p, q, r, s = a0 * b0, a0 * b1, a1 * b0, a1 * b1
    t = q + ((p >> 32) & mask)
    u = r + (t & mask)
    return s + ((t >> 32) & mask) + ((u >> 32) & mask), (u << 32) | (p & mask)


def _signed(v):
    return v - (1 << 64) if v >= 1 << 63 else v


def _noise64(g, M, I0, var, seed, base):
    """The noisy values of elements 2 base, 2 base + 1, ... (Philox4x64-10 blocks of the counters
    base, base + 1, ..., Box-Muller, Poisson counts by their normal limit)."""
    pairs = (g.numel() + 1) // 2
    c = [torch.arange(base, base + pairs, device=g.device)] + [torch.zeros(pairs, dtype=torch.int64, device=g.device)] * 3
    k0, k1 = seed, 0
    for _ in range(10):
        h0, l0 = _mulhilo(c[0], 0xD2E7470EE14C6C93)
        h1, l1 = _mulhilo(c[2], 0xCA5A826395121157)
        c = [h1 ^ c[1] ^ _signed(k0), l1, h0 ^ c[3] ^ _signed(k1), l0]
        k0, k1 = (k0 + 0x9E3779B97F4A7C15) % (1 << 64), (k1 + 0xBB67AE8584CAA73B) % (1 << 64)
    u = [((x >> 40) & 0xFFFFFF).double() for x in c]
    u1 = (torch.stack((u[0], u[2]), -1).reshape(-1)[:g.numel()] + 1) * 2.0 ** -24
    u2 = torch.stack((u[1], u[3]), -1).reshape(-1)[:g.numel()] * 2.0 ** -24
    rho = torch.sqrt(-2.0 * torch.log(u1))
    lam = I0 * torch.exp(-g / M)
    counts = lam + torch.sqrt(lam) * rho * torch.cos(2 * PI * u2) + math.sqrt(var) * rho * torch.sin(2 * PI * u2)
    return M * torch.log(I0 / counts.clamp(min=1.0))


def _data64(case, seed):
    sp = _sparse_data(case, seed)
    step, cols, ns = case["step"], case["cols"], sp.shape[-1]
    c = torch.arange(cols, device="cuda")
    j0, j1 = c // step, (c // step + 1).clamp(max=ns - 1)
    t = (c % step).double() / step
    full = torch.empty(sp.shape[:-1] + (cols,), dtype=torch.float64, device="cuda")
    for a in range(0, sp.shape[0], 256):
        s = sp[a:a + 256].double()
        full[a:a + 256] = s[..., j0] + t * (s[..., j1] - s[..., j0])
    M = float(full.float().max())
    flat, noisy = full.reshape(-1), torch.empty(full.numel(), dtype=torch.float64, device="cuda")
    for a in range(0, flat.numel(), 1 << 24):
        noisy[a:a + (1 << 24)] = _noise64(flat[a:a + (1 << 24)], M, 1e5, 0.5, seed, a // 2)
    return full, noisy.reshape(full.shape)


def _metrics64(case, seed):
    f, r = (v.double() for v in _volumes(case, seed))
    L = float(r.max() - r.min())
    c1, c2 = (0.01 * L) ** 2, (0.03 * L) ** 2
    mf, mr = f.mean(), r.mean()
    cov = ((f - mf) * (r - mr)).mean()
    ssim = (2 * mf * mr + c1) * (2 * cov + c2) / (
        (mf * mf + mr * mr + c1) * (((f - mf) ** 2).mean() + ((r - mr) ** 2).mean() + c2))
    return torch.stack((((f - r) ** 2).mean().sqrt(), ssim))


def _subnet64(case, seed):
    convs, acts, last = _weights(case, seed)
    train = case["train"]
    leaf = lambda t: t.double().cuda().requires_grad_(train)  # noqa: E731
    convs, acts, last = [[leaf(t) for t in c] for c in convs], [leaf(a) for a in acts], [leaf(t) for t in last]
    x = _image(case, seed).double().requires_grad_(train)
    conv = torch.nn.functional.conv3d
    with torch.set_grad_enabled(train):
        h, total = x, 0.0
        for (w, b), a in zip(convs, acts):
            h = torch.nn.functional.prelu(conv(h, w, b, padding=1), a)
            total = total + h
        y = x + conv(total, last[0], last[1], padding=1)
    if not train:
        return y
    y.backward(torch.randn(x.shape, device="cuda", generator=_generator(seed + 3)).double())
    params = [t for c in convs for t in c] + acts + last
    return y.detach(), x.grad, [p.grad for p in params]


def exact(case, seed):
    kind = case["kind"]
    if kind == "data":
        return _data64(case, seed)
    if kind == "metrics":
        return _metrics64(case, seed)
    if kind == "subnet":
        return _subnet64(case, seed)
    if kind == "group":
        out = []
        for i, c in enumerate(_group(case)):
            geom, grid = _geometry(c)
            out.append(_Scan64(geom, grid).recon(_sinogram(geom, grid, seed * 131 + i)))
        return out
    geom, grid = _geometry(case)
    # scattering every (voxel, view) pair of a large volume in float64 takes minutes
    if kind in ("adjoint", "train") and work(case)["flops"] > 4e11:
        return None
    scan = _Scan64(geom, grid, case.get("half", False))
    if kind == "adjoint":
        return scan.adjoint(_cotangent(grid, seed))
    sino = _scan_input(case, seed)
    if kind != "train":
        return scan.recon(sino)
    G = _cotangent(grid, seed, case["batch"])
    return (torch.stack([scan.recon(s) for s in sino]), torch.stack([scan.adjoint(f) for f in G]))
