"""Backprojector and adjoint over the footprint-box shapes their kernels are built for: boxes of
at most 32 and 64 columns, wider ones, deeper than 32 rows, and beyond the LDS (HBM path), on
ragged grids, against the FP64 oracle; and the backprojector's splits of small grids over more
workgroups."""
import numpy as np
import pytest

import oracle as O
from synth import configs, phantom

torch = pytest.importorskip("torch")
K = pytest.importorskip("paper_2201_02309_amd")

pytestmark = pytest.mark.gpu

# nxy, columns, rows, slices per pitch -> box rows x columns
SHAPES = [(40, 24, 24, 24, 28, 17), (20, 47, 8, 12, 12, 46), (20, 100, 12, 12, 16, 90),
          (40, 24, 48, 10, 52, 17), (24, 60, 40, 8, 44, 48), (20, 130, 16, 12, 20, 116),
          (20, 180, 20, 12, 24, 158), (18, 420, 40, 12, 44, 405)]


@pytest.mark.parametrize("bp_slices", [16, 8, 32])
@pytest.mark.parametrize("nxy,cols,rows,spp,box_rows,box_cols", SHAPES)
def test_box_shapes(nxy, cols, rows, spp, box_rows, box_cols, bp_slices):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    wl = configs.tiny(nxy=nxy, nz=14, cols=cols, rows=rows, views_per_turn=72, turns=3, feed=24.0,
                      dxy=2.0, slices_per_pitch=spp)
    geom, gr = wl.geom.as_dict(), wl.grid.as_dict()
    print(f"[case] {nxy}^2, detector {rows} x {cols}, runs of {bp_slices}", flush=True)
    plan = K.Plan(geom, gr, device=0, bp_slices=bp_slices)
    det = K.Plan(geom, gr, device=0, bp_slices=bp_slices, deterministic_adjoint=True)
    if bp_slices == 16:
        assert (plan.info["bp_box_rows"], plan.info["bp_box_cols"]) == (box_rows, box_cols)
    sino = phantom.project(phantom.make_phantom(wl.phantom, gr, wl.seed), geom).astype(np.float32)
    ref, valid = O.recon(O.Scan(geom), gr, sino)
    vol = K.recon(plan, torch.from_numpy(sino).cuda()).cpu().numpy()
    err = np.linalg.norm((vol - ref)[valid]) / np.linalg.norm(ref[valid])
    y = np.random.default_rng(nxy).normal(size=ref.shape).astype(np.float32)
    tref = O.recon_T(O.Scan(geom), gr, y.astype(np.float64))
    yd = torch.from_numpy(y).cuda()
    errs = []
    for p in (plan, det):
        g = K.recon_backward(p, yd).double().cpu().numpy()
        errs.append(np.linalg.norm(g - tref) / np.linalg.norm(tref))
    print(f"[parity] recon {err:.2e}, adjoint {errs[0]:.2e}, deterministic {errs[1]:.2e}", flush=True)
    # the parity bar; a random cotangent sees the column coordinate's float32 rounding itself,
    # up to an ulp of the box's width in cells
    assert np.all(vol[~valid] == 0) and err <= 1e-5
    assert max(errs) <= 1e-5 + 2.0 ** -23 * box_cols


# whole 16 x 16 x 16 tasks' worth of voxels: 64, 144, 294 and 478, on either side of each limit
@pytest.mark.parametrize("nxy,nz", [(64, 64), (96, 64), (112, 96), (140, 100)])
def test_splits(nxy, nz):
    """16-slice runs, split over workgroups by the grid's size, against 8-slice runs, which never
    are: sums of the same ~50 float32 terms in another order.  Alone, in stages and in a group the
    bits are the same."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    wl = configs.tiny(nxy=nxy, nz=nz, cols=96, rows=16, views_per_turn=72, turns=6, feed=48.0, dxy=2.0,
                      slices_per_pitch=24)
    geom, gr = wl.geom.as_dict(), wl.grid.as_dict()
    print(f"[case] {nxy}^2 x {nz}", flush=True)
    plan, ref_plan = K.Plan(geom, gr, device=0), K.Plan(geom, gr, device=0, bp_slices=8)
    torch.manual_seed(0)
    sino = torch.rand(geom["n_views"], geom["det_rows"], geom["det_cols"], device="cuda")
    vol, ref = K.recon(plan, sino), K.recon(ref_plan, sino)
    assert bool(((vol == 0) == (ref == 0)).all())
    err = float((vol - ref).double().norm() / ref.double().norm())
    print(f"[parity] {err:.2e}", flush=True)
    assert err <= 25 * 2.0 ** -24
    gF = K.filter_views(plan, sino)
    assert torch.equal(K.backproject(plan, gF), vol)
    other = K.filter_views(ref_plan, sino * 2)
    both = K.backproject_batch([plan, plan], [gF, other])
    assert torch.equal(both[0], vol) and torch.equal(both[1], K.backproject(plan, other))


@pytest.mark.parametrize("bad", [float("nan"), float("inf"), 3.0e38])
def test_adjoint_of_values_that_are_not_finite(bad):
    """One voxel's cotangent not finite, or near the largest float: views that none of its tile's
    voxels see are unchanged, and a finite one is the float64 transpose's."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    wl = configs.tiny(nxy=20, nz=14, cols=100, rows=12, views_per_turn=72, turns=3, feed=24.0, dxy=2.0,
                      slices_per_pitch=12)
    geom, gr = wl.geom.as_dict(), wl.grid.as_dict()
    plan = K.Plan(geom, gr, device=0)
    y = np.random.default_rng(3).normal(size=(14, 20, 20)).astype(np.float32)
    clean = y.copy()
    clean[7, 4, 9] = 0.0
    y[7, 4, 9] = bad
    got = K.recon_backward(plan, torch.from_numpy(y).cuda()).cpu().numpy()
    if np.isfinite(bad):
        ref = O.recon_T(O.Scan(geom), gr, y.astype(np.float64))
        err = np.linalg.norm(got / 1e30 - ref / 1e30) / np.linalg.norm(ref / 1e30)
        print(f"[parity] adjoint of {bad}: {err:.2e}", flush=True)
        assert err <= 1e-5 + 2.0 ** -23 * 90
        return
    base = K.recon_backward(plan, torch.from_numpy(clean).cuda()).cpu().numpy()
    tile = np.zeros(y.shape)
    tile[:, :16, :16] = 1.0
    seen = (O.recon_T(O.Scan(geom), gr, tile) != 0).any(axis=(1, 2))
    assert not np.isfinite(got).all() and not seen.all()
    assert np.array_equal(np.isfinite(got[~seen]), np.ones_like(got[~seen], dtype=bool))
    assert np.allclose(got[~seen], base[~seen], atol=1e-5 * np.abs(base).max())


# tiles of a layer: 528 = 16 * 33 and 567 (ragged rows), in plain order, and 1023, 1056, 1089 around the
# least of the adjoint's order by XCD; slices of one and of two layers
@pytest.mark.parametrize("nx,ny,nz", [(520, 256, 5), (330, 432, 20), (528, 490, 5), (513, 505, 5), (520, 513, 18)])
def test_tile_order(nx, ny, nz):
    """Many tiles, in whatever order their blocks take them, against the same voxels in grids of few
    tiles: every voxel written, the adjoint the sum of the parts' adjoints."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    wl = configs.tiny(nxy=40, nz=nz, cols=96, rows=16, views_per_turn=72, turns=4, feed=24.0, dxy=2.0,
                      slices_per_pitch=12)
    geom, gr = wl.geom.as_dict(), wl.grid.as_dict()
    d = 80.0 / max(nx, ny)
    gr.update(nx=nx, ny=ny, dx=d, dy=d, x_first=-d * (nx - 1) / 2, y_first=-d * (ny - 1) / 2)
    print(f"[case] {nx} x {ny} x {nz}", flush=True)
    plan = K.Plan(geom, gr, device=0)
    torch.manual_seed(0)
    sino = torch.rand(geom["n_views"], geom["det_rows"], geom["det_cols"], device="cuda")
    y = torch.randn(nz, ny, nx, device="cuda")
    vol = K.recon(plan, sino, out=torch.full((nz, ny, nx), float("nan"), device="cuda"))
    gsino = K.recon_backward(plan, y)
    two = torch.full((2, nz, ny, nx), float("nan"), device="cuda")
    gF = K.filter_views(plan, sino)
    K.backproject_batch([plan, plan], [gF, gF], vols=[two[0], two[1]])
    assert torch.equal(two[0], vol) and torch.equal(two[1], vol)
    ref, gref = torch.empty_like(vol), torch.zeros_like(gsino, dtype=torch.float64)
    for j in range(0, ny, 176):
        for i in range(0, nx, 176):
            m, n = min(176, ny - j), min(176, nx - i)
            part = K.Plan(geom, dict(gr, nx=n, ny=m, x_first=gr["x_first"] + i * d, y_first=gr["y_first"] + j * d),
                          device=0)
            ref[:, j:j + m, i:i + n] = K.recon(part, sino)
            gref += K.recon_backward(part, y[:, j:j + m, i:i + n].contiguous()).double()
            part.close()
    # two float32 results, each within the parity bar of 1e-5
    assert bool(torch.isfinite(vol).all())
    assert float((vol - ref).double().norm() / ref.double().norm()) <= 2e-5
    assert float((gsino.double() - gref).norm() / gref.norm()) <= 2e-5 + 2.0 ** -22 * plan.info["bp_box_cols"]


# boxes of 65 to 80 columns, at most 48 rows and more
@pytest.mark.parametrize("rows,box_rows", [(44, 48), (60, 64)])
def test_box_shapes_of_80_columns(rows, box_rows):
    test_box_shapes(24, 100, rows, 8, box_rows, 75, 16)


def test_batch_of_unlike_boxes():
    """Requests with few tasks join one launch whatever their boxes: the same bits as alone."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    plans, gFs = [], []
    for nxy, cols, rows, spp in ((40, 24, 24, 24), (24, 100, 44, 8), (24, 100, 60, 8), (40, 24, 48, 10)):
        wl = configs.tiny(nxy=nxy, nz=14, cols=cols, rows=rows, views_per_turn=72, turns=3, feed=24.0,
                          dxy=2.0, slices_per_pitch=spp)
        geom = wl.geom.as_dict()
        plans.append(K.Plan(geom, wl.grid.as_dict(), device=0))
        torch.manual_seed(rows)
        gFs.append(K.filter_views(plans[-1], torch.rand(geom["n_views"], rows, cols, device="cuda")))
    alone = [K.backproject(p, g) for p, g in zip(plans, gFs)]
    for order in ((0, 1, 2, 3), (3, 2, 1, 0), (2, 1), (0, 2)):
        for i, v in zip(order, K.backproject_batch([plans[i] for i in order], [gFs[i] for i in order])):
            assert torch.equal(v, alone[i])
    # a plan alone has few tasks and is split over teams; as many voxels as are not, over two shapes
    big = []
    for cols, rows, spp in ((160, 16, 24), (60, 32, 12)):
        wl = configs.tiny(nxy=200, nz=48, cols=cols, rows=rows, views_per_turn=72, turns=4, feed=24.0, dxy=0.4,
                          slices_per_pitch=spp)
        geom = wl.geom.as_dict()
        p = K.Plan(geom, wl.grid.as_dict(), device=0)
        sino = torch.rand(geom["n_views"], rows, cols, device="cuda")
        big.append((p, K.filter_views(p, sino)))
    alone = [K.backproject(p, g) for p, g in big]
    for v, a in zip(K.backproject_batch(*zip(*big)), alone):
        assert torch.equal(v, a)


# volumes of at most 8 slices with many tiles, which take tasks of 8 slices, and of 9, which do not
@pytest.mark.parametrize("nxy,nz", [(440, 1), (300, 4), (300, 8), (300, 9)])
def test_thin_volumes(nxy, nz):
    """Against runs of 32 slices, which are never split, as in test_splits; alone, in stages and in a
    group the bits are the same."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    wl = configs.tiny(nxy=nxy, nz=nz, cols=96, rows=16, views_per_turn=72, turns=4, feed=48.0, dxy=200.0 / nxy,
                      slices_per_pitch=24)
    geom, gr = wl.geom.as_dict(), wl.grid.as_dict()
    print(f"[case] {nxy}^2 x {nz}", flush=True)
    plan, ref_plan = K.Plan(geom, gr, device=0), K.Plan(geom, gr, device=0, bp_slices=32)
    torch.manual_seed(0)
    sino = torch.rand(geom["n_views"], geom["det_rows"], geom["det_cols"], device="cuda")
    vol, ref = K.recon(plan, sino), K.recon(ref_plan, sino)
    assert bool(((vol == 0) == (ref == 0)).all())
    err = float((vol - ref).double().norm() / ref.double().norm())
    print(f"[parity] {err:.2e}", flush=True)
    assert err <= 25 * 2.0 ** -24
    gF = K.filter_views(plan, sino)
    assert torch.equal(K.backproject(plan, gF), vol)
    both = torch.full((2, nz, nxy, nxy), float("nan"), device="cuda")
    K.backproject_batch([plan, plan], [gF, gF], vols=[both[0], both[1]])
    assert torch.equal(both[0], vol) and torch.equal(both[1], vol)


def test_many_pitches():
    """A column of few voxels over more pitches than a launch has layers for the adjoint's largest
    split, against the same slices in four volumes."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    nz = 2200
    wl = configs.tiny(nxy=6, nz=nz, cols=24, rows=8, views_per_turn=16, turns=nz + 4, feed=24.0, dxy=2.0,
                      slices_per_pitch=1)
    geom, gr = wl.geom.as_dict(), wl.grid.as_dict()
    plan = K.Plan(geom, gr, device=0)
    assert plan.info["n_pitches"] == nz
    print(f"[case] {nz} pitches", flush=True)
    torch.manual_seed(0)
    sino = torch.rand(geom["n_views"], geom["det_rows"], geom["det_cols"], device="cuda")
    y = torch.randn(nz, 6, 6, device="cuda")
    vol = K.recon(plan, sino, out=torch.full((nz, 6, 6), float("nan"), device="cuda"))
    gsino = K.recon_backward(plan, y).double()
    ref, gref = torch.empty_like(vol), torch.zeros_like(gsino)
    for a in range(0, nz, nz // 4):
        part = K.Plan(geom, dict(gr, nz=nz // 4, z_first=gr["z_first"] + a * gr["dz"]), device=0)
        ref[a:a + nz // 4] = K.recon(part, sino)
        gref += K.recon_backward(part, y[a:a + nz // 4].contiguous()).double()
        part.close()
    # two float32 results, each within the parity bar of 1e-5
    assert bool((vol != 0).any(dim=(1, 2))[1:-1].all())
    assert float((vol - ref).double().norm() / ref.double().norm()) <= 2e-5
    assert float((gsino - gref).norm() / gref.norm()) <= 2e-5 + 2.0 ** -22 * plan.info["bp_box_cols"]


# 767, 768 and 783 tiles a layer, ragged rows and columns: around the least of the forward's order by XCD
@pytest.mark.parametrize("nx,ny,nz", [(201, 939, 3), (384, 512, 3), (425, 460, 18)])
def test_tile_order_of_the_forward(nx, ny, nz):
    test_tile_order(nx, ny, nz)
