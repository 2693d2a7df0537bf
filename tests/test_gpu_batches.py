"""Unsplit plans of every box shape, alone and in batches whose classes share a launch or stay apart
(the rules' own answer, asked of the host driver, says which): the same bits as alone, and alone the
values of 8-slice runs, which have other instances."""
import pytest

from synth import configs
from test_bp_rules import rules  # noqa: F401  (fixture)

torch = pytest.importorskip("torch")
K = pytest.importorskip("paper_2201_02309_amd")

pytestmark = pytest.mark.gpu

# box shape: voxels across, detector columns and rows
SPECS = {0: (200, 330, 16), 1: (200, 100, 48), 2: (160, 400, 48), 3: (160, 600, 32), 4: (160, 600, 48),
         5: (160, 740, 32), 6: (160, 950, 32), 7: (160, 100, 64)}
BATCHES = [((0, 3), (3, 3)), ((0, 1), (2, 2)), ((1, 3), (4, 4)), ((2, 3), (4, 4)), ((0, 6), (6, 6)),
           ((1, 6), (1, 6)), ((3, 7), (3, 7)), ((5, 2, 7), (5, 2, 7)), ((0, 1, 2, 3, 4, 5, 6, 7), None)]


def _geometry(shape):
    nxy, cols, rows = SPECS[shape]
    wl = configs.tiny(nxy=nxy, nz=48, cols=cols, rows=rows, views_per_turn=72, turns=4, feed=24.0, dxy=1.2,
                      slices_per_pitch=24)
    return wl.geom.as_dict(), wl.grid.as_dict()


def _line(name, plan, grid):
    i = plan.info
    tiles = -(-grid["nx"] // 16)
    return (f"plan {name} {i['bp_slices']} {i['bp_box_rows']} {i['bp_box_cols']} {i['atan_degree']} "
            f"{i['n_valid_voxels']} {tiles} {tiles} {grid['nz']} {i['slices_per_pitch']} {i['n_pitches']} "
            f"{-(-i['n_table_slices'] // 16)}")


@pytest.fixture(scope="module")
def items():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    out = {}
    for shape in SPECS:
        geom, grid = _geometry(shape)
        plan = K.Plan(geom, grid, device=0)
        torch.manual_seed(shape)
        sino = torch.rand(geom["n_views"], geom["det_rows"], geom["det_cols"], device="cuda")
        gF = K.filter_views(plan, sino)
        out[shape] = (plan, gF, K.backproject(plan, gF), _line(shape, plan, grid), sino)
    return out


@pytest.mark.parametrize("shape", SPECS)
def test_unsplit_shapes(items, rules, shape):  # noqa: F811
    plan, gF, vol, line, sino = items[shape]
    assert rules(line, f"class {shape}") == [[str(shape), "0", "1"]]
    geom, grid = _geometry(shape)
    other = K.Plan(geom, grid, device=0, bp_slices=8)
    ref = K.recon(other, sino)
    assert bool(((vol == 0) == (ref == 0)).all())
    err = float((vol - ref).double().norm() / ref.double().norm())
    print(f"[parity] shape {shape}: {err:.2e}", flush=True)
    # sums of the same ~50 float32 terms in another order
    assert err <= 25 * 2.0 ** -24
    other.close()


@pytest.mark.parametrize("names,shapes", BATCHES)
def test_batches(items, rules, names, shapes):  # noqa: F811
    said = rules(*(items[n][3] for n in names), "batch " + " ".join(map(str, names)))[0]
    print(f"[case] {names}: {said}", flush=True)
    assert shapes is None or tuple(map(int, said[::3])) == shapes
    for order in (names, names[::-1]):
        vols = K.backproject_batch([items[n][0] for n in order], [items[n][1] for n in order])
        for n, v in zip(order, vols):
            assert torch.equal(v, items[n][2])
