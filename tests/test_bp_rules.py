"""The backprojectors' launch rules on the host: the order in which a layer's tiles are taken, the
kernel instance and split of a plan, the launches of a batch, the adjoint's split."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CXX = "/opt/rocm/lib/llvm/bin/clang++"


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    if not os.path.exists(CXX):
        pytest.skip("ROCm clang++ not available")
    exe = str(tmp_path_factory.mktemp("rules") / "rules")
    r = subprocess.run([CXX, "-x", "c++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                        os.path.join(ROOT, "tests", "sanitize", "rules_driver.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]

    def ask(*lines):
        r = subprocess.run([exe], input="\n".join(lines) + "\n", capture_output=True, text=True, timeout=60)
        assert r.returncode == 0, r.stderr
        return [line.split() for line in r.stdout.splitlines()]
    return ask


# around the least tiles of the forward (768) and the adjoint (1024), ragged bands and remainders
@pytest.mark.parametrize("tx,ty", [(24, 32), (13, 59), (27, 29), (769, 1), (1, 800), (32, 32), (33, 32), (31, 33),
                                   (35, 37), (41, 25), (64, 64), (130, 7)])
def test_every_tile_once(rules, tx, ty):
    assert rules(*(f"order {tx} {ty} 9 {least}" for least in (768, 1024, 1))) == [["ok"]] * 3


# shapes 32x64, 64x32, 64x64, 48x80, 64x80, 48x96, 48x128, then the HBM path (7)
PLANS = {"clinical": (32, 44, 32, 4), "half-clinical": (32, 44, 32, 2), "quarter-clinical": (32, 44, 32, 1),
         "sparse": (49, 25, 16, 3), "wide": (42, 103, 13, 4), "flat": (28, 79, 16, 2), "square": (58, 46, 16, 2),
         "tall": (53, 79, 16, 2), "long": (49, 79, 16, 6), "far": (70, 140, 16, 2)}


def _plan(name):
    """16-slice runs of full tiles, every voxel valid; a plan of `layers` 16-slice layers."""
    rows, cols, tiles, layers = PLANS[name]
    layers = {"clinical": 10, "half-clinical": 4, "quarter-clinical": 2}.get(name, layers)
    return (f"plan {name} 16 {rows} {cols} 4 {tiles * tiles * 256 * layers * 16} {tiles} {tiles} {16 * layers} "
            f"{16 * layers} 1 {layers}")


@pytest.mark.parametrize("names,shapes", [
    # no launch of an LDS shape is moved to the HBM path
    (("sparse", "wide"), (1, 6)), (("wide", "sparse"), (6, 1)), (("square", "wide"), (2, 6)),
    (("flat", "far"), (3, 7)), (("far", "far"), (7, 7)),
    # the nearest shape that can be joined, past one that cannot
    (("sparse", "wide", "tall"), (4, 6, 4)), (("flat", "wide", "square"), (4, 6, 4)),
    # a class of many tasks keeps its shape unless the new one serves it as well
    (("clinical", "sparse"), (0, 1)), (("half-clinical", "square"), (0, 2)), (("clinical", "tall"), (0, 4)),
    (("half-clinical", "tall"), (0, 4)), (("clinical", "flat"), (3, 3)),
    # few tasks join
    (("quarter-clinical", "flat"), (3, 3)), (("quarter-clinical", "square"), (2, 2)),
    (("quarter-clinical", "tall"), (4, 4)), (("long", "flat"), (4, 4)), (("half-clinical", "flat"), (3, 3))])
def test_batches(rules, names, shapes):
    out = rules(*(_plan(n) for n in set(names)), *(f"class {n}" for n in names), "batch " + " ".join(names))
    alone, got = out[:-1], [out[-1][i:i + 3] for i in range(0, len(out[-1]), 3)]
    # splits and polynomials, which decide the bits, stay as they are alone
    assert [c[1:] for c in got] == [c[1:] for c in alone] == [["0", "1"]] * len(names)
    assert tuple(int(c[0]) for c in got) == shapes


# voxels across, slices; whether teams of 256 lanes share a task's views
@pytest.mark.parametrize("nxy,nz,teams", [(512, 1, False), (512, 2, False), (480, 1, False), (448, 1, True), (400, 1, True),
                                          (400, 2, True), (304, 4, True), (320, 4, False), (256, 4, True),
                                          (256, 12, True), (352, 5, False), (64, 64, True), (96, 16, True)])
def test_thin_volumes(rules, nxy, nz, teams):
    """Layers of many workgroups keep single ones however few their voxels are."""
    tiles = nxy // 16
    line = f"plan p 16 15 24 4 {tiles * tiles * 256 * nz * 4 // 5} {tiles} {tiles} {nz} 49 {-(-nz // 49)} {-(-min(nz, 49) // 16)}"
    split = rules(line, "class p")[0][1]
    assert (split in ("2", "3")) == teams


@pytest.mark.parametrize("nz,box,split", [(1, "15 24", "4"), (5, "32 64", "4"), (8, "15 24", "4"), (9, "15 24", "1"),
                                          (5, "33 40", "0"), (8, "20 70", "0")])
def test_tasks_of_8_slices(rules, nz, box, split):
    """Volumes of at most 8 slices and the small box, at 16-slice runs only."""
    tiles, voxels = 27, 27 * 27 * 256 * nz
    line = f"plan p %d {box} 4 {voxels} {tiles} {tiles} {nz} 49 1 1"
    assert rules(line % 16, "class p")[0][1:] == [split, "0" if split == "1" else "1"]
    assert rules(line % 8, "class p")[0][1:] == ["0", "1"]


# boxes measured on either side of the line, slices a run; whether rows' sums are kept in a window
@pytest.mark.parametrize("kz,box,window", [
    (16, "20 36", 1), (16, "20 57", 1), (16, "32 44", 0), (16, "32 51", 0), (16, "32 53", 0), (16, "34 43", 0),
    (16, "40 49", 0), (16, "40 58", 0), (16, "40 62", 0), (16, "40 67", 1), (16, "53 66", 1), (32, "55 44", 1),
    (32, "65 49", 1), (8, "22 49", 0), (8, "20 57", 1)])
def test_adjoint_window(rules, kz, box, window):
    line = f"plan p {kz} {box} 4 {1 << 21} 16 16 32 49 1 2"
    assert rules(line, "adjoint p")[0][1:] == [str(window), "1"]


@pytest.mark.parametrize("pitches,split,parts", [(200, "3", 32), (2047, "3", 32), (2048, "3", 31), (16383, "3", 4),
                                                 (16384, "4", 3), (65535, "4", 1), (70000, "4", 1)])
def test_tall_volumes(rules, pitches, split, parts):
    """Layers times the tasks or parts of each stay within 65535 where the layers alone do."""
    line = f"plan p 16 12 14 4 {16 * pitches // 4} 1 1 {pitches} 1 {pitches} 1"
    out = rules(line, "class p", "adjoint p")
    assert out[0][1] == split and int(out[1][0]) == parts


def test_wide_volumes(rules):
    """Tasks times the threads of each stay below 2^32."""
    for tiles, split in ((1023, "3"), (1025, "0")):
        line = f"plan p 16 12 80 4 4096 {tiles} {tiles} 3 3 1 1"
        assert rules(line, "class p")[0][1] == split
