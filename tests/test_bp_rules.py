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
