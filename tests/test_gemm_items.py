"""The backward GEMM's work-item order (csrc/hdl_internal.h), enumerated on the
CPU by a compiled checker."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def checker(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    exe = str(tmp_path_factory.mktemp("items") / "gemm_items_check")
    subprocess.run([hipcc, "-O2", "-std=c++17", "--offload-arch=gfx950", os.path.join(HERE, "gemm_items_check.cpp"),
                    "-o", exe], check=True, capture_output=True)
    return exe


# tiles_m, tiles_n, splits, gm, gn: one tile; fewer tiles than a group; whole
# groups; remainders in both directions; the vocabulary by d of the largest
@pytest.mark.parametrize("grid", [(1, 1, 1, 1, 1), (2, 8, 16, 2, 4), (3, 1, 64, 3, 1), (16, 8, 2, 8, 4), (11, 7, 3, 8, 4),
                                  (9, 2, 5, 16, 2), (594, 20, 1, 8, 4)])
def test_every_item_once(checker, grid):
    r = subprocess.run([checker, *map(str, grid)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout
