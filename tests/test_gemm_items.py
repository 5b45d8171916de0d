"""The backward GEMM's work-item order (csrc/hdl_internal.h), enumerated on the
CPU by a compiled checker."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


def _build(tmp_path_factory, name):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    exe = str(tmp_path_factory.mktemp("items") / name)
    subprocess.run([hipcc, "-O2", "-std=c++17", "--offload-arch=gfx950", os.path.join(HERE, name + ".cpp"),
                    "-o", exe], check=True, capture_output=True)
    return exe


@pytest.fixture(scope="module")
def checker(tmp_path_factory):
    return _build(tmp_path_factory, "gemm_items_check")


@pytest.fixture(scope="module")
def split_checker(tmp_path_factory):
    return _build(tmp_path_factory, "dh_split_check")


# tiles_m, tiles_n, splits, gm, gn: one tile; fewer tiles than a group; whole
# groups; remainders in both directions; the vocabulary by d of the largest
@pytest.mark.parametrize("grid", [(1, 1, 1, 1, 1), (2, 8, 16, 2, 4), (3, 1, 64, 3, 1), (16, 8, 2, 8, 4), (11, 7, 3, 8, 4),
                                  (9, 2, 5, 16, 2), (594, 20, 1, 8, 4)])
def test_every_item_once(checker, grid):
    r = subprocess.run([checker, *map(str, grid)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout


# every number of scored rows (in steps) of: one tile; a small vocabulary with
# an odd number of slices; 16 splits; 1 split; a ragged last tile row; wide rows;
# a whole chunk
@pytest.mark.parametrize("shape", [(40, 8, 300), (200, 256, 448), (300, 2048, 151936), (4096, 4096, 151936),
                                   (3000, 1024, 32000), (700, 5120, 20000), (32768, 2048, 32000)])
def test_split_for_the_scored_rows(split_checker, shape):
    r = subprocess.run([split_checker, *map(str, shape)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout
