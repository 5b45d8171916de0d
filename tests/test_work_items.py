"""The fused kernel's work-item order for any number of scored rows
(csrc/plan.h), enumerated on the CPU by a compiled checker."""
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
    exe = str(tmp_path_factory.mktemp("items") / "work_items_check")
    subprocess.run([hipcc, "-O2", "-std=c++17", "--offload-arch=gfx950", os.path.join(HERE, "work_items_check.cpp"),
                    "-o", exe], check=True, capture_output=True)
    return exe


# one row; less than a tile; a tile and a remainder; several groups of row
# tiles with 1, 2 and 3 left; many chunks, few, one; a large launch
@pytest.mark.parametrize("n_rows,vocab,d", [(1, 1, 8), (1, 151936, 2048), (96, 151936, 2048), (300, 4096, 256),
                                            (384, 151936, 2048), (513, 151936, 2048), (700, 21000, 64),
                                            (1554, 151936, 4096), (3333, 50257, 1000), (9 * 256, 9000, 64),
                                            (65024, 151936, 2048)])
def test_every_item_once_and_shared_tiles(checker, n_rows, vocab, d):
    r = subprocess.run([checker, str(n_rows), str(vocab), str(d)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout
