"""The rank form of an ensemble, checked on the host.

`paper_2411_10764_amd/csrc/rank_pack.cpp` (threshold codes, search tables and
tree records of the rank walks) is compiled under the address and
undefined-behaviour sanitizers with `tests/rank_check_driver.cpp`, which packs
random ensembles (perfect trees of depth 4 to 12 in byte, half-word and packed
tiles; ragged trees with default directions; tables longer than a slot;
thresholds with infinities, signed zeros and subnormals),
ranks and walks rows with the kernels' arithmetic, checks every access against
its table, slot or tile, and compares every leaf with the unpacked tree's.
"""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2411_10764_amd", "csrc")


def test_rank_form_walks_to_the_same_leaves(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "rank_check_driver")
    r = subprocess.run([gxx, "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined",
                        "-fno-sanitize-recover=all", "-ffp-contract=off", "-Wall", "-Werror",
                        "-I", CSRC, os.path.join(HERE, "rank_check_driver.cpp"),
                        os.path.join(CSRC, "rank_pack.cpp"), os.path.join(CSRC, "pack.cpp"),
                        "-pthread", "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    lines = r.stdout.splitlines()
    assert len(lines) == 23 and all(line.startswith("ok ") for line in lines), r.stdout
    for mode in ("byte", "half", "packed", "ragged byte", "ragged half"):
        assert any(f", {mode}, " in line for line in lines), r.stdout
