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


def _run_driver(tmp_path, name, sources, sanitize="address,undefined"):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / name)
    r = subprocess.run([gxx, "-std=c++17", "-O1", "-g", "-fsanitize=" + sanitize,
                        "-fno-sanitize-recover=all", "-ffp-contract=off", "-Wall", "-Werror",
                        "-I", CSRC, os.path.join(HERE, name + ".cpp"),
                        *(os.path.join(CSRC, s) for s in sources), "-pthread", "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout


def test_rank_form_walks_to_the_same_leaves(tmp_path):
    out = _run_driver(tmp_path, "rank_check_driver", ["rank_pack.cpp", "pack.cpp"])
    lines = out.splitlines()
    assert len(lines) == 23 and all(line.startswith("ok ") for line in lines), out
    for mode in ("byte", "half", "packed", "ragged byte", "ragged half"):
        assert any(f", {mode}, " in line for line in lines), out


def test_every_tile_and_depth_has_a_launch_shape(tmp_path):
    """rank_plan.cpp: a shape for every tile and depth, and launches that stage
    whole slots within the LDS; the estimates choose the faster of two measured
    walks (tests/rank_plan_driver.cpp)."""
    assert _run_driver(tmp_path, "rank_plan_driver", ["rank_plan.cpp"]).strip() == "ok"


def test_loading_loops(tmp_path):
    """host_parallel.h under the thread sanitizer (tests/host_parallel_driver.cpp)."""
    assert _run_driver(tmp_path, "host_parallel_driver", [], "thread").strip() == "ok"
