"""The walk kernels' table (csrc/walk_common.hpp, Probe) compiled for the host and driven by
the 64 lanes of a modelled wavefront (tests/lane_model): a key is held by the table or by
the spill set, never by both, and its sum is that of its additions."""
import os
import re
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
MODEL = os.path.join(HERE, "lane_model")


@pytest.fixture(scope="module")
def clang():
    exe = "/opt/rocm/llvm/bin/clang++"
    exe = exe if os.path.exists(exe) else shutil.which("clang++")
    if not exe:
        pytest.skip("no clang++ (the headers use its vector types)")
    return exe


def run_model(clang, tmp_path, name):
    exe = str(tmp_path / name)
    subprocess.run([clang, "-O1", "-std=c++17", "-w", "-I", MODEL, os.path.join(MODEL, name + ".cpp"), "-o", exe],
                   check=True, capture_output=True, text=True)
    return subprocess.run([exe], check=True, capture_output=True, text=True, timeout=300).stdout


def test_a_key_is_in_one_place(clang, tmp_path):
    out = run_model(clang, tmp_path, "probe")
    print(out)
    lines = re.findall(r"(\d+) both, (\d+) twice, (\d+) wrong, (\d+) spilled", out)
    assert len(lines) == 12
    for both, twice, wrong, spilled in lines:
        assert both == twice == wrong == "0" and int(spilled) > 0
