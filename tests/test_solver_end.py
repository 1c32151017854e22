"""The BiCGstab kernels (csrc/krylov.hip) compiled for the host: the waves of a workgroup
agree on whether the solve has ended, also where it ends while they start."""
import os
import subprocess

import pytest

from test_probe_lanes import HERE, MODEL, clang  # noqa: F401

KRYLOV = os.path.join(HERE, "..", "paper_2409_03095_amd", "csrc", "krylov.hip")


def test_waves_agree_on_the_end(clang, tmp_path):  # noqa: F811
    text = open(KRYLOV).read()
    kernels = text[text.index("namespace {\n\nconstexpr int kDotBlocks"):text.index("unsigned grid_dot(")]
    part = tmp_path / "kernels.hpp"
    part.write_text(kernels + "}\n")
    exe = str(tmp_path / "solver_end")
    subprocess.run([clang, "-O1", "-std=c++17", "-w", "-I", MODEL, f'-DSOLVER_KERNELS="{part}"',
                    os.path.join(MODEL, "solver_end.cpp"), "-o", exe], check=True, capture_output=True, text=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
