"""Top-k selection of the wavefront kernel (csrc/walk.hip, select_top) compiled for the host
and run by 64 modelled lanes against a sort."""
import os
import subprocess

from test_probe_lanes import HERE, MODEL, clang  # noqa: F401

WALK = os.path.join(HERE, "..", "paper_2409_03095_amd", "csrc", "walk.hip")


def test_selection_is_that_of_a_sort(clang, tmp_path):  # noqa: F811
    text = open(WALK).read()
    begin = text.index("template <bool kCmp>\n__device__ __forceinline__ void select_top")
    part = tmp_path / "select_top.hpp"
    part.write_text(text[begin:text.index("\n}\n", begin) + 3])
    exe = str(tmp_path / "select")
    subprocess.run([clang, "-O1", "-std=c++17", "-w", "-I", MODEL, f'-DSELECT_TOP="{part}"',
                    os.path.join(MODEL, "select.cpp"), "-o", exe],
                   check=True, capture_output=True, text=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr[-2000:]
