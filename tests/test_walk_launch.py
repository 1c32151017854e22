"""Tables that are no power of two launch in the small-table instance of the walk only (on
the host, without a GPU: what is not refused ends with the runtime's no-device error)."""
import ctypes
import os
import subprocess

import pytest

from test_probe_lanes import MODEL, clang  # noqa: F401

INVALID = 1  # hipErrorInvalidValue
SYMBOL = "_ZN4mcmi11launch_walkERKNS_8WalkArgsEbiiP12ihipStream_t"


def test_table_sizes_of_the_instances(clang, tmp_path):  # noqa: F811
    import torch
    if torch.cuda.is_available():
        pytest.skip("launches nothing: for machines without a GPU")
    from paper_2409_03095_amd import mcmi
    so = str(tmp_path / "launch.so")
    subprocess.run([clang, "-O1", "-std=c++17", "-w", "-shared", "-fPIC", "-I", MODEL,
                    os.path.join(MODEL, "launch.cpp"), "-o", so], check=True, capture_output=True, text=True)
    lib = ctypes.CDLL(so)
    fn = ctypes.cast(getattr(mcmi._lib, SYMBOL), ctypes.c_void_p)
    for f32, slots, lanes, chains, topk, ok in [
            (1, 848, 64, 1, 0, True), (1, 848, 0, 1, 0, True), (1, 512, 64, 1, 0, True), (1, 1024, 16, 1, 0, True),
            (0, 1024, 64, 2, 3, True), (1, 848, 64, 2, 0, False), (1, 848, 32, 1, 0, False),
            (1, 848, 64, 1, 5, False), (0, 848, 64, 1, 0, False), (1, 846, 64, 1, 0, False),
            (1, 1536, 64, 1, 0, False), (1, 0, 64, 1, 0, False)]:
        rc = lib.try_launch(fn, f32, slots, lanes, chains, topk)
        assert (rc != INVALID) == ok, (f32, slots, lanes, chains, topk, rc)
