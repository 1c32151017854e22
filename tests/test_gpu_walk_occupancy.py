"""The grid of a walk is sized for the instance that runs: with tables of 512 slots the
small-table instance holds four waves per SIMD, all the others three."""
import ctypes

import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("f32,top,lanes,chains,workgroups",
                         [(1, 0, 64, 1, 4), (1, 0, 0, 1, 4), (1, 1, 64, 1, 3), (1, 0, 64, 2, 3), (1, 0, 32, 1, 3),
                          (1, 0, 16, 1, 3), (1, 0, 8, 1, 3), (0, 0, 64, 1, 3), (0, 0, 64, 2, 3), (0, 1, 64, 1, 3)])
def test_workgroups_per_cu(f32, top, lanes, chains, workgroups):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2409_03095_amd import mcmi
    torch.zeros(1, device="cuda")
    fn = mcmi._lib["_ZN4mcmi14walk_occupancyEbbiiiiPi"]
    fn.argtypes = [ctypes.c_bool, ctypes.c_bool] + [ctypes.c_int] * 4 + [ctypes.POINTER(ctypes.c_int)]
    got = ctypes.c_int()
    assert fn(bool(f32), bool(top), lanes, chains, 512, 4, ctypes.byref(got)) == 0
    print(f"[gpu] f32={f32} top={top} lanes={lanes} chains={chains}: {got.value} workgroups of 4 waves", flush=True)
    assert got.value == workgroups
