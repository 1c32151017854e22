"""Room of the first output pool of a top-k run: what chunked reservations leave unused is
added, but never past the pool's bound (a quarter of the free device memory)."""
import ctypes

import pytest


@pytest.mark.parametrize("cap,waves", [(65536, 12), (8_388_608, 3072), (1 << 29, 3072), (1000, 1)])
def test_slack_stays_within_the_bound(cap, waves):
    from paper_2409_03095_amd import mcmi
    fn = mcmi._lib["_ZN4mcmi15pool_with_slackElll"]
    fn.restype = ctypes.c_int64
    fn.argtypes = [ctypes.c_int64] * 3
    chunk = min(max(cap // (4 * waves), 256), 32768)
    want = cap + cap // 8 + waves * chunk
    assert fn(cap, 1 << 31, waves) == want
    for most in (cap, cap + 1, want - 1, want, want + 1):
        assert fn(cap, most, waves) == min(want, most)
    assert fn(cap, cap // 2, waves) == cap  # the least that a run starts with
