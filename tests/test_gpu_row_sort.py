"""Column order of a row's survivors in the wavefront kernel at the edges of its
register sort (64, 128 and 256 words), of its fallback, and of its 24-bit key span."""
import numpy as np
import pytest

import oracle as O
from paper_2409_03095_amd import inputs as I
from parity import compare_spai

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def mc():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2409_03095_amd import mcmi
    return mcmi


def check(mc, B, rows, prec, **kw):
    """A chain on a cycle visits max_len + 1 columns, which wrap around for the last rows."""
    print(f"[gpu] cycle n={B.n} prec={prec} {kw}", flush=True)
    run = dict(seed=3, chains=3, delta=1e-300, eps=0.0, max_len=kw["max_len"])
    cdf = mc.Cdf(mc.DeviceCsr.from_host(B))
    p = mc.params(walk_prec=prec, lanes_per_row=kw.get("lanes", 0), hash_slots=kw.get("hash_slots", 0), **run)
    t = None if rows is None else torch.from_numpy(np.asarray(rows, np.int32)).cuda()
    res = mc.spai(cdf, p, rows=t)
    out = res.to_numpy()
    o = O.Oracle(B)
    ref = o.spai(fp32=prec == 32, rows=rows, **run)
    assert res.stats.transitions == ref["transitions"]
    assert np.array_equal(np.diff(out[0]), np.full(out[0].size - 1, kw["max_len"] + 1))
    compare_spai(out, ref, o.diag, 3, rows=rows)


@pytest.mark.parametrize("prec", [32, 64])
@pytest.mark.parametrize("slots", [0, 1024])
@pytest.mark.parametrize("kept", [2, 63, 64, 65, 127, 128, 129, 255, 256, 257, 300])
def test_sorted_columns_at_word_counts(mc, kept, slots, prec):
    check(mc, I.scaled_cycle(401, -0.95), None, prec, max_len=kept - 1, hash_slots=slots)


@pytest.mark.parametrize("prec", [32, 64])
@pytest.mark.parametrize("kept", [5, 64, 65])
def test_sorted_columns_in_shared_wavefronts(mc, kept, prec):
    check(mc, I.scaled_cycle(401, -0.95), None, prec, max_len=kept - 1, lanes=16, hash_slots=1024)


def test_keys_spanning_more_than_24_bits(mc):
    """Record offsets of the first and last rows are 1.7e7 units apart: the last rows' chains wrap."""
    n = 8_500_000
    rows = np.array([0, 1, n // 2, n - 150, n - 100, n - 60, n - 3, n - 1], np.int32)
    check(mc, I.scaled_cycle(n, 0.9), rows, 32, max_len=99)
