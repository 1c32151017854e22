"""Binary64 walks on record sets of more than 1 GiB: survivors sorted in LDS (also up to 256
of them) and rows taken off the queues three at a time."""
import numpy as np
import pytest

import oracle as O
from paper_2409_03095_amd import inputs as I
from parity import compare_spai

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def cycle():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2409_03095_amd import mcmi as mc
    B = I.scaled_cycle(8_500_000, -0.95)  # 128 bytes of full records per row
    return mc, mc.Cdf(mc.DeviceCsr.from_host(B)), O.Oracle(B)


# a chain on the cycle visits max_len + 1 columns; the last rows' chains wrap around
@pytest.mark.parametrize("kept", [2, 63, 64, 65, 128, 129, 255, 256, 257, 300])
@pytest.mark.parametrize("count", [1, 3, 4, 49])
def test_rows_of_a_large_record_set(cycle, kept, count):
    mc, cdf, o = cycle
    print(f"[gpu] large records kept={kept} rows={count}", flush=True)
    rows = np.unique(np.linspace(0, o.n - 1, count).astype(np.int32))
    run = dict(seed=3, chains=3, delta=1e-300, eps=0.0, max_len=kept - 1)
    res = mc.spai(cdf, mc.params(walk_prec=64, **run), rows=torch.from_numpy(rows).cuda())
    ref = o.spai(rows=rows, **run)
    assert res.stats.transitions == ref["transitions"]
    out = res.to_numpy()
    assert np.array_equal(np.diff(out[0]), np.full(rows.size, kept))
    compare_spai(out, ref, o.diag, 3, rows=rows)
