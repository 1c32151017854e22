"""Top-k retention under the M filter where kept values M_rc underflow to zero: the places
left are filled by ascending column."""
import numpy as np
import pytest

import oracle as O
from paper_2409_03095_amd import inputs as I
from parity import compare_topk

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("prec", [32, 64])
@pytest.mark.parametrize("k", [3, 40, 70, 100])
def test_underflowing_values(prec, k):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2409_03095_amd import mcmi as mc
    # N_rc = 2^-j exactly; M_rc = N_rc / 1e308 is zero from j = 52 on
    B = I.scaled_cycle(300, 0.5, 1e308)
    run = dict(seed=5, chains=2, delta=1e-300, eps=0.0, topk=k, max_len=100)
    res = mc.spai(mc.Cdf(mc.DeviceCsr.from_host(B)), mc.params(walk_prec=prec, filter=1, **run))
    o = O.Oracle(B)
    orc = o.spai(fp32=prec == 32, filter_on_m=True, **run)
    rp, col, val = res.to_numpy()
    print(f"[gpu] k={k} prec={prec}: {np.count_nonzero(val == 0.0)} of {val.size} values are zero", flush=True)
    assert np.array_equal(rp, np.arange(301) * k)
    compare_topk((rp, col, val), orc, o.diag, 2)
