"""Pilot walks at the edges of a chain's own table: around its first, second and last
size (48, 96 and 160 states), full tables, one and several chains per lane."""
import numpy as np
import pytest

import oracle as O
from paper_2409_03095_amd import inputs as I

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def mc():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2409_03095_amd import mcmi
    return mcmi


@pytest.mark.parametrize("prec", [64, 32])
@pytest.mark.parametrize("pilot", [1, 64, 130])
@pytest.mark.parametrize("max_len", [1, 3, 4, 46, 47, 48, 95, 96, 159])
def test_pilot_at_table_sizes(mc, max_len, pilot, prec):
    # a cycle fills max_len + 1 slots in every chain; on the grid chains revisit states
    B = I.block_diag([I.scaled_cycle(211, -0.97), I.grid2d_5pt(9, 8, diag=4.1)])
    print(f"[gpu] pilot tables max_len={max_len} pilot={pilot} prec={prec}", flush=True)
    cdf = mc.Cdf(mc.DeviceCsr.from_host(B))
    p = mc.params(seed=4, delta=1e-30, walk_prec=prec, max_len=max_len)
    var, ln = (t.cpu().numpy() for t in mc.pilot_variance(cdf, p, pilot))
    rv, rl = O.Oracle(B).pilot(seed=4, pilot=pilot, delta=1e-30, fp32=prec == 32, max_len=max_len)
    assert np.array_equal(ln, rl)
    assert np.all(np.abs(var - rv) <= 1e-10 * np.abs(rv) + 1e-12)


def test_pilot_chain_longer_than_the_largest_table(mc):
    cdf = mc.Cdf(mc.DeviceCsr.from_host(I.scaled_cycle(211, 0.97)))
    with pytest.raises(mc.McmiError) as e:
        mc.pilot_variance(cdf, mc.params(seed=4, delta=1e-30, max_len=160), 3)
    assert e.value.status == -5
