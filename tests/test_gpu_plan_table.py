"""Plans do not rerun rows: their tables hold what the row with most chains reaches (up to
1024 entries), also where the typical row would do with a smaller table."""
import numpy as np
import pytest

from paper_2409_03095_amd import inputs as I

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("slots", [0, 848])  # automatic; what an eager run reported
@pytest.mark.parametrize("hot", [70, 90, 105])
def test_plan_keeps_the_rows_with_most_chains(hot, slots):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2409_03095_amd import mcmi as mc
    # a row of `hot` chains reaches 850 to 1010 columns, one of 10 chains about 220
    B = I.random_nonsym(1200, seed=14)
    cpr = np.full(B.n, 10, np.int32)
    cpr[[5, 600, 1100]] = hot
    cpr = torch.from_numpy(cpr).cuda()
    cdf = mc.Cdf(mc.DeviceCsr.from_host(B))
    p = mc.params(seed=8, chains=1, delta=1e-4, eps=1e-9, walk_prec=32, max_len=25)
    res = mc.spai(cdf, p, chains_per_row=cpr)
    rp, col, _ = res.to_numpy()
    p.hash_slots = slots
    plan = mc.Plan(cdf, p, 400 * B.n, chains_per_row=cpr)
    plan.launch(8)
    out, st, overflow = plan.result()
    assert not overflow and st.hash_slots == 1024
    assert np.diff(rp).max() > 800 and np.array_equal(out[0], rp) and np.array_equal(out[1], col)
