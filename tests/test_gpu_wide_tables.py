"""Wavefront tables that are no power of two (FP32 walks of rows with a small typical
reach): chain counts whose reach is just below and above the limit, single rows that
overflow them, reruns with larger tables, plans."""
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


# max_len 20: N (L + 1) = 504, 525, 840, 861
@pytest.mark.parametrize("chains,slots", [(24, 512), (25, 848), (40, 848), (41, 1024)])
@pytest.mark.parametrize("eps", [1e-6, 1e-3])
def test_table_size_follows_the_reach(mc, chains, slots, eps):
    B = I.random_nonsym(1500, seed=13)
    print(f"[gpu] wide tables chains={chains} eps={eps}", flush=True)
    run = dict(seed=7, chains=chains, delta=1e-5, eps=eps, max_len=20)
    res = mc.spai(mc.Cdf(mc.DeviceCsr.from_host(B)), mc.params(walk_prec=32, **run))
    assert res.stats.hash_slots == slots
    o = O.Oracle(B)
    ref = o.spai(fp32=True, **run)
    assert ref["guard"] == 0  # no sum so near eps that its order decides
    assert res.stats.transitions == ref["transitions"]
    compare_spai(res.to_numpy(), ref, o.diag, chains)


@pytest.mark.parametrize("eps", [1e-6, 1e-3])
def test_rows_that_overflow_the_typical_table(mc, eps):
    # a mean of about 12 chains sets 848 slots; a few rows reach several thousand columns
    B = I.random_nonsym(1200, seed=14)
    cpr = I.chain_counts(B.n, mean=10.0, hi=40)
    cpr[[3, 77, 600, 1199]] = [400, 700, 1000, 64]
    res = mc.spai(mc.Cdf(mc.DeviceCsr.from_host(B)),
                  mc.params(seed=8, chains=1, delta=1e-4, eps=eps, walk_prec=32, max_len=25),
                  chains_per_row=torch.from_numpy(cpr).cuda())
    o = O.Oracle(B)
    ref = o.spai(seed=8, chains=1, delta=1e-4, eps=eps, fp32=True, max_len=25, chains_per_row=cpr)
    assert ref["guard"] == 0
    assert res.stats.spilled > 0 and res.stats.transitions == ref["transitions"]
    compare_spai(res.to_numpy(), ref, o.diag, cpr)


def test_plan_with_the_small_table(mc):
    B = I.family_5pt(3, 37, 41)
    cdf = mc.Cdf(mc.DeviceCsr.from_host(B))
    p = mc.params(seed=1, chains=9, delta=1e-3, eps=1e-3, walk_prec=32)
    plan = mc.Plan(cdf, p, 400 * B.n)
    for seed in (1, 2, 3):
        plan.launch(seed)
        (rp, col, val), st, ovf = plan.result()
        p.seed = seed
        res = mc.spai(cdf, p)
        a = res.to_numpy()
        assert not ovf and st.hash_slots == res.stats.hash_slots == 848
        assert np.array_equal(rp, a[0]) and np.array_equal(col, a[1]) and np.array_equal(val, a[2])
