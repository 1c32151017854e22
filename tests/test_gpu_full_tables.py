"""Wavefront tables that most rows fill up or overflow: every row's columns are unique and in
order, and pattern and values are those of a run whose table holds all of a row."""
import numpy as np
import pytest

from paper_2409_03095_amd import inputs as I

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def mc():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2409_03095_amd import mcmi
    return mcmi


def run(mc, cdf, chains_per_row=None, **kw):
    res = mc.spai(cdf, mc.params(seed=5, eps=1e-3, **kw), chains_per_row=chains_per_row)
    return res, *res.to_torch()


def check(mc, cdf, small, cpr=None, **kw):
    res, rp, col, val = run(mc, cdf, cpr, **small, **kw)
    ref, rp2, col2, val2 = run(mc, cdf, cpr, hash_slots=4096, **kw)
    print(f"[gpu] {small} {kw}: {res.stats.spilled} of {res.stats.transitions} spilled", flush=True)
    assert res.stats.spilled > 1000 and ref.stats.spilled == 0
    up = torch.ones(col.numel(), dtype=torch.bool, device=col.device)
    up[1:] = col[1:] > col[:-1]
    up[rp[:-1]] = True  # a row's first entry
    assert bool(up.all())
    assert res.stats.transitions == ref.stats.transitions
    assert torch.equal(rp, rp2) and torch.equal(col, col2)
    assert torch.allclose(val, val2, rtol=1e-12, atol=1e-15)


# with 512, 256 and 128 slots one key in 1e4 to 1e5 was once held by table and spill set
@pytest.mark.parametrize("slots,chains,delta", [(512, 64, 1e-3), (256, 64, 1e-2), (128, 24, 1e-3)])
@pytest.mark.parametrize("prec", [32, 64])
def test_given_tables(mc, slots, chains, delta, prec):
    cdf = mc.Cdf(mc.DeviceCsr.from_host(I.aniso27(64, rho=0.75, seed=1)))
    check(mc, cdf, dict(hash_slots=slots), chains=chains, delta=delta, walk_prec=prec)


def test_automatic_table_and_many_rows_past_it(mc):
    # a mean of 22 chains takes 848 slots; every eighth row has 120
    B = I.aniso27(64, rho=0.75, seed=2)
    cpr = np.full(B.n, 8, np.int32)
    cpr[::8] = 120
    cdf = mc.Cdf(mc.DeviceCsr.from_host(B))
    check(mc, cdf, {}, cpr=torch.from_numpy(cpr).cuda(), chains=1, delta=1e-4, walk_prec=32)
    assert run(mc, cdf, torch.from_numpy(cpr).cuda(), chains=1, delta=1e-4, walk_prec=32)[0].stats.hash_slots == 848
