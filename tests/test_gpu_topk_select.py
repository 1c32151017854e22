"""Top-k retention in the wavefront kernel where its selection can go wrong: many equal
values (cut by ascending column), k at and around the number of survivors, more survivors
than the selection's registers hold, every lane grouping."""
import numpy as np
import pytest

import oracle as O
from paper_2409_03095_amd import inputs as I
from parity import compare_topk

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def mc():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2409_03095_amd import mcmi
    return mcmi


def check(mc, B, prec, k, chains, **kw):
    print(f"[gpu] topk select n={B.n} prec={prec} k={k} chains={chains} {kw}", flush=True)
    run = dict(seed=5, chains=chains, delta=kw.pop("delta", 1e-3), eps=kw.pop("eps", 0.0), topk=k)
    max_len = kw.pop("max_len", 0)
    res = mc.spai(mc.Cdf(mc.DeviceCsr.from_host(B)), mc.params(walk_prec=prec, max_len=max_len, **run, **kw))
    out = res.to_numpy()
    o = O.Oracle(B)
    orc = o.spai(fp32=prec == 32, max_len=max_len, filter_on_m=bool(kw.get("filter", 0)), **run)
    assert res.stats.transitions == orc["transitions"]
    compare_topk(out, orc, o.diag, chains)


@pytest.mark.parametrize("prec", [32, 64])
@pytest.mark.parametrize("k", [1, 2, 3, 5, 8, 63, 64, 65, 200])
def test_equal_values_are_cut_by_column(mc, k, prec):
    # one or few chains on a uniform stencil: whole groups of columns hold the same weight
    check(mc, I.grid2d_5pt(23, 19), prec, k, 3)


@pytest.mark.parametrize("prec", [32, 64])
@pytest.mark.parametrize("k", [9, 10, 11, 128, 257, 300])
def test_k_around_the_survivors(mc, k, prec):
    # a cycle's chains keep exactly max_len + 1 entries
    for kept in (10, 300):
        check(mc, I.scaled_cycle(401, -0.97), prec, k, 2, delta=1e-300, max_len=kept - 1, hash_slots=1024)


@pytest.mark.parametrize("prec", [32, 64])
def test_more_survivors_than_the_selection_holds(mc, prec):
    check(mc, I.scaled_cycle(701, 0.99), prec, 40, 2, delta=1e-300, max_len=600, hash_slots=2048)


@pytest.mark.parametrize("lanes", [8, 16, 32, 64])
@pytest.mark.parametrize("filt", [0, 1])
def test_groupings_and_filter(mc, lanes, filt):
    check(mc, I.random_nonsym(700, seed=36), 32, 7, 24, lanes_per_row=lanes, filter=filt, eps=1e-3, delta=1e-4)


def test_exact_first_pool_needs_no_second_pass(mc):
    B = I.aniso27(24, rho=0.9, seed=2)
    res = mc.spai(mc.Cdf(mc.DeviceCsr.from_host(B)), mc.params(seed=1, chains=32, delta=1e-3, eps=1e-3, walk_prec=32,
                                                               topk=32))
    assert res.stats.retries == 0 and res.nnz == 32 * B.n
