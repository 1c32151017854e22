"""The kernel shape that a run reports can be given to another run."""
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


def test_reported_table_is_accepted(mc):
    cdf = mc.Cdf(mc.DeviceCsr.from_host(I.family_5pt(3, 37, 41)))
    run = dict(seed=1, chains=9, delta=1e-3, eps=1e-3)
    first = mc.spai(cdf, mc.params(walk_prec=32, **run))
    st = first.stats
    assert st.hash_slots == 848
    kw = dict(lanes_per_row=st.lanes_per_row, hash_slots=st.hash_slots)
    again = mc.spai(cdf, mc.params(walk_prec=32, **run, **kw))
    assert again.stats.hash_slots == 848
    assert all(np.array_equal(a, b) for a, b in zip(first.to_numpy(), again.to_numpy()))
    plan = mc.Plan(cdf, mc.params(walk_prec=32, **run, **kw), 400 * 37 * 41)
    plan.launch(1)
    got, _, ovf = plan.result()
    assert not ovf and all(np.array_equal(a, b) for a, b in zip(first.to_numpy(), got))


# a run whose kernel wants a power of two takes 1024 slots
@pytest.mark.parametrize("kw,prec,chains", [({}, 64, 9), (dict(topk=5), 32, 9), (dict(lanes_per_row=16), 32, 9),
                                            ({}, 32, 100), (dict(lanes_per_row=256), 32, 9)])
def test_reported_table_in_other_runs(mc, kw, prec, chains):
    cdf = mc.Cdf(mc.DeviceCsr.from_host(I.family_5pt(3, 37, 41)))
    run = dict(seed=1, chains=chains, delta=1e-3, eps=1e-3, walk_prec=prec, **kw)
    a = mc.spai(cdf, mc.params(hash_slots=848, **run))
    b = mc.spai(cdf, mc.params(hash_slots=1024, **run))
    assert a.stats.hash_slots == b.stats.hash_slots
    for x, y in zip(a.to_numpy(), b.to_numpy()):
        assert np.array_equal(x, y) if x.dtype.kind == "i" else np.allclose(x, y, rtol=1e-12, atol=1e-15)


@pytest.mark.parametrize("slots", [96, 840, 844, 852, 32, 16384])
def test_other_sizes_stay_refused(mc, slots):
    cdf = mc.Cdf(mc.DeviceCsr.from_host(I.family_5pt(3, 7, 9)))
    p = mc.params(seed=1, chains=9, delta=1e-3, eps=1e-3, walk_prec=32, hash_slots=slots)
    for call in (lambda: mc.spai(cdf, p), lambda: mc.Plan(cdf, p, 5000)):
        with pytest.raises(mc.McmiError) as e:
            call()
        assert e.value.status == -1
