"""Record build and CSR assembly where a wave or workgroup takes a number of rows that is
neither the smallest nor the largest, batched norms across group ends, and the reduction
cut's digit search with few and many distinct digits."""
import numpy as np
import pytest

import oracle as O
from paper_2409_03095_amd import inputs as I
from parity import check_compact_records, compare_spai, decode_records

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def mc():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2409_03095_amd import mcmi
    return mcmi


@pytest.mark.parametrize("nx,ny", [(205, 100), (131, 128)])
def test_rows_per_group(mc, nx, ny):
    B = I.family_5pt(3, nx, ny)
    cdf = mc.Cdf(mc.DeviceCsr.from_host(B))
    o = O.Oracle(B)
    rec, roff, diag = cdf.download()
    for i, r in enumerate(decode_records(rec, roff, B.n)):
        b, e = o.cptr[i], o.cptr[i + 1]
        assert r[0] == i and r[1] == e - b and np.array_equal(r[6], o.ccol[b:e])
        assert np.array_equal(r[8], o.athr[b:e].astype(np.int64))
    check_compact_records(cdf.download_compact(), roff, o, np.random.default_rng(1), draws=8)
    res = mc.spai(cdf, mc.params(seed=2, chains=3, delta=1e-3, eps=1e-3))
    ref = o.spai(seed=2, chains=3, delta=1e-3, eps=1e-3)
    compare_spai(res.to_numpy(), ref, o.diag, 3)


def test_batched_norms_at_group_ends(mc):
    mats = [I.family_5pt(k, a, b) for k, (a, b) in enumerate([(64, 64), (1, 1), (3, 1), (64, 64), (90, 91), (2, 31)])]
    cdf = mc.Cdf.batched([mc.DeviceCsr.from_host(m) for m in mats])
    _, base, norm = cdf.batch_info()
    assert np.array_equal(np.diff(base), [m.n for m in mats])
    assert np.array_equal(norm, [O.Oracle(m).norm_inf for m in mats])


@pytest.mark.parametrize("frac", [0.01, 0.37, 0.99])
@pytest.mark.parametrize("name", ["one_value", "few_values", "many_values"])
def test_reduction_cut(mc, name, frac):
    B = {"one_value": lambda: I.grid2d_5pt(40, 30), "few_values": lambda: I.aniso27(13, noise=0.0),
         "many_values": lambda: I.random_nonsym(4000, seed=3)}[name]()
    cdf = mc.Cdf(mc.DeviceCsr.from_host(B), drop_frac=frac)
    c = np.sort(np.abs(O.Oracle(B).cval))
    cut = c[int(np.floor(frac * c.size))]
    _, got, dropped = cdf.prep_info()
    assert got == cut and dropped == int(np.sum(c < cut))
