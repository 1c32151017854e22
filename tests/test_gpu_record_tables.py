"""Record build: alias tables on both sides of the length that LDS holds, in one wave and
around a wave's rows, and the norm of B across the pieces that its entries come in."""
import numpy as np
import pytest

import oracle as O
from paper_2409_03095_amd import inputs as I
from parity import check_compact_records, decode_records

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def mc():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2409_03095_amd import mcmi
    return mcmi


def matrix(lengths, n, seed):
    """Row i has lengths[i % len] off-diagonal entries (and its diagonal), both signs, of widely
    different sizes."""
    g = np.random.default_rng(seed)
    r, c, v = [], [], []
    for i in range(n):
        m = min(lengths[i % len(lengths)], n - 1)
        cols = g.choice(n - 1, m, replace=False)
        cols += cols >= i
        a = g.choice([-1.0, 1.0], m) * np.exp2(g.uniform(-12, 0, m))
        r += [i] * (m + 1)
        c += [*cols, i]
        v += [*a, 1.5 * np.abs(a).sum() + 1.0]
    return I.from_coo(n, np.array(r), np.array(c), np.array(v))


@pytest.mark.parametrize("n,lengths", [(1, (0,)), (5, (4, 0)), (17, (1, 2)), (70, (31, 32, 33)), (300, (0, 65, 32)),
                                       (1500, (3, 1100, 7)), (65600, (2, 3, 1, 0, 40))])
def test_tables_and_norm(mc, n, lengths):
    print(f"[gpu] records n={n} lengths={lengths}", flush=True)
    B = matrix(lengths, n, n)
    o = O.Oracle(B)
    cdf = mc.Cdf(mc.DeviceCsr.from_host(B))
    rec, roff, diag = cdf.download()
    for i, r in enumerate(decode_records(rec, roff, B.n)):
        b, e = o.cptr[i], o.cptr[i + 1]
        assert r[0] == i and r[1] == e - b and np.array_equal(r[6], o.ccol[b:e])
        assert np.array_equal(r[8], o.athr[b:e].astype(np.int64))
    check_compact_records(cdf.download_compact(), roff, o, np.random.default_rng(1), draws=4)
    # ||B||_inf: each row summed in column order
    norm, _, _ = mc.Cdf(mc.DeviceCsr.from_host(B), alpha=1.0).prep_info()
    sums = [0.0] * n
    for i in range(n):
        for x in np.abs(B.val[B.row_ptr[i]:B.row_ptr[i + 1]]).tolist():
            sums[i] += x
    assert norm == max(sums)
