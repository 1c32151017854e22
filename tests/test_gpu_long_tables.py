"""Alias tables of rows around the length from which a whole wavefront fills their stacks,
several of them in one wavefront."""
import numpy as np
import pytest

import oracle as O
from parity import check_compact_records, decode_records
from test_gpu_record_tables import matrix, mc  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,lengths", [(600, (511, 512, 513)), (700, (2, 640, 32, 641, 33)), (1030, (1029, 0, 576, 575, 5))])
def test_long_tables(mc, n, lengths):  # noqa: F811
    print(f"[gpu] long tables n={n} lengths={lengths}", flush=True)
    from paper_2409_03095_amd import mcmi
    B = matrix(lengths, n, n)
    o = O.Oracle(B)
    cdf = mcmi.Cdf(mcmi.DeviceCsr.from_host(B))
    rec, roff, _ = cdf.download()
    for i, r in enumerate(decode_records(rec, roff, B.n)):
        b, e = o.cptr[i], o.cptr[i + 1]
        assert r[1] == e - b and np.array_equal(r[6], o.ccol[b:e])
        assert np.array_equal(r[8], o.athr[b:e].astype(np.int64))
    check_compact_records(cdf.download_compact(), roff, o, np.random.default_rng(1), draws=4)
