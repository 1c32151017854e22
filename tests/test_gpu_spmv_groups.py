"""y = M x: a row's sum is that of V strided partial sums added as a binary tree, bit for
bit, in every lane grouping (row lengths around V, empty rows, one very long row)."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def mc():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2409_03095_amd import mcmi
    return mcmi


def tree_sum(prod, V):
    acc = np.zeros(V)
    for k0 in range(0, prod.size, V):
        part = prod[k0:k0 + V]
        acc[:part.size] += part
    while acc.size > 1:
        acc = acc[:acc.size // 2] + acc[acc.size // 2:]
    return acc[0]


@pytest.mark.parametrize("mean_len,V", [(1, 8), (6, 8), (13, 16), (23, 16), (25, 32), (33, 32), (41, 32), (90, 32),
                                        (120, 16), (250, 64)])
def test_row_sums_are_the_tree_of_strided_partial_sums(mc, mean_len, V):
    rng = np.random.default_rng(mean_len)
    n = 1003
    lens = rng.integers(max(mean_len - 5, 0), mean_len + 6, n)
    lens[::50] = 0
    lens[7] = n
    while not {8: 0, 16: 12 if mean_len < 96 else 96, 32: 24, 64: 192}[V] <= lens.sum() / n:
        lens[rng.integers(8, n, 40)] += 1
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    col = np.concatenate([np.sort(rng.choice(n, int(k), replace=False)) for k in lens]).astype(np.int32)
    val, x = rng.standard_normal(col.size), rng.standard_normal(n)
    print(f"[gpu] spmv tree mean={col.size / n:.2f} V={V}", flush=True)
    t = [torch.from_numpy(a).cuda() for a in (rp, col, val, x)]
    y = torch.full((n,), np.nan, dtype=torch.float64, device="cuda")
    M = mc.CsrOut(n, int(col.size), t[0].data_ptr(), t[1].data_ptr(), t[2].data_ptr())
    mc._check(mc._lib.mcmi_apply(ctypes.byref(M), ctypes.c_int64(n), ctypes.c_void_p(t[3].data_ptr()),
                                 ctypes.c_void_p(y.data_ptr()), mc._stream(None)))
    ref = np.array([tree_sum(val[rp[i]:rp[i + 1]] * x[col[rp[i]:rp[i + 1]]], V) for i in range(n)])
    assert np.array_equal(y.cpu().numpy(), ref)
