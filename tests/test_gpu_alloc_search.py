"""The allocation's lambda search takes a sequential bisection's decisions exactly (equal
predictions make exp exact): budgets around the smallest total, one that ends the search
early, one that no lambda reaches; and row features where rows outgrow their lanes."""
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


def search(csum, budget):
    """lambda for equal rows (e = 1): total(lam) = clip(rint(lam), 1, 2^31 - 1) csum."""
    def total(lam):
        return int(min(max(np.rint(lam), 1.0), 2147483647.0)) * csum

    lo, hi = 0.0, 1.0
    while total(hi) <= budget and hi < 1e30:
        hi *= 2.0
    for _ in range(100):
        mid = 0.5 * (lo + hi)
        if total(mid) <= budget:
            lo = mid
        else:
            hi = mid
    return lo


@pytest.mark.parametrize("n", [1, 256, 257, 200001])
@pytest.mark.parametrize("mult", [0.5, 1.0, 1.5, 2.0, 63.7, 32768.0, 1e6, 4e9])
def test_lambda_is_the_sequential_search(mc, n, mult):
    rng = np.random.default_rng(n)
    cost = rng.integers(1, 40, size=n).astype(np.int32)
    csum = int(cost.sum())
    budget = max(1, int(mult * csum))
    print(f"[gpu] allocation n={n} budget={budget}", flush=True)
    chains, lam, fb = mc.allocate(torch.zeros(n, device="cuda"), torch.from_numpy(cost).cuda(), budget)
    ref = search(csum, budget)
    assert fb == (ref == 0.0) and lam == ref
    want = max(1, budget // csum) if fb else int(min(max(np.rint(ref), 1.0), 2147483647.0))
    assert np.all(chains.cpu().numpy() == want)


def test_features_of_rows_longer_than_their_lanes(mc):
    B = I.block_diag([I.grid2d_5pt(40, 41), I.wide_rows(150, {0: 149, 3: 65, 9: 64, 11: 63}, seed=3)])
    assert B.nnz / B.n - 1 < 10
    f = mc.row_features(mc.Cdf(mc.DeviceCsr.from_host(B)), 1e-3).cpu().numpy()
    ref = O.Oracle(B).features(1e-3)
    assert np.allclose(f, ref, rtol=2e-6, atol=1e-6), np.abs(f - ref).max(axis=0)
