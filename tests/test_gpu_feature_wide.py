"""Row features of rows that a whole wavefront takes (more than 256 entries) among short ones."""
import numpy as np
import pytest

import oracle as O
from paper_2409_03095_amd import inputs as I

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("grid", [None, (60, 61)])  # 16 and 4 lanes per row
def test_features_of_wide_rows(grid):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2409_03095_amd import mcmi as mc
    wide = I.wide_rows(900, {0: 256, 1: 257, 2: 255, 3: 899, 40: 300, 897: 258, 899: 512, 450: 513}, seed=4)
    B = wide if grid is None else I.block_diag([wide, I.grid2d_5pt(*grid), I.grid2d_5pt(*grid)])
    per_row = B.nnz / B.n - 1
    assert 10 < per_row <= 40 if grid is None else per_row <= 10
    f = mc.row_features(mc.Cdf(mc.DeviceCsr.from_host(B)), 1e-3).cpu().numpy()
    # binary64 sums rounded once: a few units of binary32
    assert np.allclose(f, O.Oracle(B).features(1e-3), rtol=2e-6, atol=1e-6)
