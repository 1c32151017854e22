"""Allocation network: the order of a training step's FP32 sums. A tile of 16 samples adds
its squared errors four at a time (samples q, 4 + q, 8 + q, 12 + q), a workgroup its four
tiles' shares of dW2 and db3 in index order."""
import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def mc():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2409_03095_amd import mcmi
    return mcmi


def net_and_samples(mc, seed):
    rng = np.random.default_rng(seed)
    x = torch.from_numpy(rng.normal(0, 1, size=(400, 8)).astype(np.float32)).cuda()
    t = torch.from_numpy(rng.normal(0, 1, size=400).astype(np.float32)).cuda()
    p = O.mlp_init(seed)
    net = mc.Mlp()
    net.set_params(np.concatenate([p[k].reshape(-1) for k, _ in O.MLP_SHAPES]).astype(np.float32))
    return net, x, t, rng


@pytest.mark.parametrize("batch", [1, 7, 16, 37, 64, 200])
def test_loss_is_the_sum_in_tile_order(mc, batch):
    # bit for bit: squares of the FP32 errors of the network's own predictions, then one
    # FP32 addition after the other
    net, x, t, rng = net_and_samples(mc, 3)
    idx = rng.integers(0, 400, size=batch).astype(np.int32)
    _, loss = net.gradient(x, t, torch.from_numpy(idx).cuda())
    err = (net.predict(x).cpu().numpy() - t.cpu().numpy())[idx]
    sq = np.zeros(-(-batch // 64) * 64, np.float32)
    sq[:batch] = err * err
    total = np.float32(0)
    for wg in sq.reshape(-1, 4, 4, 4):  # workgroup, tile, sample / 4, sample mod 4
        s = np.float32(0)
        for a, b, c, d in wg.transpose(0, 2, 1).reshape(-1, 4):
            s = np.float32(s + np.float32(np.float32(np.float32(a + b) + c) + d))
        total = np.float32(total + s)
    assert np.float32(loss) == total / np.float32(batch)


@pytest.mark.parametrize("seed", range(4))
def test_gradient_adds_its_tiles_in_order(mc, seed):
    # dW2 and db3; a power of two of samples: a tile's share is its own gradient times
    # 16 / batch exactly
    net, x, t, rng = net_and_samples(mc, 4 + seed)
    idx = rng.integers(0, 400, size=64).astype(np.int32)
    g = net.gradient(x, t, torch.from_numpy(idx).cuda())[0]
    s = np.zeros_like(g)
    for k in range(4):
        s = s + net.gradient(x, t, torch.from_numpy(idx[16 * k:16 * k + 16]).cuda())[0] * np.float32(0.25)
    assert np.array_equal(g[576:4672], s[576:4672])
    assert g[4800] == s[4800]
