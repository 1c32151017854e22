"""Allocation network: gradients at batch sizes around a tile (16), a workgroup's round (64)
and the grid's limit (several rounds per workgroup), reruns of a training, and the
feature statistics at row counts around the workgroup size."""
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


def flat(p):
    return np.concatenate([p[k].reshape(-1) for k, _ in O.MLP_SHAPES]).astype(np.float32)


def bf16(a):
    return O.bf16_round(np.asarray(a, np.float32)).astype(np.float64)


def reference(p, x, t):
    """The network in FP64 on the operands the matrix cores get, rounded to BF16: weights,
    inputs, layer-1 activations and the layer-2 gradient (so that a ReLU of an activation
    near zero opens on both sides, which a batch of a few samples feels)."""
    q = {k: v.astype(np.float64) for k, v in p.items()}
    w1, w2, w3 = (bf16(p[k]) for k in ("w1", "w2", "w3"))
    xb = bf16(x)
    h1 = bf16(np.maximum(xb @ w1.T + q["b1"], 0.0))
    h2 = np.maximum(h1 @ w2.T + q["b2"], 0.0)
    diff = h2 @ w3.reshape(-1) + q["b3"].reshape(-1)[0] - t
    dy = 2.0 * diff / t.size
    dz2 = np.where(h2 > 0, dy[:, None] * w3.reshape(1, -1), 0.0)
    dz2b = bf16(dz2)
    dz1 = np.where(h1 > 0, dz2b @ w2, 0.0)
    return float(np.mean(diff ** 2)), {"w1": dz1.T @ xb, "b1": dz1.sum(0), "w2": dz2b.T @ h1, "b2": dz2.sum(0),
                                       "w3": dy @ h2, "b3": dy.sum()}


@pytest.mark.parametrize("batch", [1, 15, 16, 17, 63, 64, 65, 129, 70001])
def test_gradient_at_round_sizes(mc, batch):
    # against the reference on the same BF16 operands; 2e-2 in norm per block as for the FP64 one
    rng = np.random.default_rng(batch)
    p = O.mlp_init(11)
    for k in ("b1", "b2", "b3"):
        p[k] = rng.normal(0, 0.1, size=p[k].shape).astype(np.float32)
    x = rng.normal(0, 1, size=(500, 8)).astype(np.float32)
    t = rng.normal(0, 1, size=500).astype(np.float32)
    idx = rng.integers(0, 500, size=batch).astype(np.int32)
    print(f"[gpu] mlp gradient batch={batch}", flush=True)
    net = mc.Mlp()
    net.set_params(flat(p))
    g, loss = net.gradient(*(torch.from_numpy(a).cuda() for a in (x, t, idx)))
    rl, rg = reference(p, x[idx], t[idx])
    assert abs(loss - rl) <= 1e-2 * rl + 1e-6
    o = 0
    for k, shape in O.MLP_SHAPES:
        size = int(np.prod(shape))
        ref = np.asarray(rg[k]).reshape(-1)
        assert np.linalg.norm(g[o:o + size] - ref) <= 2e-2 * np.linalg.norm(ref) + 1e-6, k
        o += size


def test_training_reruns_are_bit_identical(mc):
    rng = np.random.default_rng(1)
    x = torch.from_numpy(rng.normal(0, 1, size=(3000, 8)).astype(np.float32)).cuda()
    t = torch.from_numpy(rng.normal(0, 1, size=3000).astype(np.float32)).cuda()
    got = []
    for _ in range(2):
        net = mc.Mlp()
        net.set_params(flat(O.mlp_init(2)))
        net.fit_normalization(x)
        losses = net.train(x, t, steps=40, batch=1000, lr=3e-3, seed=4)
        got.append((losses, net.get_params()["params"]))
    assert np.array_equal(got[0][0], got[1][0]) and np.array_equal(got[0][1], got[1][1])


@pytest.mark.parametrize("n", [1, 2, 255, 256, 257, 32769, 100003])
def test_feature_statistics(mc, n):
    rng = np.random.default_rng(n)
    x = (rng.normal(0, 1, size=(n, 8)) * 10.0 ** rng.uniform(-2, 2, size=8)).astype(np.float32)
    x[:, 6] = 1.0  # a constant column
    net = mc.Mlp()
    net.fit_normalization(torch.from_numpy(x).cuda())
    norm = net.get_params()["norm"].astype(np.float64)
    xd = x.astype(np.float64)
    mean, var = xd.mean(axis=0), xd.var(axis=0)
    std = np.where(var > 1e-12, np.sqrt(var), 1.0)
    # sums of n FP64 terms, then one rounding to binary32; the variance loses mean^2 / var of FP64
    assert np.all(np.abs(norm[:8] - mean) <= 2.0 ** -23 * np.abs(mean) + 1e-12 * np.abs(xd).max(axis=0))
    assert np.all(np.abs(norm[8:] * std - 1.0) <= 2.0 ** -22 + 1e-13 * n * (1.0 + mean ** 2 / np.maximum(var, 1e-12)))
