"""Performance cases of the Monte Carlo sparse approximate inverse.

Each case is one pass through the public entry points of ``mcmi`` as a program
calls them: building sampling records, walking, applying or solving with M,
replaying a captured plan, and the learned chain allocation (targets, training,
allocation). Matrices come from ``inputs`` with the sizes and options of the
repository's benchmark workloads, its tests and their neighbourhood.

A case is a dict of plain values with a "kind":

* "step"    - records + walk + one product y = M x, M handed over to the program's
              own buffers (sized once; entries past nnz(M) stay as they were)
* "batched" - the same over many small matrices in one record set
* "plan"    - replay of a captured plan, M read back to the host
* "solve"   - BiCGstab with or without M as right preconditioner
* "targets" - training targets of the allocation network: records, row features,
              pilot variance, regression target
* "train"   - the allocation network's training from fresh parameters
* "learned" - features, inference, chain costs, allocation, walk with per-row chains
"""
import math

import numpy as np
import torch

from paper_2409_03095_amd import inputs, learned, mcmi

EPS, DELTA = 1e-3, 1e-4


def listed():
    return [
        # the benchmark's default step: 3D 27-point anisotropic diffusion, 4.1M rows
        dict(name="step_aniso27_160", kind="step", matrix="aniso27", nx=160, chains=64, prec=32, cell=4096),
        # the benchmark's second workload: no locality, workgroup-per-row kernel
        dict(name="step_random_262144", kind="step", matrix="random", n=262144, chains=512, prec=32, cell=0),
        # binary64 walks on a ragged mid-size stencil
        dict(name="step_aniso27_77_f64", kind="step", matrix="aniso27", nx=77, chains=64, prec=64, cell=4096),
        # the smallest whole call: 2D 5-point 32 x 32, many chains, binary64
        dict(name="step_grid2d_32_f64", kind="step", matrix="grid2d", nx=32, ny=32, chains=2000, prec=64, cell=0,
             delta=1e-3),
        # a matrix that is not contractive: augmented splitting, reduction, top-k retention
        dict(name="step_prepass_topk_64", kind="step", matrix="aniso27", nx=64, rho=1.3, chains=32, prec=32, cell=0,
             delta=1e-3, alpha=1.0, drop=0.06, topk=32),
        # a batch of small convection-diffusion systems in one launch
        dict(name="batched_convdiff_48", kind="batched", count=48, nmin=1000, nmax=100000, chains=128, prec=32),
        # time stepping on a small grid: the captured plan replayed per step
        dict(name="plan_family_33x31", kind="plan", nx=33, ny=31, chains=64, prec=32),
        # the solver with the approximate inverse as preconditioner
        dict(name="solve_aniso27_64_M", kind="solve", matrix="aniso27", nx=64, rho=0.95, chains=32, precond=True,
             topk=32),
        # a small plain solve, where launches and latency count
        dict(name="solve_grid2d_100x77", kind="solve", matrix="grid2d", nx=100, ny=77, diag=4.2, precond=False),
        # training data of the allocation network from a family of small grids
        dict(name="targets_family_200", kind="targets", mats=200, pilot=64, prec=64),
        # training of the allocation network
        dict(name="train_200k_200", kind="train", rows=200000, steps=200, batch=4096),
        # the learned allocation on a grid of the size of the held-out instance
        dict(name="learned_family_1024", kind="learned", nx=1024, ny=1024, mean=12, prec=32),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "batched", "plan", "solve", "solve", "targets", "train", "learned"])
    prec = rng.choice([32, 32, 64])
    if kind == "step":
        matrix = rng.choice(["aniso27", "aniso27", "random", "grid2d"])
        c = dict(kind=kind, matrix=matrix, prec=prec, cell=0, delta=rng.choice([1e-4, 1e-3]))
        if matrix == "aniso27":
            c.update(nx=_log_int(rng, 12, 110), chains=rng.choice([24, 64, 64, 100]), cell=rng.choice([0, 4096]))
            if rng.random() < 0.3:
                c.update(rho=1.3, alpha=1.0, drop=rng.choice([0.0, 0.02, 0.06]), topk=rng.choice([0, 16, 32]))
        elif matrix == "random":
            c.update(n=_log_int(rng, 1500, 150000), chains=rng.choice([64, 256, 512]))
        else:
            c.update(nx=_log_int(rng, 20, 300), ny=_log_int(rng, 20, 300), chains=rng.choice([64, 300, 1000]))
        return c
    if kind == "batched":
        return dict(kind=kind, count=_log_int(rng, 5, 40), nmin=1000, nmax=_log_int(rng, 5000, 80000),
                    chains=rng.choice([48, 64, 128]), prec=prec)
    if kind == "plan":
        return dict(kind=kind, nx=_log_int(rng, 20, 200), ny=_log_int(rng, 20, 200), chains=rng.choice([16, 64, 100]),
                    prec=prec)
    if kind == "solve":
        if rng.random() < 0.5:
            return dict(kind=kind, matrix="grid2d", nx=_log_int(rng, 30, 600), ny=_log_int(rng, 30, 600), diag=4.2,
                        precond=False)
        return dict(kind=kind, matrix="aniso27", nx=_log_int(rng, 20, 80), rho=rng.choice([0.75, 0.95]), chains=32,
                    precond=rng.random() < 0.7, topk=rng.choice([16, 32]))
    if kind == "targets":
        return dict(kind=kind, mats=_log_int(rng, 10, 250), pilot=rng.choice([32, 64]), prec=prec)
    if kind == "train":
        return dict(kind=kind, rows=_log_int(rng, 3000, 300000), steps=_log_int(rng, 20, 200),
                    batch=rng.choice([512, 1000, 4096]))
    return dict(kind=kind, nx=_log_int(rng, 60, 1000), ny=_log_int(rng, 60, 1000), mean=rng.choice([4, 8, 12, 20]),
                prec=prec)


# ------------------------------------------------------------------ inputs
def _host_matrix(case, seed):
    m = case["matrix"]
    if m == "aniso27":
        return inputs.aniso27(case["nx"], rho=case.get("rho", 0.75), seed=seed)
    if m == "random":
        return inputs.random_nonsym(case["n"], seed=seed)
    return inputs.grid2d_5pt(case["nx"], case["ny"], case.get("diag", 5.0), -1.0)


def _vector(n, seed):
    rng = np.random.default_rng(seed + 77)
    return torch.from_numpy(rng.uniform(-1.0, 1.0, size=n)).cuda()


def _train_set(case, seed):
    """Rows of features and targets distributed like the 5-point family's: smooth
    row sums in [0.6, 0.9], their neighbours' mean and maximum, chain length."""
    rng = np.random.default_rng(seed + 5)
    n = case["rows"]
    s = 0.75 + 0.15 * np.cos(rng.uniform(0, 2 * np.pi, n)) * np.cos(rng.uniform(0, 2 * np.pi, n))
    m = rng.choice([2, 3, 4], size=n, p=[0.004, 0.12, 0.876])
    f = np.empty((n, 8), np.float32)
    f[:, 0] = np.log(m)
    f[:, 1] = s
    f[:, 2] = s / m * rng.uniform(1.0, 1.5, n)
    f[:, 3] = s + 0.01 * rng.standard_normal(n)
    f[:, 4] = s + 0.02 * np.abs(rng.standard_normal(n))
    f[:, 5] = 3.9 - 0.2 * rng.random(n)
    f[:, 6] = 1.0
    f[:, 7] = np.minimum(66, np.log(1e-3) / np.log(s))
    y = -0.4 + 1.2 * (s - 0.75) + 0.1 * np.log(m) + 0.02 * rng.standard_normal(n)
    return torch.from_numpy(f).cuda(), torch.from_numpy(y.astype(np.float32)).cuda()


def _norm(seed):
    """Feature normalisation (mean, 1/std) of the 5-point family."""
    mean = [1.36, 0.75, 0.24, 0.75, 0.77, 3.9, 1.0, 26.0]
    inv = [12.0, 13.0, 30.0, 13.0, 13.0, 5.0, 1.0, 0.09]
    return np.array(mean + inv, np.float32)


def _family_mats(case, seed):
    """Grids of 24 to 40 points a side, the sides the same for every seed."""
    return [inputs.family_5pt(1000 * seed + 17 + k, 24 + (7 * k + 3) % 17, 24 + (11 * k + 5) % 17)
            for k in range(case["mats"])]


def _convdiff_mats(case, seed):
    """Convection-diffusion systems, sizes spread evenly over the logarithm."""
    rng = np.random.default_rng(seed)
    mats = []
    for k in range(case["count"]):
        t = k / max(case["count"] - 1, 1)
        n = case["nmin"] * (case["nmax"] / case["nmin"]) ** t
        v = rng.normal(size=3)
        v /= np.linalg.norm(v)
        mats.append(inputs.convdiff3d_7pt(int(round(n)), float(rng.uniform(0.0, 5.0)), v, float(rng.uniform(0.5, 0.85))))
    return mats


def _buffers(case, n):
    """The program's own column and value buffers, with room for every kept entry."""
    per_row = 220 if case.get("matrix") == "aniso27" and case["chains"] == 64 and not case.get("alpha") else 700
    cap = n * min(n, per_row)
    return torch.zeros(cap, dtype=torch.int32, device="cuda"), torch.zeros(cap, dtype=torch.float64, device="cuda")


def _hand_over(st, res):
    rp, col, val = res.to_torch()
    st["col"][:col.numel()].copy_(col)
    st["val"][:val.numel()].copy_(val)
    return {"row_ptr": rp, "col": st["col"], "val": st["val"]}


def prepare(case, seed):
    kind = case["kind"]
    st = {"case": case, "seed": seed}
    if kind == "step":
        B = _host_matrix(case, seed)
        st["B"] = mcmi.DeviceCsr.from_host(B)
        st["x"] = _vector(B.n, seed)
        st["col"], st["val"] = _buffers(case, B.n)
        st["p"] = mcmi.params(seed=seed, chains=case["chains"], delta=case.get("delta", DELTA), eps=EPS,
                              walk_prec=case["prec"], topk=case.get("topk", 0))
    elif kind == "batched":
        mats = _convdiff_mats(case, seed)
        st["B"] = [mcmi.DeviceCsr.from_host(m) for m in mats]
        st["col"], st["val"] = _buffers(case, sum(m.n for m in mats))
        st["p"] = mcmi.params(seed=seed, chains=case["chains"], delta=DELTA, eps=EPS, walk_prec=case["prec"])
    elif kind == "plan":
        B = inputs.family_5pt(seed, case["nx"], case["ny"])
        cdf = mcmi.Cdf(mcmi.DeviceCsr.from_host(B))
        p = mcmi.params(seed=seed, chains=case["chains"], delta=DELTA, eps=EPS, walk_prec=case["prec"])
        cap = B.n * min(B.n, 700)
        st["plan"] = mcmi.Plan(cdf, p, cap)
        st["col"], st["val"] = np.zeros(cap, np.int32), np.zeros(cap)
    elif kind == "solve":
        B = _host_matrix(case, seed)
        st["B"] = mcmi.DeviceCsr.from_host(B)
        st["b"] = _vector(B.n, seed)
        st["M"] = None
        if case["precond"]:
            st["M"] = mcmi.spai(mcmi.Cdf(st["B"]), mcmi.params(seed=seed, chains=case["chains"], delta=1e-3, eps=EPS,
                                                               walk_prec=32, topk=case["topk"]))
    elif kind == "targets":
        st["B"] = mcmi.DeviceCsr.from_host(inputs.block_diag(_family_mats(case, seed)))
    elif kind == "train":
        st["feat"], st["y"] = _train_set(case, seed)
        st["init"] = learned.init_params(seed)
        st["net"] = mcmi.Mlp()
    else:
        B = inputs.family_5pt(seed, case["nx"], case["ny"])
        st["B"] = mcmi.DeviceCsr.from_host(B)
        st["col"], st["val"] = _buffers(dict(case, chains=0), B.n)
        st["net"] = mcmi.Mlp()
        st["net"].set_params(0.5 * learned.init_params(seed), _norm(seed))
        st["p"] = mcmi.params(seed=seed, chains=1, delta=1e-3, eps=EPS, walk_prec=case["prec"])
    torch.cuda.synchronize()
    return st


def run(st):
    case, kind = st["case"], st["case"]["kind"]
    if kind == "step":
        cdf = mcmi.Cdf(st["B"], alpha=case.get("alpha", 0.0), drop_frac=case.get("drop", 0.0),
                       order_cell=case.get("cell", 0))
        res = mcmi.spai(cdf, st["p"])
        y = res.apply(st["x"])
        return {"y": y, **_hand_over(st, res)}
    if kind == "batched":
        cdf = mcmi.Cdf.batched(st["B"])
        return _hand_over(st, mcmi.spai(cdf, st["p"]))
    if kind == "plan":
        st["plan"].launch(st["seed"])
        (rp, col, val), _, _ = st["plan"].result()
        st["col"][:col.size] = col
        st["val"][:val.size] = val
        return {"row_ptr": rp, "col": st["col"], "val": st["val"]}
    if kind == "solve":
        x, _ = mcmi.bicgstab(st["B"], st["M"], st["b"])
        return {"x": x}
    if kind == "targets":
        cdf = mcmi.Cdf(st["B"])
        feat = mcmi.row_features(cdf, 1e-3)
        var, ln = mcmi.pilot_variance(cdf, mcmi.params(seed=st["seed"], delta=1e-3, walk_prec=case["prec"]),
                                      case["pilot"])
        return {"feat": feat, "var": var, "len": ln, "target": mcmi.neyman_target(var, ln)}
    if kind == "train":
        net = st["net"]
        net.set_params(st["init"])
        net.fit_normalization(st["feat"])
        losses = net.train(st["feat"], st["y"], steps=case["steps"], batch=case["batch"], lr=2e-3, seed=st["seed"])
        return {"losses": losses, "params": net.get_params()["params"], "pred": net.predict(st["feat"])}
    cdf = mcmi.Cdf(st["B"])
    feat = mcmi.row_features(cdf, 1e-3)
    pred = st["net"].predict(feat)
    cost, total = mcmi.chain_cost(feat)
    chains, lam, _ = mcmi.allocate(pred, cost, case["mean"] * total)
    res = mcmi.spai(cdf, st["p"], chains_per_row=chains)
    return {"feat": feat, "pred": pred, "chains": chains, "lambda": lam, **_hand_over(st, res)}


# ------------------------------------------------------------- least work
def work(case):
    """Input read once, output written once, and two operations per transition (a
    weight product and a sum), per matrix entry of a product, or per network weight."""
    kind = case["kind"]
    d = case.get("delta", DELTA)
    if kind in ("step", "solve"):
        if case["matrix"] == "aniso27":
            n, per, kept, rho = case["nx"] ** 3, 27, 165, case.get("rho", 0.75)
        elif case["matrix"] == "random":
            n, per, kept, rho = case["n"], 18.5, 188, 0.7
        else:
            n, per, rho = case["nx"] * case["ny"], 5, 4.0 / case.get("diag", 5.0)
            kept = 90
        if case.get("alpha"):
            rho = 0.57
        if case.get("topk"):
            kept = min(kept, case["topk"])
        steps = math.ceil(math.log(d) / math.log(rho))
        if kind == "step":
            return {"bytes": n * (per * 12 + kept * 12 + 32), "flops": 2.0 * n * case["chains"] * steps + 2.0 * n * kept}
        nnz = n * (per + (kept if case["precond"] else 0))
        return {"bytes": nnz * 12 + n * 24, "flops": 4.0 * 8 * nnz}
    if kind == "batched":
        n = case["count"] * (case["nmax"] - case["nmin"]) / math.log(case["nmax"] / case["nmin"])
        return {"bytes": n * (7 * 12 + 190 * 12 + 8), "flops": 2.0 * n * case["chains"] * 24}
    if kind == "plan":
        n = case["nx"] * case["ny"]
        return {"bytes": n * (4 * 32 + 70 * 12 + 8), "flops": 2.0 * n * case["chains"] * 32}
    if kind == "targets":
        n = case["mats"] * 1024
        return {"bytes": n * (5 * 12 + 8 + 32 + 8 + 8 + 4), "flops": 4.0 * n * case["pilot"] * 24}
    if kind == "train":
        return {"bytes": case["steps"] * case["batch"] * 36.0 + case["rows"] * 36.0,
                "flops": 6.0 * 4800 * case["steps"] * case["batch"] + 2.0 * 4800 * case["rows"]}
    n = case["nx"] * case["ny"]
    return {"bytes": n * (5 * 12 + 8 + 32 + 4 + 4 + 40 * 12), "flops": 2.0 * n * case["mean"] * 24 + 2.0 * 4800 * n}


# ------------------------------------------------------- values in 64 bits
def _philox(c0, c1, c2, c3, seed):
    """Philox4x32-10 on int64 tensors that hold 32-bit words."""
    mask = 0xFFFFFFFF

    def mul(a, b):
        p0, p1 = a * (b & 0xFFFF), a * (b >> 16)
        lo = p0 + ((p1 & 0xFFFF) << 16)
        return (p1 >> 16) + (lo >> 32), lo & mask

    k0, k1 = seed & mask, (seed >> 32) & mask
    for _ in range(10):
        ha, la = mul(0xD2511F53, c0)
        hb, lb = mul(0xCD9E8D57, c2)
        c0, c1, c2, c3 = hb ^ c1 ^ k0, lb, ha ^ c3 ^ k1, la
        k0, k1 = (k0 + 0x9E3779B9) & mask, (k1 + 0xBB67AE85) & mask
    return c0, c1, c2, c3


def _alias_tables(B):
    """Per row of C = I - D^-1 B: number of entries, |C| row sum, total weight, and
    padded (threshold, column, alias column, sign, alias sign) arrays."""
    n = B.n
    width = int(np.diff(B.row_ptr).max())
    m_of, W_of, S_of = np.zeros(n, np.int64), np.zeros(n, np.int64), np.zeros(n)
    T, col, acol = (np.zeros((n, width), np.int64) for _ in range(3))
    sg, asg = np.ones((n, width)), np.ones((n, width))
    diag = np.zeros(n)
    for r in range(n):
        b, e = B.row_ptr[r], B.row_ptr[r + 1]
        cs, vs = B.col[b:e], B.val[b:e]
        d = vs[cs == r][0]
        diag[r] = d
        keep = (cs != r) & (vs != 0)
        c, v = cs[keep], -vs[keep] / d
        m = c.size
        m_of[r] = m
        if not m:
            continue
        q = 31 - max(0, int(m - 1).bit_length())
        amax = np.abs(v).max()
        w = np.maximum(1, np.floor(np.ldexp(np.abs(v) / amax, q))).astype(np.int64)
        W = int(w.sum())
        W_of[r], S_of[r] = W, math.ldexp(amax * W, -q)
        mass = [int(m * x) for x in w]
        small = [k for k in range(m) if mass[k] < W]
        large = [k for k in range(m) if mass[k] >= W]
        al = list(range(m))
        thr = list(mass)
        while small and large:
            s, g = small.pop(), large.pop()
            al[s] = g
            thr[s] = mass[s]
            mass[g] -= W - mass[s]
            thr[g] = mass[g]
            (small if mass[g] < W else large).append(g)
        for k in small + large:
            thr[k] = W
        T[r, :m], col[r, :m], acol[r, :m] = thr, c, c[al]
        sg[r, :m], asg[r, :m] = np.sign(v), np.sign(v[al])
    return diag, m_of, S_of, W_of, T, col, acol, sg, asg


def _walk64(B, seed, N, delta):
    """Dense N-estimate (n x n) of all rows by N chains each, binary64."""
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    diag, m_of, S_of, W_of, T, col, acol, sg, asg = _alias_tables(B)
    m_t, S_t, W_t, T_t, c_t, a_t, s_t, z_t = (torch.from_numpy(v).to(dev)
                                              for v in (m_of, S_of, W_of, T, col, acol, sg, asg))
    n, width = B.n, T.shape[1]
    lmax, prod = 0, 1.0
    while prod >= delta:
        prod *= float(S_of.max())
        lmax += 1
    row = torch.arange(n, device=dev).repeat_interleave(N)
    chain = torch.arange(N, device=dev).repeat(n)
    state, w = row.clone(), torch.ones(n * N, dtype=torch.float64, device=dev)
    acc = torch.zeros(n * n, dtype=torch.float64, device=dev)
    acc.index_add_(0, row * n + state, w)
    zero = torch.zeros_like(row)
    blk = None
    for j in range(lmax):
        wn = w * S_t[state]
        go = (m_t[state] > 0) & (wn.abs() >= delta)
        if not bool(go.any()):
            break
        row, chain, state, wn = row[go], chain[go], state[go], wn[go]
        blk = _philox(zero[:row.numel()] + j // 4, chain, row, zero[:row.numel()], seed) if j % 4 == 0 else \
            tuple(b[go] for b in blk)
        um = blk[j % 4] * m_t[state]
        k, f = um >> 32, um & 0xFFFFFFFF
        Ws = W_t[state]
        pos = ((f >> 16) * Ws + (((f & 0xFFFF) * Ws) >> 16)) >> 16
        at = state * width + k
        own = pos < T_t.reshape(-1)[at]
        w = wn * torch.where(own, s_t.reshape(-1)[at], z_t.reshape(-1)[at])
        state = torch.where(own, c_t.reshape(-1)[at], a_t.reshape(-1)[at])
        acc.index_add_(0, row * n + state, w)
    return acc.reshape(n, n) / N, torch.from_numpy(diag).to(dev)


def _exact_step(case, seed):
    if case.get("alpha") or case.get("topk"):
        return None
    B = _host_matrix(case, seed)
    if B.n > 3000 or B.n * case["chains"] > 4_000_000:
        return None
    Nhat, diag = _walk64(B, seed, case["chains"], case.get("delta", DELTA))
    keep = (Nhat.abs() >= EPS) & (Nhat != 0)
    keep |= torch.eye(B.n, dtype=torch.bool, device=Nhat.device)
    M = torch.where(keep, Nhat / diag[None, :], torch.zeros_like(Nhat))
    x = _vector(B.n, seed).to(M.device)
    val = torch.zeros(B.n * min(B.n, 700), dtype=torch.float64, device=M.device)
    val[:int(keep.sum())] = M[keep]
    return {"row_ptr": None, "col": None, "val": val, "y": (M * x[None, :]).sum(1)}


def _entries(B, dev):
    rows = np.repeat(np.arange(B.n), np.diff(B.row_ptr))
    off = B.col != rows
    diag = np.zeros(B.n)
    diag[rows[~off]] = B.val[~off]
    r = torch.from_numpy(rows[off]).to(dev)
    c = torch.from_numpy(B.col[off].astype(np.int64)).to(dev)
    d = torch.from_numpy(diag).to(dev)
    return r, c, torch.from_numpy(-B.val[off]).to(dev) / d[r], d


def _exact_solve(case, seed):
    """x = C x + D^-1 b iterated to rest (||C||_inf < 1)."""
    B = _host_matrix(case, seed)
    b = _vector(B.n, seed)
    r, c, v, d = _entries(B, b.device)
    x = b / d
    base = x.clone()
    for _ in range(2000):
        new = base.index_add(0, r, v * x[c])
        done = float((new - x).abs().max()) <= 1e-17 * float(new.abs().max())
        x = new
        if done:
            break
    return {"x": x}


def _exact_features(B, delta):
    r, c, v, _ = _entries(B, "cpu")
    n = B.n
    a = v.abs()
    m = torch.zeros(n, dtype=torch.float64).index_add_(0, r, torch.ones_like(a))
    S = torch.zeros(n, dtype=torch.float64).index_add_(0, r, a)
    p = a / S[r]

    def most(x):
        return torch.zeros(n, dtype=torch.float64).scatter_reduce_(0, r, x, "amax")

    lmax, prod = 0, 1.0
    while prod >= delta:
        prod *= float(S.max())
        lmax += 1
    f = torch.empty((n, 8), dtype=torch.float64)
    f[:, 0] = torch.log(m.clamp(min=1))
    f[:, 1] = S
    f[:, 2] = most(a)
    f[:, 3] = torch.zeros(n, dtype=torch.float64).index_add_(0, r, p * S[c])
    f[:, 4] = most(S[c])
    f[:, 5] = torch.zeros(n, dtype=torch.float64).index_add_(0, r, p * m[c])
    f[:, 6] = torch.zeros(n, dtype=torch.float64).index_add_(0, r, v).abs() / S
    f[:, 7] = (math.log(delta) / torch.log(S)).clamp(max=lmax)
    return f


def _exact_predict(feat, params, norm):
    p = torch.from_numpy(np.asarray(params, np.float64))
    nm = torch.from_numpy(np.asarray(norm, np.float64))
    h = (feat - nm[:8]) * nm[8:]
    h = torch.relu(h @ p[:512].reshape(64, 8).T + p[512:576])
    h = torch.relu(h @ p[576:4672].reshape(64, 64).T + p[4672:4736])
    return h @ p[4736:4800] + p[4800]


def exact(case, seed):
    kind = case["kind"]
    if kind == "step":
        return _exact_step(case, seed)
    if kind == "solve":
        return _exact_solve(case, seed)
    if kind == "targets":
        f = _exact_features(inputs.block_diag(_family_mats(case, seed)), 1e-3)
        return {"feat": f, "var": None, "len": None, "target": None}
    if kind == "learned":
        f = _exact_features(inputs.family_5pt(seed, case["nx"], case["ny"]), 1e-3)
        pred = _exact_predict(f, 0.5 * learned.init_params(seed), _norm(seed))
        return {"feat": f, "pred": pred, "chains": None, "lambda": None, "row_ptr": None, "col": None, "val": None}
    return None
