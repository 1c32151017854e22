"""How a BiCGstab solve ends: iteration limits, a converged start, a half step that
converges, breakdowns, sizes around a workgroup, and reruns."""
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


def reference(A, b, x, rtol, maxiter):
    """(x, iterations, converged, ||r|| / ||b||) of the textbook recurrence in numpy."""
    bn = np.linalg.norm(b)
    r = b - A @ x
    rhat, rr = r.copy(), r @ r
    if bn == 0:
        return np.zeros_like(b), 0, True, 0.0
    if np.sqrt(rr) <= rtol * bn:
        return x, 0, True, np.sqrt(rr) / bn
    rho_prev = alpha = omega = 1.0
    p, v = np.zeros_like(b), np.zeros_like(b)
    for it in range(1, maxiter + 1):
        rho = rhat @ r
        if rho == 0:
            return x, it, False, np.sqrt(rr) / bn
        beta = 0.0 if it == 1 else (rho / rho_prev) * (alpha / omega)
        p = r + beta * (p - omega * v)
        v = A @ p
        rv = rhat @ v
        if rv == 0:
            return x, it, False, np.sqrt(rr) / bn
        alpha = rho / rv
        s = r - alpha * v
        ss = s @ s
        if np.sqrt(ss) <= rtol * bn:
            return x + alpha * p, it, True, np.sqrt(ss) / bn
        t = A @ s
        tt = t @ t
        if tt == 0:
            return x, it, False, np.sqrt(rr) / bn
        omega = (t @ s) / tt
        x = x + alpha * p + omega * s
        r = s - omega * t
        rr = r @ r
        if np.sqrt(rr) <= rtol * bn:
            return x, it, True, np.sqrt(rr) / bn
        if omega == 0:
            return x, it, False, np.sqrt(rr) / bn
        rho_prev = rho
    return x, maxiter, False, np.sqrt(rr) / bn


def check(mc, B, b, x0, rtol, maxiter):
    print(f"[gpu] bicgstab ends n={B.n} rtol={rtol} maxiter={maxiter}", flush=True)
    x, st = mc.bicgstab(mc.DeviceCsr.from_host(B), None, torch.from_numpy(b).cuda(),
                        x0=None if x0 is None else torch.from_numpy(x0).cuda(), rtol=rtol, maxiter=maxiter)
    rx, it, conv, res = reference(B.to_scipy(), b, np.zeros(B.n) if x0 is None else x0, rtol, maxiter)
    assert st.iterations == it and bool(st.converged) == conv
    assert abs(st.rel_residual - res) <= 1e-6 * res + 1e-14
    assert np.linalg.norm(x.cpu().numpy() - rx) <= 1e-9 * np.linalg.norm(rx) + 1e-14
    return st


@pytest.mark.parametrize("maxiter", [1, 2, 3, 4, 5, 9])
def test_iteration_limit(mc, maxiter):
    B = I.grid2d_5pt(31, 17, diag=4.1)
    check(mc, B, np.random.default_rng(1).normal(size=B.n), None, 1e-12, maxiter)


@pytest.mark.parametrize("n", [1, 2, 255, 256, 257, 1000])
def test_sizes_around_a_workgroup(mc, n):
    # Rounding decides the 30 or so iterations that the larger ones take (a renumbering of
    # the rows moves numpy's own count by up to 6), so the end is checked against b - B x: the
    # recurrence's residual leaves it by rounding only, 50 iterations of some 1e-16 ||x_i||.
    B = I.dense_small(2, 0.4, 1) if n == 2 else I.diag_only(1, 3) if n == 1 else I.random_nonsym(n, kmin=2, kmax=4)
    b = np.random.default_rng(n).normal(size=B.n)
    print(f"[gpu] bicgstab ends n={n}", flush=True)
    x, st = mc.bicgstab(mc.DeviceCsr.from_host(B), None, torch.from_numpy(b).cuda(), rtol=1e-6, maxiter=50)
    res = np.linalg.norm(b - B.to_scipy() @ x.cpu().numpy()) / np.linalg.norm(b)
    assert st.converged and st.rel_residual <= 1e-6 and 1 <= st.iterations <= 50
    assert abs(st.rel_residual - res) <= 1e-10


def test_more_rows_than_the_dot_grid_covers_once(mc):
    B = I.grid2d_5pt(701, 613)  # 429713 > 1024 x 256
    check(mc, B, np.random.default_rng(2).normal(size=B.n), None, 1e-5, 60)


def test_converged_start_and_half_step(mc):
    B = I.grid2d_5pt(20, 20)
    x = np.random.default_rng(3).normal(size=B.n)
    b = B.to_scipy() @ x
    assert check(mc, B, b, x, 1e-8, 10).iterations == 0
    # B = 3 I: the first half step is exact
    n = 300
    D = I.from_coo(n, np.arange(n), np.arange(n), np.full(n, 4.0))
    assert check(mc, D, np.ones(n), None, 1e-10, 10).iterations == 1


def test_breakdown_of_the_first_product(mc):
    # rhat . B r = 0 in the first iteration: skew part only along r
    B = I.from_coo(2, np.array([0, 0, 1, 1]), np.array([0, 1, 0, 1]), np.array([1.0, 1.0, -1.0, -1.0]))
    st = check(mc, B, np.array([1.0, 1.0]), None, 1e-10, 5)
    assert st.iterations == 1 and not st.converged


def test_zero_right_side_after_other_solves(mc):
    B = I.grid2d_5pt(40, 9)
    for b in (np.ones(B.n), np.zeros(B.n), np.ones(B.n)):
        check(mc, B, b, np.full(B.n, 0.5), 1e-9, 40)
