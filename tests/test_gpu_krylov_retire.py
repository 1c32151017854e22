"""BiCGstab: numbers of iterations around those at which the host waits for the stream, solves
one after the other on one stream and from several threads."""
import threading

import numpy as np
import pytest

from paper_2409_03095_amd import inputs as I

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def system():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2409_03095_amd import mcmi as mc
    B = I.grid2d_5pt(100, 77, 4.2, -1.0)
    b = torch.from_numpy(np.random.default_rng(3).uniform(-1, 1, B.n)).cuda()
    return mc, mc.DeviceCsr.from_host(B), b


@pytest.mark.parametrize("maxiter", [1, 2, 3, 4, 5, 7, 8, 9, 11, 12, 16, 17])
def test_stops_at_the_given_iteration(system, maxiter):
    mc, B, b = system
    x, st = mc.bicgstab(B, b=b, rtol=1e-14, maxiter=maxiter)
    assert st.iterations == maxiter and not st.converged
    y, _ = mc.bicgstab(B, b=b, rtol=1e-14, maxiter=maxiter)
    assert torch.equal(x, y)  # fixed order of every sum


def test_threads_and_streams(system):
    mc, B, b = system
    ref, st = mc.bicgstab(B, b=b, rtol=1e-9)
    got = [[] for _ in range(4)]

    def solve(k):
        s = torch.cuda.Stream()
        s.wait_stream(torch.cuda.default_stream())
        with torch.cuda.stream(s):
            for _ in range(5):
                x, w = mc.bicgstab(B, b=b, rtol=1e-9, stream=s)
                got[k].append((x.cpu(), w.iterations))

    threads = [threading.Thread(target=solve, args=(k,)) for k in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for k in range(4):
        assert len(got[k]) == 5
        for x, it in got[k]:
            assert it == st.iterations and torch.equal(x, ref.cpu())
