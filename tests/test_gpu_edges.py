"""Device parity at the edges of the kernels' tiles, vectors and dispatch rules: small shapes just below, at and above
them, against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2603_17803_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def sw():
    from paper_2603_17803_amd import binding
    s = binding.Swarm(0)
    yield s
    s.close()


def dev(a):
    a = np.ascontiguousarray(a)
    return torch.from_numpy(a.view(np.int16) if a.dtype == np.uint16 else a).cuda()


@pytest.mark.parametrize("N", [1, 2, 3, 5, 63, 65, 66, 67, 127, 129, 130, 131, 191, 193, 254, 255, 257, 319, 387])
def test_counts_of_ragged_matrices(sw, N):
    """Rows of C that are not multiples of 16 bytes, tiles that end inside a vector: all three update forms, the density
    of a fresh build, and nothing written past the matrix."""
    H, k, rows = 2, max(1, N // 5), 67
    idx = W.random_selections(rows, H, k, N, seed=N)
    flat = torch.full((H * N * N + 64,), -12345, dtype=torch.int32, device="cuda")
    Cd = flat[:H * N * N].view(H, N, N)
    sw.coact_accumulate(dev(idx), N, Cd, decay_q16=0)
    ref = oracle.coact_update(idx, N, nthreads=4)
    assert np.array_equal(Cd.cpu().numpy(), ref)
    more = W.random_selections(29, H, k, N, seed=N + 1)
    for decay in (65536, 64881):
        sw.coact_accumulate(dev(more), N, Cd, decay_q16=decay)
        oracle.coact_update(more, N, ref, decay, nthreads=4)
        assert np.array_equal(Cd.cpu().numpy(), ref)
    total = rows * k * k
    for tau in (1.0 - 3.0 / total, 1.0 - 0.3 / k):
        rho, queue, tot = sw.coact_build_density(dev(idx), N, Cd, tau)
        r = oracle.density(Cd.cpu().numpy(), tau, 0, nthreads=4)
        for g, e in zip((rho, queue, tot), r):
            assert np.array_equal(g.cpu().numpy(), e)
        rho, queue, tot = sw.coact_density(Cd, tau)
        for g, e in zip((rho, queue, tot), r):
            assert np.array_equal(g.cpu().numpy(), e)
    assert (flat[H * N * N:] == -12345).all()
    assert sw.device_status() == 0
