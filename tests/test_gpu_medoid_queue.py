"""GPU parity of the medoid queue (descending density, ties by ascending id) at the sizes where its sort changes shape."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def densities(kind, H, N):
    rng = np.random.default_rng(N)
    if kind == "equal":
        return np.full((H, N), N // 3, np.int64)
    if kind == "few":
        return rng.integers(0, 3, (H, N)) * (N // 2)                     # 0 and N among them for even N
    if kind == "extremes":
        return rng.integers(0, 2, (H, N)) * N
    return rng.integers(0, N + 1, (H, N))


def counts_with(rho, N):
    """C whose row i has rho[i] ones: with a radius that one co-activation reaches, that is its density."""
    return (torch.arange(N, device="cuda")[None, None] < torch.from_numpy(rho).cuda()[..., None]).int().contiguous()


# single wave, whole and partial steps of 1024 threads, the largest single-workgroup sort, the first of several workgroups with two
# digits, their partial last one
@pytest.mark.parametrize("N", [1, 2, 63, 64, 65, 127, 128, 1023, 1024, 1025, 2048, 2049, 4096, 4097, 8191, 8192, 8193, 10241])
@pytest.mark.parametrize("kind", ["equal", "few", "extremes", "any"])
def test_queue_order(N, kind):
    from paper_2603_17803_amd import binding
    sw = binding.Swarm(0)
    H = 2
    rho = densities(kind, H, N)
    C = counts_with(rho, N)
    total = torch.full((H,), 4, dtype=torch.int64, device="cuda")
    got, queue, _ = sw.coact_density(C, 0.75, totals_in=total)               # d = 1 - 1/4 <= 0.75
    assert np.array_equal(got.cpu().numpy(), rho)
    assert np.array_equal(queue.cpu().numpy(), np.argsort(-rho, axis=1, kind="stable"))
    assert sw.last_way()[1] == (binding.SWARM_WAY_QUEUE_LDS if N <= 8192 else binding.SWARM_WAY_QUEUE_SORTED)
    assert sw.last_way()[2] == (0 if N <= 8192 else 4 * (H * N + H * ((N + 2047) // 2048) * 512))      # as the header says
    sw.close()


@pytest.mark.parametrize("first_N", [0, 8192, 8300])
def test_recorded_first_call_needs_no_scratch(first_N):
    """The queue of more than 8192 entries is sorted with scratch; a recording that finds none compares instead."""
    from paper_2603_17803_amd import binding
    N = 8193
    sw = binding.Swarm(0, stream=torch.cuda.Stream())
    out = [torch.empty(1, N, dtype=torch.int32, device="cuda"), torch.empty(1, N, dtype=torch.int32, device="cuda"), torch.empty(1, dtype=torch.int64, device="cuda")]
    total = torch.full((1,), 4, dtype=torch.int64, device="cuda")
    C = counts_with(densities("any", 1, N), N)
    if first_N:
        C0 = counts_with(densities("any", 1, first_N), first_N)
        torch.cuda.synchronize()
        sw.coact_density(C0, 0.75, totals_in=total)
    torch.cuda.synchronize()
    sw.capture_begin()
    sw.coact_density(C, 0.75, totals_in=total, out=tuple(out))
    graph = sw.capture_end()
    assert sw.last_way()[1] == (binding.SWARM_WAY_QUEUE_SORTED if first_N > 8192 else binding.SWARM_WAY_QUEUE_COMPARED)
    for kind in ("few", "any", "equal"):
        rho = densities(kind, 1, N)
        C.copy_(counts_with(rho, N))
        out[1].fill_(-1)
        torch.cuda.synchronize()
        sw.graph_launch(graph)
        sw.stream.synchronize()
        assert np.array_equal(out[1].cpu().numpy(), np.argsort(-rho, axis=1, kind="stable"))
    binding.swarm_graph_destroy(graph)
    sw.close()
