"""GPU parity of the request mapping where a list of 64 to 95 clusters is divided because its replicas look paired."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("D", [2, 4, 6, 8, 12, 32, 64])
@pytest.mark.parametrize("items", [63, 64, 65, 80, 95, 96, 97])
@pytest.mark.parametrize("kind", ["paired", "unused second slots", "paired where it is looked at", "heavy"])
def test_queues_of_paired_replicas(D, items, kind):
    from paper_2603_17803_amd import binding
    sw = binding.Swarm(0)
    rng = np.random.default_rng(D * 1000 + items)
    H, Nc, N = 3, 257, 600
    e2c = np.stack([np.concatenate([rng.permutation(Nc), rng.integers(0, Nc, N - Nc)]) for _ in range(H)]).astype(np.int32)
    sel = np.stack([np.concatenate([np.arange(items), rng.integers(0, items, 140 - items)]) for _ in range(H)]).astype(np.int32)   # cluster of entry i < Nc: all distinct
    first = rng.integers(0, D, H * Nc)
    rep = np.stack([first, (first + D // 2) % D], 1).astype(np.int32)
    if kind == "unused second slots":
        rep[rng.random(H * Nc) < 0.5, 1] = -1
    if kind == "paired where it is looked at":
        seen = np.zeros(Nc, bool)
        seen[np.arange(64) * Nc >> 6] = True
        other = np.tile(~seen, H)
        rep[other, 1] = (rep[other, 0] + rng.integers(1, D, int(other.sum()))) % D      # any other SSD
    weight = rng.integers(0, 1 << 21 if kind == "heavy" else 50, H * Nc).astype(np.int32)
    got = sw.map_requests(torch.from_numpy(sel).cuda(), H, N, torch.from_numpy(e2c).cuda(), Nc, torch.from_numpy(rep).cuda(), D, torch.from_numpy(weight).cuda(), None)
    ref = oracle.map_requests(sel, H, N, e2c, Nc, rep, D, weight, None, None, nthreads=4)
    torch.cuda.synchronize()
    for g, r in zip(got, ref):
        assert np.array_equal(g.cpu().numpy(), r)
    sw.close()
