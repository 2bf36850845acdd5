"""GPU parity of the request mapping where a list of 64 to 95 clusters is divided because its replicas look paired."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("D", [2, 4, 6, 8, 12, 32, 64])
@pytest.mark.parametrize("items", [63, 64, 65, 75, 76, 80, 95, 96, 97])
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


# each bound lies between the ratio before the rule was narrowed (1.28, 2.05; 1.08, 1.10) and since (0.99 to 1.0)
@pytest.mark.parametrize("D,items,Nc,bound", [(36, 75, 128, 1.15), (64, 75, 128, 1.15), (4, 64, 1024, 1.05), (8, 64, 1024, 1.05)])
def test_paired_replicas_are_no_slower(D, items, Nc, bound):
    """A list of clusters whose replicas stand half the SSDs apart, against the same list with the second replica one SSD further on, which is one
    chain: what finding more than 16 sub-problems costs is more than their chains save (64 SSDs 45 and 22 us), and so is finding a few of 64
    clusters, which a wave takes in one pass (8 SSDs, 1024 clusters 8.5 and 7.2 us)."""
    from paper_2603_17803_amd import binding
    sw = binding.Swarm(0)
    H, N = 8, Nc
    e2c = torch.arange(N, dtype=torch.int32, device="cuda").expand(H, N).contiguous()
    sel = torch.stack([torch.randperm(N, device="cuda")[torch.arange(120, device="cuda") % items] for _ in range(H)]).int()      # 120 picks
    first = torch.arange(H * Nc, dtype=torch.int32, device="cuda") % D
    tables = [torch.stack([first, (first + D // 2 + i) % D], 1).int().contiguous() for i in range(2)]
    out = sw.map_requests(sel, H, N, e2c, Nc, tables[0], D, None, None)
    best = [float("inf")] * 2
    for rep in range(9):
        for i in range(2):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            torch.cuda.synchronize()
            a.record()
            for _ in range(40):
                sw.map_requests(sel, H, N, e2c, Nc, tables[i], D, None, None, out=out)
            b.record()
            b.synchronize()
            if rep:
                best[i] = min(best[i], a.elapsed_time(b) / 40)
    sw.close()
    assert best[0] < bound * best[1], best
