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


@pytest.mark.parametrize("Wn,k,N,n_new,Nc", [
    (1, 3, 40, 1, 1), (128, 7, 300, 31, 31), (129, 8, 300, 32, 33), (256, 12, 513, 33, 32), (257, 5, 700, 255, 64), (512, 16, 900, 256, 65),
    (513, 9, 900, 257, 40), (1024, 4, 600, 513, 96), (1025, 20, 1500, 300, 130), (2048, 6, 515, 17, 95),
    (3, 24001, 30000, 40, 70), (3, 24000, 30000, 70, 40)])
def test_window_edges(sw, Wn, k, N, n_new, Nc):
    """Window lengths around the kernel's register widths, entries and clusters around its runs and half waves, selections
    whose length is no multiple of four and long enough that their list is divided, not multiplied by a reciprocal."""
    H, D = 2, 5
    rng = np.random.default_rng(N + Wn)
    sel = np.stack([np.stack([np.sort(rng.choice(N, k, replace=False)) for _ in range(H)]) for _ in range(Wn)]).astype(np.int32)
    new_ids = np.stack([rng.choice(N, n_new, replace=False) for _ in range(H)]).astype(np.int32)
    med = np.stack([rng.choice(N, Nc, replace=False) for _ in range(H)]).astype(np.int32)
    primary = rng.integers(0, D, (H, Nc)).astype(np.int32)
    size = rng.integers(0, 2 ** 31 - 1, (H, Nc)).astype(np.int32)
    for tau in (1.0, 1.0 - 0.5 / Wn, 1.0 - 1.5 / Wn, 0.0, -0.5):
        got = sw.window_assign(dev(sel), N, dev(new_ids), dev(med), tau, dev(primary), dev(size), D)
        for g, e in zip(got, oracle.window_assign(sel, N, new_ids, med, tau, primary, size, D)):
            assert np.array_equal(g.cpu().numpy(), e), tau
    assert sw.device_status() == 0


@pytest.mark.parametrize("Wn,N,n_new,Nc", [
    (40, 900, 700, 1), (256, 1500, 33, 64), (300, 2500, 2000, 600), (130, 9500, 9000, 600), (700, 1200, 1100, 65), (1100, 1300, 1000, 31), (2048, 400, 17, 300)])
def test_window_membership_without_places(sw, Wn, N, n_new, Nc):
    """Membership alone, with and without the counts: new entries in shares of one to several passes, a last share that is not
    full, workgroups of either size; entries and medoids out of range count as never activated and are flagged."""
    from paper_2603_17803_amd import binding
    H, k = 2, max(1, N // 9)
    rng = np.random.default_rng(n_new + Nc)
    sel = W.random_selections(Wn, H, k, N, seed=Nc)
    new_ids = np.stack([rng.choice(N, n_new, replace=False) for _ in range(H)]).astype(np.int32)
    med = np.stack([rng.choice(N, Nc, replace=False) for _ in range(H)]).astype(np.int32)
    for tau in (1.0 - 1.5 / Wn, 1.0):
        f, member, _ = oracle.window_assign(sel, N, new_ids, med, tau)
        for counts in (True, False):
            got = sw.window_assign(dev(sel), N, dev(new_ids), dev(med), tau, want_counts=counts)
            assert np.array_equal(got[1].cpu().numpy(), member) and got[2] is None
            assert np.array_equal(got[0].cpu().numpy(), f) if counts else got[0] is None
    assert sw.device_status() == 0
    new_ids[0, -1], med[1, 0] = N, -1
    got = sw.window_assign(dev(sel), N, dev(new_ids), dev(med), 0.99)
    f = f.copy()
    f[0, -1], f[1, :, 0] = 0, 0
    assert np.array_equal(got[0].cpu().numpy(), f)
    assert np.array_equal(got[1].cpu().numpy(), 1.0 - f / Wn < 0.99)
    assert sw.device_status() == binding.SWARM_DEV_BAD_ENTRY


@pytest.mark.parametrize("n_new,Nc", [(9, 3), (300, 33)])
def test_window_places_from_negative_first_disks(sw, n_new, Nc):
    """First SSDs and sizes below zero, sums that pass zero while entries join and sums beyond 32 bits: the place is the
    remainder as C defines it, that of a negative sum negative or zero."""
    N, H, D, Wn = 400, 2, 5, 60
    rng = np.random.default_rng(Nc)
    sel = W.random_selections(Wn, H, 90, N, seed=3)
    new_ids = np.stack([rng.choice(N, n_new, replace=False) for _ in range(H)]).astype(np.int32)
    med = np.stack([rng.choice(N, Nc, replace=False) for _ in range(H)]).astype(np.int32)
    primary, size = rng.integers(-12, 3, (H, Nc)).astype(np.int32), rng.integers(-9, 3, (H, Nc)).astype(np.int32)
    primary[:, 0], size[:, 0] = -2 ** 31, -2 ** 31
    primary[0, 1], size[0, 1] = -2, 1                                     # the sum is zero for the first to join
    primary[1, 1], size[1, 1] = 2 ** 31 - 1, 2 ** 31 - 1
    for tau in (1.0, 1.0 - 2.5 / Wn):
        f, member, disk = sw.window_assign(dev(sel), N, dev(new_ids), dev(med), tau, dev(primary), dev(size), D)
        rf, rm, _ = oracle.window_assign(sel, N, new_ids, med, tau)
        assert np.array_equal(f.cpu().numpy(), rf) and np.array_equal(member.cpu().numpy(), rm)
        before = np.cumsum(rm, 1, dtype=np.int64) - rm
        place = np.fmod(primary.astype(np.int64)[:, None] + size[:, None] + before + 1, D)
        assert np.array_equal(disk.cpu().numpy(), np.where(rm == 1, place, -1))
    assert sw.device_status() == 0


def test_window_of_the_most_new_entries(sw):
    """As many new entries as a call can name: the last share ends short of 2^31, the last pass of it beyond."""
    n_new = (1 << 31) - 1
    sel = torch.tensor([[[0]], [[1]]], dtype=torch.int32, device="cuda")
    new_ids = torch.zeros((1, n_new), dtype=torch.int32, device="cuda")
    new_ids[0, -1] = 1
    _, member, _ = sw.window_assign(sel, 2, new_ids, torch.zeros((1, 1), dtype=torch.int32, device="cuda"), 0.6, want_counts=False)
    member = member.view(-1)
    assert int(member[-1]) == 0 and bool(member[:-1].all()) and sw.device_status() == 0


def test_window_of_nearly_all_of_the_most_entries(sw):
    """128 steps that each select all but one of 2^24 entries: the list of a run's ids ends 128 short of 2^31, less than what
    the trace builder steps past it.  A few seconds: each of the 2048 spans scans the whole list."""
    N, k, steps = 1 << 24, (1 << 24) - 1, 128
    sel = torch.arange(k, dtype=torch.int32, device="cuda").repeat(steps, 1).view(steps, 1, k)
    new_ids = torch.tensor([[0, 8191, 8192, N - 2, N - 1]], dtype=torch.int32, device="cuda")
    med = torch.tensor([[1, N - 1, N - 2, N // 2]], dtype=torch.int32, device="cuda")
    f, member, _ = sw.window_assign(sel, N, new_ids, med, 0.5)
    want = np.where((new_ids.cpu().numpy()[0][:, None] < k) & (med.cpu().numpy()[0][None] < k), steps, 0)
    assert np.array_equal(f.cpu().numpy()[0], want) and np.array_equal(member.cpu().numpy()[0], want == steps)
    assert sw.device_status() == 0


@pytest.mark.parametrize("rows,k,N,shift", [(130, 8, 9000, 0), (130, 8, 9000, 1), (5, 21, 8193, 2), (300, 4, 1025, 3), (640, 33, 520, 0)])
def test_trace_spans_and_alignment(sw, rows, k, N, shift):
    """Selections that start at any 4-byte address, several spans of entries per run."""
    sel = W.random_selections(rows, 1, k, N, seed=rows)
    flat = torch.zeros(sel.size + 4, dtype=torch.int32, device="cuda")
    idx = flat[shift:shift + sel.size].view(sel.shape)
    idx.copy_(dev(sel))
    Cd = torch.zeros((1, N, N), dtype=torch.int32, device="cuda")
    sw.coact_accumulate(idx, N, Cd, decay_q16=0)
    ref = oracle.coact_update(sel, N, nthreads=8)
    assert np.array_equal(Cd.cpu().numpy(), ref)
    tau = 1.0 - 2.0 / (rows * k * k)
    rho, queue, tot = sw.coact_build_density(idx, N, Cd, tau)
    assert np.array_equal(Cd.cpu().numpy(), ref) and int(tot[0]) == rows * k * k
    assert np.array_equal(rho.cpu().numpy(), oracle.density(ref, tau, 0, nthreads=8)[0])
    assert sw.device_status() == 0


@pytest.mark.parametrize("unit,d,H,G,B,N", [
    ("page", 128, 8, 4, 4, 33), ("page", 128, 1, 3, 3, 31), ("page", 128, 3, 5, 2, 64), ("page", 64, 2, 4, 1, 65), ("page", 32, 4, 2, 7, 129),
    ("token", 256, 2, 1, 2, 32), ("token", 128, 5, 1, 1, 63), ("token", 128, 2, 8, 5, 97), ("token", 64, 1, 4, 9, 127), ("token", 64, 6, 1, 4, 1),
    ("page", 128, 2, 4, 8, 1), ("token", 256, 1, 2, 12, 31), ("page", 64, 3, 5, 33, 33), ("token", 128, 2, 1, 8, 130)])
def test_grouped_and_few_stream_scores(sw, unit, d, H, G, B, N):
    """The sweep that shares a read of the keys between streams and folds grouped heads once per workgroup: partial groups of
    streams, heads that are not a power of two, rows past the last workgroup; whole sweeps and row lists with a bad id."""
    cfg = W.CONFIGS["llama8b_32k"].scaled(N=N, k=1, T=1, H=H, G=G, B=B, d=d, unit=unit, page_size=16 if unit == "page" else 1)
    K, q = W.keys(cfg), W.queries(cfg, 0, 1)[0]
    flat = torch.full((B * H * N + 64,), -7.5, dtype=torch.float32, device="cuda")
    sw.score(unit, dev(K), dev(q), G=G, out_scores=flat[:B * H * N].view(B, H, N))
    _, ref64, ab = oracle.score(unit, K, q, G)
    # fp32 sums: one rounding per addition, each below 2^-24 of the terms -- a row and the heads folded before it, or (a whole
    # sweep of rows of 128 or 256 values for eight streams and more, on the matrix cores) a row per head
    L = d * (2 if unit == "page" else 1)
    fold = (L + G) * 2.0 ** -24 * ab
    tol = L * G * 2.0 ** -24 * ab if B >= 8 and L in (128, 256) else fold
    assert (np.abs(flat[:B * H * N].view(B, H, N).cpu().numpy() - ref64) <= tol).all()
    assert (flat[B * H * N:] == -7.5).all()
    M = 45
    ids = np.random.default_rng(N).integers(0, N, (H, M)).astype(np.int32)
    ids[:, 7] = N
    _, sc = sw.score_select_indexed(unit, dev(K), dev(ids), dev(q), 1, G=G, want_scores=True)
    h = np.arange(H)[:, None]
    ok = np.arange(M) != 7
    sc = sc.cpu().numpy()
    assert (np.abs(sc - ref64[:, h, np.minimum(ids, N - 1)]) <= fold[:, h, np.minimum(ids, N - 1)])[..., ok].all()
    assert (sc[..., 7] == 0).all()
    from paper_2603_17803_amd import binding
    assert sw.device_status() == binding.SWARM_DEV_BAD_ENTRY


@pytest.mark.parametrize("Sc,Nc,most,cap", [
    (1, 1, 5, 7), (3, 33, 0, 4), (31, 64, 1, 31), (32, 1024, 16, 300), (256, 257, 9, 3000), (257, 8193, 4, 2000), (2048, 9000, 7, 20000),
    (2048, 500, 7, 1000), (2049, 9000, 7, 20000), (300, 1 << 18, 3, 1000)])
def test_expansion_edges(sw, Sc, Nc, most, cap):
    """Picks on both sides of the listed form, repeated and skipped ones, empty clusters, bitmaps of many words, truncation."""
    H, groups = 2, 4
    rng = np.random.default_rng(Sc * 7 + Nc)
    sizes = rng.integers(0, most + 1, (H, Nc))
    off = np.zeros((H, Nc + 1), np.int32)
    off[:, 1:] = np.cumsum(sizes, 1)
    E = max(1, int(off.max()))
    ent = rng.integers(0, 1 << 20, (H, E)).astype(np.int32)
    picks = rng.integers(0, Nc, (groups, Sc)).astype(np.int32)
    picks[rng.random((groups, Sc)) < 0.1] = -1
    entries, count = sw.expand_clusters(dev(picks), H, Nc, dev(off), dev(ent), cap)
    ref, ref_n = oracle.expand_clusters(picks, H, Nc, off, ent, max(cap, E))           # the oracle refuses to truncate
    assert np.array_equal(entries.cpu().numpy(), ref[:, :cap]) and np.array_equal(count.cpu().numpy(), np.minimum(ref_n, cap))
    from paper_2603_17803_amd import binding
    assert sw.device_status() == (binding.SWARM_DEV_CAP if ref_n.max() > cap else 0)


@pytest.mark.parametrize("unit,d,H,G,B,N", [
    ("token", 256, 8, 1, 6, 1024), ("token", 256, 8, 1, 6, 1025), ("page", 128, 8, 1, 2, 3072), ("page", 128, 8, 1, 2, 3073), ("token", 64, 8, 1, 9, 2731),
    ("page", 128, 4, 3, 4, 1024), ("page", 128, 4, 3, 4, 1025), ("token", 128, 3, 1, 5, 2184), ("token", 128, 3, 1, 5, 2185), ("token", 64, 2, 4, 11, 2999)])
def test_streams_apart_and_together(sw, unit, d, H, G, B, N):
    """Sweeps just short and just long enough that streams share a read of the keys, of whole heads and of row lists."""
    cfg = W.CONFIGS["llama8b_32k"].scaled(N=N, k=1, T=1, H=H, G=G, B=B, d=d, unit=unit, page_size=16 if unit == "page" else 1)
    K, q = W.keys(cfg), W.queries(cfg, 0, 1)[0]
    flat = torch.full((B * H * N + 64,), -7.5, dtype=torch.float32, device="cuda")
    sw.score(unit, dev(K), dev(q), G=G, out_scores=flat[:B * H * N].view(B, H, N))
    _, ref64, ab = oracle.score(unit, K, q, G, nthreads=8)
    tol = (d * (2 if unit == "page" else 1) + G) * 2.0 ** -24 * ab              # as above: no shape here reaches the matrix cores
    assert (np.abs(flat[:B * H * N].view(B, H, N).cpu().numpy() - ref64) <= tol).all()
    assert (flat[B * H * N:] == -7.5).all()
    bytes_per_row = B * H * d * 2 * (2 if unit == "page" else 1)
    for M in ((8 << 20) // bytes_per_row, (8 << 20) // bytes_per_row + 1):      # the last list that is read apart, the first that is not
        ids = np.random.default_rng(M).integers(0, N, (H, M)).astype(np.int32)
        _, sc = sw.score_select_indexed(unit, dev(K), dev(ids), dev(q), 1, G=G, want_scores=True)
        h = np.arange(H)[:, None]
        assert (np.abs(sc.cpu().numpy() - ref64[:, h, ids]) <= tol[:, h, ids]).all()
    assert sw.device_status() == 0


@pytest.mark.parametrize("order", [(0, 1, 2, 3), (3, 2, 1, 0)])
def test_every_many_stream_scorer_on_a_context_of_its_own(order):
    """The four forms of the scorer for many streams, two of which need more LDS than a kernel gets unasked, one after the other
    on a fresh context."""
    from paper_2603_17803_amd import binding
    s = binding.Swarm(0)
    try:
        for i in order:
            unit, d = (("page", 128), ("token", 256), ("page", 64), ("token", 128))[i]
            cfg = W.CONFIGS["llama8b_32k"].scaled(N=140, k=1, T=1, H=2, G=4, B=33, d=d, unit=unit, page_size=16 if unit == "page" else 1)
            K, q = W.keys(cfg), W.queries(cfg, 0, 1)[0]
            got = s.score(unit, dev(K), dev(q), G=4).cpu().numpy()
            _, ref64, ab = oracle.score(unit, K, q, 4)
            assert (np.abs(got - ref64) <= d * (2 if unit == "page" else 1) * 4 * 2.0 ** -24 * ab).all(), (unit, d)
        assert s.device_status() == 0
    finally:
        s.close()


def expanded(picks, H, Nc, off, ent, cap):
    """Picks out of range and clusters with unusable offsets are passed over: entries, counts and whether any was met."""
    E = ent.shape[1]
    out, count, bad = np.full((len(picks), cap), -1, np.int32), np.zeros(len(picks), np.int32), False
    for g, row in enumerate(picks):
        h = g % H
        bad |= bool(((row < -1) | (row >= Nc)).any())
        got = [np.zeros(0, np.int32)]
        for c in np.unique(row[(row >= 0) & (row < Nc)]):
            lo, hi = int(off[h, c]), int(off[h, c + 1])
            if lo < 0 or hi < lo or hi > E:
                bad = True
            else:
                got.append(ent[h, lo:hi])
        got = np.concatenate(got)[:cap]
        out[g, :len(got)], count[g] = got, len(got)
    return out, count, bad


@pytest.mark.parametrize("Sc,groups", [(1, 6), (2, 1030), (17, 6), (63, 1024), (64, 1023), (64, 1025), (64, 2049), (65, 6), (300, 6), (2048, 4), (2049, 4)])
def test_expansion_passes_over_bad_picks_and_offsets(sw, Sc, groups):
    """Picks just outside the clusters and offset pairs below zero, falling or past the end, each alone and together, in
    ascending lists and in any order, on both sides of the kernels' numbers of picks and groups."""
    from paper_2603_17803_amd import binding
    H, Nc = 2, max(40, Sc)
    rng = np.random.default_rng(Sc + groups)
    off = np.zeros((H, Nc + 1), np.int32)
    off[:, 1:] = np.cumsum(rng.integers(0, 6, (H, Nc)), 1)
    E = int(off.max())
    ent = rng.integers(0, 1 << 20, (H, E)).astype(np.int32)
    broken = off.copy()
    for h in range(H):
        broken[h, 3], broken[h, 11], broken[h, 20] = -5, off[h, 9] - 1, E + 1          # below zero; falling; past the end
    for ascending in (True, False):
        picks = rng.integers(0, Nc, (groups, Sc)).astype(np.int32)
        if ascending:
            picks = np.sort(np.stack([rng.permutation(Nc)[:Sc] for _ in range(groups)]), 1).astype(np.int32)
        foreign = picks.copy()
        foreign[rng.random(picks.shape) < 0.2] = -1
        foreign[:, -1], foreign[::2, 0] = Nc, -2
        for p in (picks, foreign):
            for o in (off, broken):
                for cap in (max(1, Sc), 7 * Sc):
                    entries, count = sw.expand_clusters(dev(p), H, Nc, dev(o), dev(ent), cap)
                    ref, n, bad = expanded(p, H, Nc, o, ent, cap)
                    assert np.array_equal(entries.cpu().numpy(), ref) and np.array_equal(count.cpu().numpy(), n)
                    flags = sw.device_status()
                    assert bool(flags & binding.SWARM_DEV_BAD_CLUSTER) == bad and not flags & ~(binding.SWARM_DEV_BAD_CLUSTER | binding.SWARM_DEV_CAP)


@pytest.mark.parametrize("N,k,Nc,R,H", [
    (1, 1, 1, 1, 1), (3, 2, 5, 2, 3), (255, 255, 33, 3, 3), (1023, 64, 341, 3, 2), (1025, 100, 1023, 2, 3), (2047, 300, 65, 1, 5), (2049, 17, 700, 3, 2),
    (4095, 512, 1365, 3, 1), (4097, 256, 1024, 4, 2), (8191, 1024, 2047, 2, 3), (8193, 200, 1024, 3, 2), (16383, 900, 1000, 2, 1), (33001, 640, 1500, 2, 2), (8300, 5, 260000, 1, 2),
    (8000, 5, 260000, 1, 2), (20000, 7, 250000, 1, 1)])
def test_one_call_step_edges(sw, N, k, Nc, R, H):
    """The one-call step against the separate calls and the oracle, with resident clusters: tables parked with and without
    room, ragged in every length, on both sides of each block size; equal scores in quantity and NaN among them."""
    rng = np.random.default_rng(N + k)
    D, d = 6, 8
    K = rng.integers(0, 7, (H, N, d)).astype(np.float32)
    K = (K.view(np.uint32) >> 16).astype(np.uint16)                       # small whole numbers: many equal scores
    K[:, rng.integers(0, N, max(1, N // 50)), 0] = 0x7FC0                 # NaN
    q = np.full((1, H, d), 0x3F80, np.uint16)
    e2c = rng.integers(0, Nc, (H, N)).astype(np.int32)
    rep = np.stack([rng.permutation(D)[:R] for _ in range(H * Nc)]).astype(np.int32)
    weight = rng.integers(0, 50, H * Nc).astype(np.int32)
    res = rng.integers(0, 2 ** 32, (H * Nc + 31) // 32, dtype=np.uint32) & rng.integers(0, 2 ** 32, (H * Nc + 31) // 32, dtype=np.uint32)
    args = (dev(e2c), Nc, dev(rep), D)
    for resident in (None, res):
        r = None if resident is None else dev(resident)
        got = sw.step("token", dev(K), dev(q[0]), k, *args, weight=dev(weight), resident=r)
        idx, sc = sw.score_select("token", dev(K), dev(q), k, want_scores=True)
        assert np.array_equal(idx.cpu().numpy(), oracle.select(sc.cpu().numpy(), k))
        got_idx = got[0].cpu().numpy().reshape(H, k)
        assert np.array_equal(got_idx, idx.cpu().numpy()[0])
        ref = oracle.map_requests(got_idx, H, N, e2c, Nc, rep, D, weight, resident, cap=min(k, Nc))
        for g, e in zip(got[2], ref):
            assert np.array_equal(g.cpu().numpy(), e)
    assert sw.device_status() == 0


@pytest.mark.parametrize("D,Nc,S,R,heavy", [
    (1, 200, 150, 1, False), (5, 97, 400, 3, False), (6, 3000, 300, 3, False), (15, 8192, 512, 4, False), (16, 4100, 700, 2, True), (17, 700, 900, 3, False),
    (40, 9000, 500, 4, False), (64, 300, 3000, 5, False), (8, 2049, 96, 1, False), (12, 130, 2048, 4, True)])
def test_mapping_of_lists_with_single_copies(sw, D, Nc, S, R, heavy):
    """Clusters with no, one and several copies side by side, in few and many sub-problems, long and short bitmaps, loads
    beyond the packed chain's range (heavy), short lists that stay one chain; queues against the oracle."""
    H, N, groups = 2, Nc + 50, 5
    rng = np.random.default_rng(D * 1000 + S)
    e2c = np.stack([rng.permutation(np.concatenate([np.arange(Nc), rng.integers(0, Nc, 50)])) for _ in range(H)]).astype(np.int32)
    rep = np.stack([rng.permutation(D)[:R] for _ in range(H * Nc)]).astype(np.int32)
    if D % 4 == 0:                                                   # families of four SSDs: independent sub-problems
        fam = rng.integers(0, D // 4, H * Nc) * 4
        rep = fam[:, None] + np.stack([rng.permutation(4)[:min(R, 4)] for _ in range(H * Nc)]).astype(np.int64)
        rep = rep.astype(np.int32)
    keep = rng.integers(1, rep.shape[1] + 1, H * Nc)
    rep[np.arange(rep.shape[1])[None] >= keep[:, None]] = -1
    rep[rng.random(H * Nc) < 0.4, 1:] = -1
    weight = (rng.integers(0, 1 << 20, H * Nc) if heavy else rng.integers(0, 300, H * Nc)).astype(np.int32)
    for s in (S, max(1, S // 8)):
        sel = rng.integers(0, N, (groups, s)).astype(np.int32)
        cap = min(s, Nc)
        got = sw.map_requests(dev(sel), H, N, dev(e2c), Nc, dev(rep), D, dev(weight), cap=cap)
        for g, e in zip(got, oracle.map_requests(sel, H, N, e2c, Nc, rep, D, weight, cap=cap)):
            assert np.array_equal(g.cpu().numpy(), e)
    assert sw.device_status() == 0


@pytest.mark.parametrize("N,Nc,S,D,top", [
    (1024, 300, 2048, 8, 4), (1023, 200, 2049, 6, 1), (700, 110, 4097, 2, 3), (513, 513, 9000, 8, 40), (2050, 640, 16500, 12, 2), (1300, 97, 2600, 4, 9),
    (3, 3, 2048, 4, 2), (1500, 180, 3000, 16, 5000000)])
def test_merged_lists_of_replica_pairs(sw, N, Nc, S, D, top):
    """More picks than entries (the entries are marked, then looked up), just beyond and short of that rule, with padding,
    foreign ids and foreign clusters among them; pairs of SSDs as sub-problems with weights small enough for ties and zeros."""
    H, groups = 2, 3
    rng = np.random.default_rng(N + S)
    e2c = rng.integers(0, Nc, (H, N)).astype(np.int32)
    first = rng.integers(0, D // 2, H * Nc)
    rep = np.stack([first, first + D // 2], 1).astype(np.int32)
    rep[rng.random(H * Nc) < 0.5] = rep[0, ::-1]                                   # many of one pair, listed the other way round
    weight = rng.integers(0, top + 1, H * Nc).astype(np.int32)
    res = rng.integers(0, 2 ** 32, (H * Nc + 31) // 32, dtype=np.uint32) & rng.integers(0, 2 ** 32, (H * Nc + 31) // 32, dtype=np.uint32)
    for bad in (False, True):
        if bad:
            e2c[rng.random((H, N)) < 0.02] = Nc
        for s in (S, 2 * N - 1):
            sel = rng.integers(0, N, (groups, s)).astype(np.int32)
            if bad:
                sel[rng.random(sel.shape) < 0.05] = -1
                sel[:, 0], sel[:, -1] = N, -7
            good = sel.copy()                                        # what of it is left when foreign ids and clusters are passed over
            for g in range(groups):
                ok = (sel[g] >= 0) & (sel[g] < N)
                good[g] = np.where(ok & (e2c[g % H][np.where(ok, sel[g], 0)] < Nc), sel[g], -1)
            cap = min(s, Nc)
            got = sw.map_requests(dev(sel), H, N, dev(e2c), Nc, dev(rep), D, dev(weight), dev(res), cap=cap)
            for g, e in zip(got, oracle.map_requests(good, H, N, np.minimum(e2c, Nc - 1), Nc, rep, D, weight, res, cap=cap)):
                assert np.array_equal(g.cpu().numpy(), e)
        assert (sw.device_status() != 0) == bad


@pytest.mark.parametrize("D,R,picks,singles", [
    (8, 2, 95, 23), (8, 2, 96, 24), (8, 3, 97, 25), (16, 2, 96, 95), (17, 2, 60, 7), (24, 1, 95, 95), (24, 3, 130, 8), (64, 2, 95, 9), (64, 1, 200, 200),
    (6, 2, 200, 100), (4, 2, 40, 23), (4, 2, 40, 24)])
def test_mapping_on_both_sides_of_the_split(sw, D, R, picks, singles):
    """Lists of just fewer and just more clusters than are divided into sub-problems, by the number of picks and by what residency
    leaves of them; just fewer and just more single copies than are placed without the chain, on both sides of 16 SSDs."""
    H, Nc = 2, 700
    rng = np.random.default_rng(D * picks + singles)
    rep = np.stack([rng.permutation(D)[:R] for _ in range(H * Nc)]).astype(np.int32)
    weight = rng.integers(0, 5, H * Nc).astype(np.int32)
    e2c = np.stack([np.arange(Nc), rng.permutation(Nc)]).astype(np.int32)
    sel = np.stack([rng.permutation(Nc)[:picks] for _ in range(4)]).astype(np.int32)
    clusters = np.stack([e2c[g % H][sel[g]] for g in range(4)])
    for g in range(2):                                               # heads 0 and 1: the first `singles` picks of groups 0 and 1
        rep[g * Nc + clusters[g][:singles], 1:] = -1
    for left in (picks, 96, 95, singles, 1, 0):                      # what is left of groups 0 and 1 after residency
        if left > picks:
            continue
        bits = np.zeros(H * Nc, bool)
        for g in range(2):
            bits[g * Nc + clusters[g][left:]] = True
        res = np.packbits(np.pad(bits, (0, -len(bits) % 32)), bitorder="little").view(np.uint32)
        for s in (sel, np.concatenate([sel, sel[:, ::-1], np.full((4, 3), -1, np.int32)], 1)):   # picks repeated, padding
            cap = min(s.shape[1], Nc)
            got = sw.map_requests(dev(s), H, Nc, dev(e2c), Nc, dev(rep), D, dev(weight), dev(res.view(np.int32)), cap=cap)
            for a, e in zip(got, oracle.map_requests(s, H, Nc, e2c, Nc, rep, D, weight, res, cap=cap)):
                assert np.array_equal(a.cpu().numpy(), e), left
        streams = np.ascontiguousarray(np.stack([sel[:2], sel[2:]], 0))                          # [B][H][k]: both streams of a head merged
        merged = np.concatenate([sel[:2], sel[2:]], 1)
        cap = min(2 * picks, Nc)
        got = sw.map_requests_streams(dev(streams), Nc, dev(e2c), Nc, dev(rep), D, dev(weight), dev(res.view(np.int32)), cap=cap)
        for a, e in zip(got, oracle.map_requests(merged, H, Nc, e2c, Nc, rep, D, weight, res, cap=cap)):
            assert np.array_equal(a.cpu().numpy(), e), left
    assert sw.device_status() == 0


@pytest.mark.parametrize("N,Nc", [(59, 64), (60, 64), (1, 1), (1024, 128), (1025, 128)])
def test_marks_of_entries_and_clusters(sw, N, Nc):
    """2048 picks of few entries and of few clusters: their byte marks on both sides of the room they share, and on both sides of
    two picks to an entry."""
    H, D, groups = 2, 4, 3
    rng = np.random.default_rng(N)
    e2c = rng.integers(0, Nc, (H, N)).astype(np.int32)
    rep = rng.integers(0, D, (H * Nc, 1)).astype(np.int32)
    for cap in sorted({min(N, Nc), (Nc + N + 3) // 8, (Nc + N + 4 + 7) // 8, (Nc + 64 + 7) // 8, (Nc + 63) // 8, Nc}):
        if cap < min(N, Nc):
            continue
        sel = rng.integers(0, N, (groups, 2048)).astype(np.int32)
        got = sw.map_requests(dev(sel), H, N, dev(e2c), Nc, dev(rep), D, cap=cap)
        for a, e in zip(got, oracle.map_requests(sel, H, N, e2c, Nc, rep, D, cap=cap)):
            assert np.array_equal(a.cpu().numpy(), e), cap
    assert sw.device_status() == 0


@pytest.mark.parametrize("cap,Nc,S,R,D", [
    (1900, 5000, 1900, 2, 8), (2048, 3000, 2047, 3, 8), (2048, 3000, 2048, 1, 12), (2048, 16000, 6000, 2, 40), (2250, 2250, 9000, 2, 6), (2600, 2600, 5000, 4, 16)])
def test_mapping_of_the_longest_lists(sw, cap, Nc, S, R, D):
    """Lists that leave little of the on-chip memory: room for the split but not for marks beside it, and room for neither."""
    H, groups, N = 2, 4, Nc
    rng = np.random.default_rng(cap + S)
    e2c = np.stack([rng.permutation(Nc) for _ in range(H)]).astype(np.int32)
    rep = np.stack([rng.permutation(D)[:R] for _ in range(H * Nc)]).astype(np.int32)
    rep[rng.random(H * Nc) < 0.5, 1:] = -1
    weight = rng.integers(0, 100, H * Nc).astype(np.int32)
    pool = np.stack([rng.permutation(N)[:cap] for _ in range(groups)])          # at most cap clusters to a group
    sel = np.take_along_axis(pool, rng.integers(0, cap, (groups, S)), 1).astype(np.int32)
    sel[:, :min(S, cap)] = pool[:, :min(S, cap)]
    for w in (weight, np.full_like(weight, 1 << 20)):
        got = sw.map_requests(dev(sel), H, N, dev(e2c), Nc, dev(rep), D, dev(w), cap=cap)
        for a, e in zip(got, oracle.map_requests(sel, H, N, e2c, Nc, rep, D, w, cap=cap)):
            assert np.array_equal(a.cpu().numpy(), e)
    assert sw.device_status() == 0
