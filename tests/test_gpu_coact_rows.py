"""GPU parity of the counts of sparse traces (k <= N / 64, 6144 trace rows, 5120 entries and 2^29 counts or more, overwriting): summed row by row, against the
popcount route on the device and against the oracle; and of the forms of the dense product.  Each call's way is asserted."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

POPCOUNT = 2
DENSE, STREAMED, STAGGERED, PIECES, ROWS, BY_POPCOUNT, STAGGERED_STREAMED = range(1, 8)           # SWARM_WAY_*


@pytest.fixture(scope="module")
def sw():
    from paper_2603_17803_amd import binding
    s = binding.Swarm(0, stream=torch.cuda.Stream())
    yield s
    s.close()


def selections(kind, rows, H, k, N, seed=0):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed * 1000 + N + rows)
    if kind == "spread":                                    # ascending, one per stratum
        u = torch.rand(rows, H, k, generator=g, device="cuda", dtype=torch.float64)
        return ((torch.arange(k, device="cuda") + u) * (N / k)).long().clamp_(max=N - 1).int()
    if kind == "runs":                                      # a run of neighbours each: every entry of it in one stretch of the columns
        start = torch.randint(0, N - k + 1, (rows, H, 1), generator=g, device="cuda")
        return (start + torch.arange(k, device="cuda")).int()
    if kind == "any":                                       # any order, repeated and invalid ids
        return torch.randint(-3, N + 3, (rows, H, k), generator=g, device="cuda", dtype=torch.int32)
    if kind == "crowded":                                   # every eighth block of 64 columns: a segment has far more than its share
        block = torch.randint(0, (N + 511) // 512, (rows, H, k), generator=g, device="cuda")
        return (block * 512 + torch.randint(0, 64, (rows, H, k), generator=g, device="cuda")).clamp_(max=N - 1).int()
    if kind == "one segment":                               # blocks of 32 columns that all fall to the first segment: most ids beyond its records
        segments = next(n for n in (1, 2, 4, 8) if N <= 8192 * n)
        block = torch.arange(N // 32, device="cuda")
        turn = ((block // segments) * 0xf2ee4e45 & 0xffffffff) >> 29
        pool = block[(block + turn) % segments == 0]
        e = torch.randint(0, pool.numel() * 32, (rows, H, k), generator=g, device="cuda")
        return (pool[e // 32] * 32 + e % 32).int()
    same = torch.randperm(N, generator=g, device="cuda")[:k].sort().values      # "same": k entries in every row
    return same.expand(rows, H, k).int().contiguous()


# one, two, four and eight segments; whole and partial last blocks of columns; the fewest rows, a partial run of rows and more
# rows than the workgroup's words cover at a time; the widest selection and a single entry
@pytest.mark.parametrize("rows,H,k,N", [(6144, 21, 64, 5120), (8199, 32, 1, 4112), (17000, 32, 60, 4096), (6200, 8, 128, 8208), (6144, 1, 300, 24576),
                                        (33000, 8, 100, 8192), (6500, 1, 512, 32784)])
@pytest.mark.parametrize("kind", ["spread", "runs", "any", "crowded", "one segment", "same"])
def test_sparse_counts_equal_the_popcount_route(sw, rows, H, k, N, kind):
    sel = selections(kind, rows, H, k, N)
    with torch.cuda.stream(sw.stream):
        sw.stream.wait_stream(torch.cuda.default_stream())
        C = torch.full((H, N, N), -7, dtype=torch.int32, device="cuda")
        ref = torch.full((H, N, N), -9, dtype=torch.int32, device="cuda")
        sw.coact_accumulate(sel, N, C, decay_q16=0)
        assert sw.last_way()[0] == ROWS
        sw.coact_accumulate(sel, N, ref, decay_q16=0, flags=POPCOUNT)
        assert sw.last_way()[0] == BY_POPCOUNT
        assert torch.equal(C, ref)
        C.fill_(-7)
        tau = 1.0 - 3.0 / float(ref.sum(dtype=torch.int64) // H + 1)
        rho, queue, totals = sw.coact_build_density(sel, N, C, tau)
        assert sw.last_way()[0] == ROWS
        assert torch.equal(C, ref)
        rho2, queue2, totals2 = sw.coact_density(ref, tau)
        assert torch.equal(totals, totals2) and torch.equal(rho, rho2) and torch.equal(queue, queue2)
    sw.stream.synchronize()
    from paper_2603_17803_amd import binding
    assert sw.device_status() == (binding.SWARM_DEV_BAD_ENTRY if kind == "any" else 0)


# just inside and just outside each bound of the rule: trace rows, counts, k against N / 64, N and its alignment, few entries
@pytest.mark.parametrize("rows,H,k,N,way", [
    (6144, 21, 80, 5120, ROWS), (6143, 21, 80, 5120, STREAMED), (6144, 20, 80, 5120, STREAMED), (6144, 21, 81, 5120, STREAMED), (6144, 21, 79, 5104, STREAMED),
    (8192, 32, 32, 4096, ROWS), (8191, 32, 32, 4096, STREAMED), (8192, 32, 33, 4096, STREAMED), (16384, 32, 64, 4096, ROWS), (16383, 32, 64, 4096, STREAMED),
    (16384, 33, 31, 4080, STREAMED), (16384, 32, 64, 4112, ROWS), (16384, 32, 64, 4104, STREAMED), (65535, 8, 8, 8192, ROWS), (65536, 8, 8, 8192, STREAMED), (6144, 1, 8, 65536, ROWS), (6144, 1, 8, 65552, STREAMED)])
def test_the_way_of_a_count(sw, rows, H, k, N, way):
    sel = selections("spread", rows, H, k, N)
    torch.cuda.synchronize()
    C = torch.empty(H, N, N, dtype=torch.int32, device="cuda")
    sw.coact_accumulate(sel, N, C, decay_q16=0)
    assert sw.last_way()[0] == way
    sw.stream.synchronize()
    sw.coact_accumulate(sel[:1], N, C, decay_q16=0)                            # no update takes the sparse way
    sw.coact_accumulate(sel, N, C, decay_q16=65536)
    assert sw.last_way()[0] == DENSE
    sw.stream.synchronize()
    assert sw.device_status() == 0


# C that starts inside a 64-byte piece (the header asks for 16): only where one segment holds all columns
@pytest.mark.parametrize("H,k,N,words,way", [(8, 128, 8192, 4, ROWS), (8, 128, 8192, 12, ROWS), (3, 200, 13392, 0, ROWS), (3, 200, 13392, 4, STREAMED), (3, 200, 13392, 8, STREAMED),
                                             (3, 200, 13392, 16, ROWS), (5, 128, 10368, 20, STREAMED), (1, 384, 24576, 12, STREAMED)])
def test_the_way_follows_where_C_starts(sw, H, k, N, words, way):
    sel = selections("spread", 6144, H, k, N)
    with torch.cuda.stream(sw.stream):
        sw.stream.wait_stream(torch.cuda.default_stream())
        room = torch.full((H * N * N + 64,), -7, dtype=torch.int32, device="cuda")
        ref = torch.empty(H, N, N, dtype=torch.int32, device="cuda")
        assert room.data_ptr() % 64 == 0
        C = room[words:words + H * N * N].view(H, N, N)
        sw.coact_accumulate(sel, N, ref, decay_q16=0, flags=POPCOUNT)
        sw.coact_accumulate(sel, N, C, decay_q16=0)
        assert sw.last_way()[0] == way and torch.equal(C, ref)
        tau = 1.0 - 3.0 / (6144.0 * k * k)
        C.fill_(-7)
        got = sw.coact_build_density(sel, N, C, tau)
        assert sw.last_way()[0] == way and torch.equal(C, ref)
        assert all(torch.equal(g, w) for g, w in zip(got, sw.coact_density(ref, tau)))
        assert bool((room[:words] == -7).all()) and bool((room[words + H * N * N:] == -7).all())
    sw.stream.synchronize()
    assert sw.device_status() == 0


# one segment and several, wide and narrow selections
@pytest.mark.parametrize("rows,H,k,N", [(6144, 8, 128, 8192), (6144, 8, 8, 8192), (6151, 2, 256, 16384), (6144, 1, 1, 24576), (6144, 1, 1024, 65536), (6144, 1, 17, 65536), (6144, 1, 1, 65536)])
def test_scratch_of_a_sparse_count(rows, H, k, N):
    """What the header says of it: at most 6 bytes for each id and 300 for each row and head, beside the trace; where one segment holds
    all columns, a record's 16 bytes for eight ids and nothing for pieces that go on."""
    from paper_2603_17803_amd import binding
    sw = binding.Swarm(0)
    sel = selections("spread", rows, H, k, N)
    sw.coact_accumulate(sel, N, torch.empty(H, N, N, dtype=torch.int32, device="cuda"), decay_q16=0)
    way, _, held = sw.last_way()
    trace = H * ((N + 255) // 256 * 256) * ((rows + 511) // 512 * 512) // 8
    records = (rows + 31) // 32 * 32 * H
    assert way == ROWS
    assert held - trace <= records * (6 * k + 300) + 4096
    if N <= 8192:
        assert held - trace <= records * (k + 7) // 8 * 16 + 4096
    sw.close()


def test_sparse_counts_equal_the_oracle(sw):
    rows, H, k, N = 8198, 32, 32, 4096                       # strata of 128 entries: distinct ids, as the oracle asks
    sel = selections("spread", rows, H, k, N, seed=5)
    torch.cuda.synchronize()
    C = torch.empty(H, N, N, dtype=torch.int32, device="cuda")
    sw.coact_accumulate(sel, N, C, decay_q16=0)
    assert sw.last_way()[0] == ROWS
    sw.stream.synchronize()
    assert np.array_equal(C.cpu().numpy(), oracle.coact_update(sel.cpu().numpy(), N, nthreads=8))


@pytest.mark.parametrize("first,then,way", [("dense", "sparse", STREAMED), ("sparse", "dense", STREAMED), ("sparse", "sparse", ROWS)])
def test_recordings_take_the_way_that_has_its_room(first, then, way):
    """A recording of either kind of trace is accepted after an eager call of either kind, and every replay is right."""
    from paper_2603_17803_amd import binding
    sw = binding.Swarm(0, stream=torch.cuda.Stream())
    N, rows, H = 8192, 6144, 8
    sparse, dense = selections("spread", rows, H, 64, N, 1), selections("spread", rows, H, 200, N, 1)
    C = torch.empty(H, N, N, dtype=torch.int32, device="cuda")
    ref = torch.empty_like(C)
    torch.cuda.synchronize()
    sw.coact_accumulate(dense if first == "dense" else sparse, N, C, decay_q16=0)
    assert sw.last_way()[0] == (STREAMED if first == "dense" else ROWS)
    sel = (sparse if then == "sparse" else dense).clone()
    torch.cuda.synchronize()
    sw.capture_begin()
    sw.coact_accumulate(sel, N, C, decay_q16=0)
    graph = sw.capture_end()
    assert sw.last_way()[0] == way
    for rep in range(3):
        sel.copy_(selections("spread", rows, H, sel.shape[2], N, 10 + rep))
        torch.cuda.synchronize()
        C.fill_(-1)
        torch.cuda.synchronize()
        sw.graph_launch(graph)
        sw.coact_accumulate(sel, N, ref, decay_q16=0, flags=POPCOUNT)
        sw.stream.synchronize()
        assert torch.equal(C, ref)
    binding.swarm_graph_destroy(graph)
    sw.close()


# 1088, 1176 (ragged rows of C) and 1368 tiles, where the dense product's workgroups finish one after the other; the fewest and the most
# of them, 1026 and 1407, and 1020, 1023 and 1410 outside (N up to 256: three tiles a head)
@pytest.mark.parametrize("rows,H,k,N,way", [(130, 8, 60, 2048, STAGGERED), (70, 1, 200, 6001, STAGGERED), (300, 8, 100, 2304, STAGGERED), (40, 102, 9, 512, STREAMED),
                                            (150, 341, 9, 256, STREAMED), (150, 342, 9, 256, STAGGERED), (40, 469, 9, 255, STAGGERED), (40, 470, 9, 255, DENSE),
                                            (40, 110, 9, 304, STAGGERED_STREAMED), (5800, 400, 3, 256, STAGGERED_STREAMED), (4700, 400, 3, 256, STAGGERED),
                                            (3584, 342, 2, 64, STREAMED), (3585, 342, 2, 64, STAGGERED_STREAMED)])
def test_dense_counts_of_a_little_more_than_the_device_holds(sw, rows, H, k, N, way):
    sel = selections("any", rows, H, k, N).clamp_(0, N - 1)
    with torch.cuda.stream(sw.stream):
        sw.stream.wait_stream(torch.cuda.default_stream())
        C = torch.randint(0, 1 << 20, (H, N, N), dtype=torch.int32, device="cuda")
        ref = C.clone()
        for decay in (65536, 64881, 0):
            sw.coact_accumulate(sel, N, C, decay_q16=decay)
            assert sw.last_way()[0] == ({STREAMED: DENSE, STAGGERED_STREAMED: STAGGERED}.get(way, way) if decay else way)
            sw.coact_accumulate(sel, N, ref, decay_q16=decay, flags=POPCOUNT)
            assert torch.equal(C, ref)
        C.fill_(-7)
        rho, queue, totals = sw.coact_build_density(sel, N, C, 1.0 - 3.0 / (rows * k * k))
        assert sw.last_way()[0] == way
        assert torch.equal(C, ref)
        for got, want in zip((rho, queue, totals), sw.coact_density(ref, 1.0 - 3.0 / (rows * k * k))):
            assert torch.equal(got, want)
    sw.stream.synchronize()
    assert sw.device_status() == 0


# which C leaves past the caches: whole 64-byte pieces below and above the last-level cache and, in between, beside a long trace; rows
# that start inside a piece beside a trace of 64 MiB, and for a larger C where the contraction covers writing them twice
@pytest.mark.parametrize("rows,H,k,N,way", [(300, 4, 9, 2800, STREAMED), (300, 12, 9, 2048, DENSE), (300, 17, 9, 2048, STREAMED), (6000, 160, 5, 512, STREAMED), (2048, 160, 5, 512, DENSE),
                                            (3584, 300, 5, 301, STREAMED), (3072, 300, 5, 301, DENSE), (10240, 1, 100, 8201, STREAMED), (6144, 1, 100, 8201, DENSE),
                                            (6144, 13, 20, 3003, STREAMED), (5120, 13, 20, 3003, DENSE), (40, 9, 9, 900, STREAMED), (40, 13, 9, 900, DENSE)])
def test_which_dense_counts_are_streamed(sw, rows, H, k, N, way):
    sel = selections("any", rows, H, k, N).clamp_(0, N - 1)
    with torch.cuda.stream(sw.stream):
        sw.stream.wait_stream(torch.cuda.default_stream())
        C = torch.full((H, N, N), -7, dtype=torch.int32, device="cuda")
        ref = torch.empty_like(C)
        sw.coact_accumulate(sel, N, C, decay_q16=0)
        assert sw.last_way()[0] == way
        sw.coact_accumulate(sel, N, ref, decay_q16=0, flags=POPCOUNT)
        assert torch.equal(C, ref)
        C.fill_(-7)
        tau = 1.0 - rows * k * k / float(N * N) / (rows * k * k)
        got = sw.coact_build_density(sel, N, C, tau)
        assert sw.last_way()[0] == way and torch.equal(C, ref)
        assert all(torch.equal(g, w) for g, w in zip(got, sw.coact_density(ref, tau)))
    sw.stream.synchronize()
    assert sw.device_status() == 0


# few tiles over many trace rows: contracted in pieces (the last one shorter), with the fewest rows, ragged rows of C, two heads; one
# step of rows below, and one tile column too many
@pytest.mark.parametrize("rows,H,k,N,way", [(8192, 1, 40, 1000, PIECES), (6144, 1, 40, 1024, PIECES), (5633, 1, 40, 1024, PIECES), (5632, 1, 40, 1024, STREAMED),
                                            (12300, 2, 30, 701, PIECES), (33000, 1, 9, 260, PIECES), (11000, 1, 60, 2048, PIECES), (21300, 1, 70, 3000, PIECES),
                                            (20992, 1, 70, 3000, DENSE)])
def test_counts_of_few_tiles_in_pieces(sw, rows, H, k, N, way):
    sel = selections("any", rows, H, k, N).clamp_(0, N - 1)
    with torch.cuda.stream(sw.stream):
        sw.stream.wait_stream(torch.cuda.default_stream())
        C = torch.randint(0, 1 << 20, (H, N, N), dtype=torch.int32, device="cuda")
        ref = C.clone()
        for decay in (65536, 64881, 0):
            sw.coact_accumulate(sel, N, C, decay_q16=decay)
            assert sw.last_way()[0] == (DENSE if decay and way == STREAMED else way)
            sw.coact_accumulate(sel, N, ref, decay_q16=decay, flags=POPCOUNT)
            assert torch.equal(C, ref)
        C.fill_(-7)
        tau = 1.0 - rows * k * k / float(N * N) / (rows * k * k)             # a pair of average count is near
        rho, queue, totals = sw.coact_build_density(sel, N, C, tau)
        assert sw.last_way()[0] == way
        assert torch.equal(C, ref)
        for got, want in zip((rho, queue, totals), sw.coact_density(ref, tau)):
            assert torch.equal(got, want)
    sw.stream.synchronize()
    assert sw.device_status() == 0


def test_recorded_pieces_need_no_room():
    """A recording that finds no room for partial counts contracts each tile whole."""
    from paper_2603_17803_amd import binding
    sw = binding.Swarm(0, stream=torch.cuda.Stream())
    N, rows = 1024, 8192
    sel = selections("spread", rows, 1, 32, N, 3)
    C = torch.empty(1, N, N, dtype=torch.int32, device="cuda")
    ref = torch.empty_like(C)
    torch.cuda.synchronize()
    sw.coact_accumulate(sel, N, ref, decay_q16=0, flags=POPCOUNT)            # the trace's room
    sw.coact_accumulate(sel[:600].contiguous(), N, C, decay_q16=0)           # the tile schedule
    sw.stream.synchronize()
    sw.capture_begin()
    sw.coact_accumulate(sel, N, C, decay_q16=0)
    graph = sw.capture_end()
    assert sw.last_way()[0] == STREAMED
    for _ in range(2):
        C.fill_(-1)
        torch.cuda.synchronize()
        sw.graph_launch(graph)
        sw.stream.synchronize()
        assert torch.equal(C, ref)
    binding.swarm_graph_destroy(graph)
    sw.close()
