"""GPU: a recorded call sequence (HIP graph) must give, on every replay, what the same calls give when run
eagerly -- with the inputs refreshed, other work of the same context and synchronisations in between."""
import numpy as np
import pytest

import oracle
from paper_2603_17803_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def dev(a):
    a = np.ascontiguousarray(a)
    if a.dtype == np.uint16:
        a = a.view(np.int16)
    if a.dtype == np.uint32:
        a = a.view(np.int32)
    return torch.from_numpy(a).cuda()


def test_replays_of_a_recorded_pass_equal_the_eager_calls():
    from paper_2603_17803_amd import binding
    cfg = W.CONFIGS["llama8b_32k"].scaled(T=5)
    T, H, N, k, D = cfg.T, cfg.H, cfg.N, cfg.k, cfg.D
    tau = 1.0 - 2e-5
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        sw = binding.Swarm(0, stream=stream)
        Kd = dev(W.keys(cfg))
        e2c, weight, rep = W.cluster_tables(cfg)
        e2c_d, rep_d, w_d = dev(e2c), dev(rep), dev(weight)
        cap = min(k, cfg.Nc)
        qsets = [dev(W.queries(cfg, s * T, (s + 1) * T)) for s in range(3)]          # [T][1][H*G][d] each
        q_buf = torch.empty_like(qsets[0])
        idx_all = torch.empty((T, H, k), dtype=torch.int32, device="cuda")
        q_off = torch.empty((T, H, D + 1), dtype=torch.int32, device="cuda")
        q_clu = torch.empty((T, H, cap), dtype=torch.int32, device="cuda")
        q_load = torch.empty((T, H, D), dtype=torch.int32, device="cuda")
        Cm = torch.zeros((H, N, N), dtype=torch.int32, device="cuda")
        rho = torch.empty((H, N), dtype=torch.int32, device="cuda")
        queue = torch.empty((H, N), dtype=torch.int32, device="cuda")
        totals = torch.empty((H,), dtype=torch.int64, device="cuda")
        outputs = (idx_all, q_off, q_clu, q_load, Cm, rho, queue, totals)

        def one_pass():
            for t in range(T):
                sw.step(cfg.unit, Kd, q_buf[t, 0], k, e2c_d, cfg.Nc, rep_d, D, G=cfg.G, weight=w_d, cap=cap,
                        out_idx=idx_all[t], out=(q_off[t], q_clu[t], q_load[t]))
            sw.coact_accumulate(idx_all, N, Cm, decay_q16=65536)                      # accumulates: a skipped replay shows
            sw.coact_density(Cm, tau, out=(rho, queue, totals))

        # eager: three passes with three sets of queries, C growing from zero
        eager = []
        for s in range(3):
            q_buf.copy_(qsets[s])
            one_pass()
            stream.synchronize()
            eager.append([o.clone() for o in outputs])
        assert sw.device_status() == 0
        # the eager passes are themselves right: first pass against the oracle
        idx0 = eager[0][0].cpu().numpy()
        assert np.array_equal(eager[0][4].cpu().numpy(), oracle.coact_update(idx0, N, nthreads=8))
        assert not torch.equal(eager[0][0], eager[1][0]) and not torch.equal(eager[1][5], eager[2][5])

        sw.capture_begin()
        one_pass()
        graph = sw.capture_end()
        try:
            Cm.zero_()
            other = dev(W.random_selections(700, H, k, N, seed=77))
            C_other = torch.zeros_like(Cm)
            for s in range(3):
                q_buf.copy_(qsets[s])
                sw.graph_launch(graph)
                # eager work of the same context between the replays; its longer trace outgrows the scratch
                # the recorded pass uses, which must stay valid for the next replay
                sw.coact_accumulate(other[: 100 + 300 * s], N, C_other, decay_q16=0)
                stream.synchronize()
                for name, got, want in zip(("idx", "q_off", "q_cluster", "q_load", "C", "rho", "queue", "totals"),
                                           outputs, eager[s]):
                    assert torch.equal(got, want), f"replay {s}: {name} differs from the eager pass"
            assert np.array_equal(C_other.cpu().numpy(), oracle.coact_update(other[:700].cpu().numpy(), N, nthreads=8))
            # a fourth replay after the scratch has grown
            Cm.zero_()
            q_buf.copy_(qsets[0])
            sw.graph_launch(graph)
            stream.synchronize()
            for got, want in zip(outputs, eager[0]):
                assert torch.equal(got, want)
            assert sw.device_status() == 0
        finally:
            binding.swarm_graph_destroy(graph)
            sw.close()


def test_recording_refuses_calls_that_would_allocate():
    from paper_2603_17803_amd import binding
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        sw = binding.Swarm(0, stream=stream)
        N, H, k = 512, 1, 16
        sel = dev(W.random_selections(64, H, k, N, seed=3))
        big = dev(W.random_selections(2048, H, k, N, seed=4))
        Cm = torch.zeros((H, N, N), dtype=torch.int32, device="cuda")
        sw.coact_accumulate(sel, N, Cm, decay_q16=0)
        stream.synchronize()
        want = Cm.clone()
        sw.capture_begin()
        sw.coact_accumulate(sel, N, Cm, decay_q16=0)
        with pytest.raises(binding.SwarmError) as e:
            sw.coact_accumulate(big, N, Cm, decay_q16=0)          # longer trace: scratch would have to grow
        assert e.value.code == binding.SWARM_EINVAL
        graph = sw.capture_end()
        try:
            Cm.zero_()
            sw.graph_launch(graph)
            stream.synchronize()
            assert torch.equal(Cm, want)
            assert np.array_equal(want.cpu().numpy(), oracle.coact_update(sel.cpu().numpy(), N, nthreads=4))
        finally:
            binding.swarm_graph_destroy(graph)
            sw.close()


@pytest.mark.parametrize("H,N,large,small", [(1, 1000, 32768, 20480), (8, 600, 4096, 2560), (3, 1500, 11264, 10752)])
def test_a_build_no_larger_than_an_earlier_one_can_be_recorded(H, N, large, small):
    """After a build over a long run of selections, one over a shorter run needs no more scratch, however the trace
    builder cuts the shorter run: it may be recorded at once, and replays give what the eager call gives."""
    from paper_2603_17803_amd import binding
    k, tau = 4, 1.0 - 1e-5
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        sw = binding.Swarm(0, stream=stream)
        sel = dev(W.random_selections(large, H, k, N, seed=5))
        Cm = torch.zeros((H, N, N), dtype=torch.int32, device="cuda")
        out = (torch.empty((H, N), dtype=torch.int32, device="cuda"), torch.empty((H, N), dtype=torch.int32, device="cuda"),
               torch.empty((H,), dtype=torch.int64, device="cuda"))
        sw.coact_build_density(sel, N, Cm, tau, out=out)
        stream.synchronize()
        sw.capture_begin()
        try:
            sw.coact_build_density(sel[:small], N, Cm, tau, out=out)
        finally:
            graph = sw.capture_end()
        try:
            ref = oracle.coact_update(sel[:small].cpu().numpy(), N, nthreads=8)
            want = oracle.density(ref, tau, 0, nthreads=8)
            for _ in range(2):
                Cm.fill_(-1)
                sw.coact_build_density(sel, N, torch.empty_like(Cm), tau, out=out)        # other work in between, on the same scratch
                sw.graph_launch(graph)
                stream.synchronize()
                assert np.array_equal(Cm.cpu().numpy(), ref)
                for g, e in zip(out, want):
                    assert np.array_equal(g.cpu().numpy(), e)
            assert sw.device_status() == 0
        finally:
            binding.swarm_graph_destroy(graph)
            sw.close()


@pytest.mark.parametrize("H,large,small", [
    (8, (5, 16500, 100), (4, 16500, 100)), (1, (1, 20000, 12000), (1, 20000, 1000)), (1, (1, 200000, 4000), (1, 60000, 3000)),
    (1, (1, 16385, 8192), (1, 16385, 4000)), (8, (2, 60000, 9000), (2, 40000, 1000))])
def test_a_selection_no_larger_than_an_earlier_one_can_be_recorded(H, large, small):
    """Streams, entries and winners (B, N, k): a call that selects in one stage followed by a smaller one that cuts its rows into
    slices.  The smaller one may be recorded at once; direct steps on the same shapes too."""
    from paper_2603_17803_amd import binding
    d, D, Nc = 8, 4, 50
    rng = np.random.default_rng(H)
    K = dev((rng.standard_normal((H, max(large[1], small[1]), d)).astype(np.float32).view(np.uint32) >> 16).astype(np.uint16))
    q = dev((rng.standard_normal((max(large[0], small[0]), H, d)).astype(np.float32).view(np.uint32) >> 16).astype(np.uint16))
    rep = torch.zeros((H * Nc, 1), dtype=torch.int32, device="cuda")

    def args(B, N, k):
        e2c = (torch.arange(N, device="cuda", dtype=torch.int32) % Nc).expand(H, N).contiguous()
        queues = tuple(torch.empty((H, n), dtype=torch.int32, device="cuda") for n in (D + 1, min(k, Nc), D))
        return (K[:, :N].contiguous(), q[:B].contiguous(), k, e2c, queues, torch.empty((B, H, k), dtype=torch.int32, device="cuda"),
                torch.empty((H, k), dtype=torch.int32, device="cuda"))

    def one(sw, a):
        keys, qs, k, e2c, queues, idx, step_idx = a
        sw.score_select("token", keys, qs, k, out_idx=idx)
        sw.step("token", keys, qs[0], k, e2c, Nc, rep, D, out_idx=step_idx, out=queues)
        return [idx, step_idx, *queues]

    stream = torch.cuda.Stream()
    a, b = args(*large), args(*small)
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        sw = binding.Swarm(0, stream=stream)
        one(sw, a)
        stream.synchronize()
        sw.capture_begin()
        try:
            out = one(sw, b)
        finally:
            graph = sw.capture_end()
        try:
            want = None
            for _ in range(2):
                for o in out:
                    o.fill_(-9)
                sw.graph_launch(graph)
                stream.synchronize()
                got = [o.clone() for o in out]
                want = want or [o.clone() for o in one(sw, b)]
                one(sw, a)
                stream.synchronize()
                for g, w in zip(got, want):
                    assert torch.equal(g, w)
            assert torch.equal(got[0][0], got[1]) and sw.device_status() == 0
        finally:
            binding.swarm_graph_destroy(graph)
            sw.close()


@pytest.mark.parametrize("kind", ["queue", "pieces", "sparse"])
def test_a_capture_of_the_callers_own_finds_no_scratch(kind):
    """Calls whose shorter way has scratch of its own, the first of their kind inside a graph that the caller captures by its own means (no
    swarm_capture_begin), after calls no smaller than them: they take the way that needs none.  Every replay is right, and an eager call
    afterwards takes the shorter way."""
    from paper_2603_17803_amd import binding
    stream = torch.cuda.Stream()
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    sw = binding.Swarm(0, stream=stream)
    if kind == "queue":
        N = 8200
        C = torch.randint(0, 9, (1, N, N), generator=g, device="cuda", dtype=torch.int32)
        out = (torch.empty(1, N, dtype=torch.int32, device="cuda"), torch.empty(1, N, dtype=torch.int32, device="cuda"), torch.empty(1, dtype=torch.int64, device="cuda"))
        total = torch.full((1,), 8, dtype=torch.int64, device="cuda")
        ways = (binding.SWARM_WAY_QUEUE_COMPARED, binding.SWARM_WAY_QUEUE_SORTED)

        def call():
            sw.coact_density(C, 0.5, totals_in=total, out=out)
            return sw.last_way()[1]

        def refresh():
            C.copy_(torch.randint(0, 9, (1, N, N), generator=g, device="cuda", dtype=torch.int32))
            rho = (C >= 4).sum(2)
            return [rho.int(), torch.sort(-rho, dim=1, stable=True).indices.int()]
    else:
        rows, H, k, N = (8192, 1, 16, 1024) if kind == "pieces" else (6144, 8, 64, 8192)
        wide = torch.randint(0, N, (rows, H, 4 * k), generator=g, device="cuda", dtype=torch.int32)
        sel = wide[:, :, :k].contiguous()
        C = torch.empty(H, N, N, dtype=torch.int32, device="cuda")
        ref = torch.empty_like(C)
        out = (C,)
        ways = (binding.SWARM_WAY_DENSE_STREAMED, binding.SWARM_WAY_DENSE_PIECES if kind == "pieces" else binding.SWARM_WAY_ROWS)
        torch.cuda.synchronize()
        sw.coact_accumulate(wide, N, ref, decay_q16=0, flags=2)                # the trace's room
        sw.coact_accumulate(wide[:600], N, C, decay_q16=0)                     # the tile schedule
        stream.synchronize()

        def call():
            sw.coact_accumulate(sel, N, C, decay_q16=0)
            return sw.last_way()[0]

        def refresh():
            sel.copy_(torch.randint(0, N, (rows, H, k), generator=g, device="cuda", dtype=torch.int32))
            torch.cuda.synchronize()
            sw.coact_accumulate(sel, N, ref, decay_q16=0, flags=2)
            stream.synchronize()
            return [ref]

    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        assert call() == ways[0]
    for _ in range(3):
        want = refresh()
        for o in out:
            o.fill_(-1)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(out, want))
    with torch.cuda.stream(stream):
        assert call() == ways[1]
    stream.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(out, want)) and sw.device_status() == 0
    del graph
    sw.close()


@pytest.mark.parametrize("kind", ["queue", "pieces", "sparse"])
def test_a_capture_of_the_callers_own_outlives_larger_calls(kind):
    """The same calls captured by the caller's own means once their scratch is there: the graph refers to it, so larger calls of the context
    afterwards, which outgrow it, leave it in place.  Every replay is right, with the larger calls between them."""
    from paper_2603_17803_amd import binding
    stream = torch.cuda.Stream()
    g = torch.Generator(device="cuda")
    g.manual_seed(4)
    sw = binding.Swarm(0, stream=stream)
    if kind == "queue":
        sizes = [8200, 9000, 12000]
        Cs = [torch.randint(0, 9, (1, n, n), generator=g, device="cuda", dtype=torch.int32) for n in sizes]
        outs = [(torch.empty(1, n, dtype=torch.int32, device="cuda"), torch.empty(1, n, dtype=torch.int32, device="cuda"),
                 torch.empty(1, dtype=torch.int64, device="cuda")) for n in sizes]
        total = torch.full((1,), 8, dtype=torch.int64, device="cuda")
        way = binding.SWARM_WAY_QUEUE_SORTED

        def call(i):
            sw.coact_density(Cs[i], 0.5, totals_in=total, out=outs[i])
            return sw.last_way()[1]

        def want(i):
            rho = (Cs[i] >= 4).sum(2)
            return [rho.int(), torch.sort(-rho, dim=1, stable=True).indices.int()]
    else:
        shapes = [(8192, 1, 16, 1024), (11000, 1, 16, 1024), (16384, 1, 16, 2048)] if kind == "pieces" else [(6144, 8, 64, 8192), (6200, 8, 128, 8192), (8192, 8, 128, 8192)]
        sels = [torch.randint(0, n, (rows, H, k), generator=g, device="cuda", dtype=torch.int32) for rows, H, k, n in shapes]
        outs = [(torch.empty(H, n, n, dtype=torch.int32, device="cuda"),) for _, H, _, n in shapes]
        way = binding.SWARM_WAY_DENSE_PIECES if kind == "pieces" else binding.SWARM_WAY_ROWS

        def call(i):
            sw.coact_accumulate(sels[i], shapes[i][3], outs[i][0], decay_q16=0)
            return sw.last_way()[0]

        def want(i):
            ref = torch.empty_like(outs[i][0])
            torch.cuda.synchronize()
            sw.coact_accumulate(sels[i], shapes[i][3], ref, decay_q16=0, flags=2)
            stream.synchronize()
            return [ref]

    torch.cuda.synchronize()
    expected = want(0)
    with torch.cuda.stream(stream):
        assert call(0) == way
    stream.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        assert call(0) == way
    held = sw.last_way()[2]
    for i in (0, 1, 2):
        if i:
            with torch.cuda.stream(stream):
                assert call(i) == way
            stream.synchronize()
            assert sw.last_way()[2] > held
            held = sw.last_way()[2]
            assert all(torch.equal(a, b) for a, b in zip(outs[i], want(i)))
        for o in outs[0]:
            o.fill_(-1)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(outs[0], expected))
    assert sw.device_status() == 0
    del graph
    sw.close()
