"""Performance cases of the hot path: what a serving program has this library do, through the binding's public calls.

A decode loop records one generated token's worth of calls (every layer of the model has key data of its own) and
replays the recording with refreshed inputs; background work (co-activation counts, density, cluster maintenance) is
called directly.  A case is a dict of plain values, its "kind" says which program it stands for:

  step     one decode step of one stream called directly (swarm_step), outputs in the caller's tensors
  token    one generated token of one stream: `layers` recorded decode steps, each on its layer's keys
  batch    one generated token of B streams: per layer score + select of all streams, then one merged request mapping
  count    co-activation counts of a run of selections, C = A^T A, C += A^T A or the decayed update
  refresh  a decayed update of the counts and the density pass over them (what re-clustering starts from)
  profile  counts and density of a fresh run of selections in one call
  window   cluster maintenance over the local window: membership and placement of newly generated entries
  medoid   retrieval through the medoid index, recorded per token: score + select over the medoids, expansion into
           entries, entry-level mapping, submission order

Sizes are those of the configurations in paper_2603_17803_amd/workloads.py and ragged ones around them (a context is
rarely a multiple of anything).  Inputs are topic mixtures as in that module, drawn on the GPU.
"""
import math
import sys

import torch

from paper_2603_17803_amd import binding

NOISE = 0.3                       # of keys and queries around their topic's centre
DEV = "cuda"


def listed():
    return [
        # the smallest call: one head of 4096 token keys, called directly; launches and the host path are all there is
        dict(name="step_tiny", kind="step", unit="token", H=1, N=4096, d=128, G=1, k=64, Nc=64, D=4, R=2, layers=8, resident=False),
        # a 32K context in 16-token pages with grouped query heads, ragged page count, part of the clusters in DRAM
        dict(name="token_32k_grouped", kind="token", unit="page", H=8, N=2003, d=128, G=4, k=128, Nc=256, D=8, R=2, layers=32, resident=True),
        # a 128K context in pages, one query per KV head
        dict(name="token_long_128k", kind="token", unit="page", H=8, N=8192, d=128, G=1, k=256, Nc=1024, D=8, R=3, layers=16, resident=False),
        # token-granular selection out of a 64K context
        dict(name="token_stress", kind="token", unit="token", H=1, N=65536, d=128, G=1, k=1024, Nc=2048, D=8, R=4, layers=8, resident=False),
        # a handful of streams over one shared prefix
        dict(name="batch_few", kind="batch", unit="page", H=8, N=4001, d=128, G=4, B=4, k=200, Nc=500, D=6, R=2, layers=16, resident=True),
        # many streams over one shared prefix
        dict(name="batch_drift", kind="batch", unit="page", H=8, N=2048, d=128, G=4, B=64, k=128, Nc=512, D=8, R=2, layers=16, resident=False),
        # the counts of a whole 4096-step run over a 128K context, built once
        dict(name="count_long_128k", kind="count", rows=4096, H=8, N=8192, k=256, decay=0),
        # the periodic decayed update: 256 steps of 64 streams
        dict(name="count_drift", kind="count", rows=16384, H=8, N=2048, k=128, decay=64881),
        # decayed update and density over a ragged number of entries
        dict(name="refresh_ragged", kind="refresh", rows=512, H=8, N=6001, k=192, decay=64881),
        # token-granular counts and density, the largest work
        dict(name="profile_stress", kind="profile", rows=8192, H=1, N=65536, k=1024),
        # the last 256 steps of a 128K context against 256 new entries
        dict(name="window_long_128k", kind="window", W=256, H=8, N=8192, k=256, n_new=256, Nc=1024, D=8),
        # medoid-indexed retrieval, 1024 clusters per head
        dict(name="medoid_long_128k", kind="medoid", unit="page", H=8, N=8192, d=128, G=4, k=32, Nc=1024, D=8, R=3, cap=512, layers=6),
    ]


def _log(rng, lo, hi):
    """A whole number from lo to hi, spread over its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))))


def draw(rng):
    kind = rng.choice(["step", "token", "token", "batch", "batch", "count", "count", "refresh", "profile", "window", "medoid"])
    c = dict(kind=kind)
    if kind in ("step", "token", "batch", "medoid"):
        c["unit"] = rng.choice(["page", "page", "token"])
        c["H"] = rng.choice([1, 2, 4, 8, 8, 8])
        c["d"] = rng.choice([64, 128, 128])
        c["G"] = rng.choice([1, 2, 4, 4, 8])
        c["D"] = rng.choice([4, 6, 8, 8, 12])
        c["R"] = rng.choice([1, 2, 2, 3, 4])
    if kind == "step":
        c.update(N=_log(rng, 512, 8192), layers=8, resident=rng.random() < 0.5)
    elif kind == "token":
        wide = c["H"] == 1 and c["unit"] == "token"
        c.update(N=_log(rng, 1024, 65536 if wide else 16384), layers=8, resident=rng.random() < 0.5)
    elif kind == "batch":
        c.update(N=_log(rng, 512, 8192), B=_log(rng, 2, 64), layers=8, resident=rng.random() < 0.5)
    elif kind == "medoid":
        c.update(N=_log(rng, 2048, 16384), layers=6)
    if kind in ("step", "token", "batch"):
        c["k"] = max(8, min(1024, c["N"] // rng.choice([8, 16, 32, 64])))
        c["Nc"] = max(16, min(2048, c["N"] // rng.choice([4, 8, 16])))
    elif kind == "medoid":
        size = rng.choice([8, 16])
        c["Nc"] = c["N"] // size
        c["k"] = rng.choice([16, 32, 64])
        c["cap"] = min(2048, 2 * c["k"] * size)
    elif kind in ("count", "refresh"):
        c.update(rows=_log(rng, 64, 16384 if kind == "count" else 2048), H=rng.choice([1, 4, 8]), N=_log(rng, 1024, 6144))
        c["k"] = max(16, c["N"] // rng.choice([16, 32]))
        c["decay"] = rng.choice([0, 65536, 64881]) if kind == "count" else 64881
    elif kind == "profile":
        c.update(rows=_log(rng, 256, 8192), N=_log(rng, 2048, 24576))
        c["H"] = rng.choice([1, 2, 4]) if c["N"] < 8192 else 1
        c["k"] = max(16, c["N"] // rng.choice([16, 32, 64]))
    elif kind == "window":
        c.update(W=_log(rng, 64, 1024), H=rng.choice([1, 4, 8]), N=_log(rng, 1024, 16384), n_new=_log(rng, 16, 256), D=rng.choice([4, 8, 12]))
        c["k"] = max(16, c["N"] // 32)
        c["Nc"] = max(64, c["N"] // rng.choice([8, 16]))
    return c


# ---- inputs -----------------------------------------------------------------------------------

class _Recording:
    """A recorded call sequence (a HIP graph) and what it needs kept alive."""

    def __init__(self, sw, calls):
        calls()                                          # eager once: scratch grows, nothing is allocated while recording
        sw.stream.synchronize()
        sw.capture_begin()
        self.out = calls()
        self.sw, self.calls, self.graph = sw, calls, sw.capture_end()      # the calls hold the buffers that the recording refers to

    def __call__(self):
        self.sw.graph_launch(self.graph)
        return self.out

    def __del__(self):
        if getattr(self, "graph", None) and not sys.is_finalizing():
            self.sw.stream.synchronize()
            binding.swarm_graph_destroy(self.graph)


_handles = {}


def _handle(recorded):
    """The program's library context: on its current stream for direct calls, on a stream of its own for recordings."""
    if recorded not in _handles:
        _handles[recorded] = binding.Swarm(0, stream=torch.cuda.Stream()) if recorded else binding.Swarm(0)
    return _handles[recorded]


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 7919 + 17)
    return g


def _zipf(M):
    w = 1.0 / torch.arange(1, M + 1, dtype=torch.float64, device=DEV) ** 1.1
    return (w / w.sum()).float()


def _topics(c, g):
    """Topic (= cluster) of every entry, int32 [H][N]: popular topics hold more entries."""
    return torch.multinomial(_zipf(c["Nc"]), c["H"] * c["N"], replacement=True, generator=g).view(c["H"], c["N"]).int()


def _keys(c, g, cen, topics):
    """Keys of one layer: bf16 [H][N][d], or the channel-wise min and max of 16-token pages, bf16 [H][N][2][d]."""
    H, N, d = c["H"], c["N"], c["d"]
    if c["unit"] == "token":
        return (cen.gather(1, topics.long()[..., None].expand(H, N, d)) + NOISE * torch.randn(H, N, d, generator=g, device=DEV)).bfloat16()
    out = torch.empty(H, N, 2, d, dtype=torch.bfloat16, device=DEV)
    for h in range(H):
        tok = (cen[h][topics[h].long()][:, None] + NOISE * torch.randn(N, 16, d, generator=g, device=DEV)).bfloat16()
        out[h, :, 0], out[h, :, 1] = tok.amin(1), tok.amax(1)
    return out


def _queries(c, g, cen, B):
    """bf16 [B][H*G][d]: every query head near a topic of its own."""
    H, G, d = c["H"], c["G"], c["d"]
    z = torch.randint(0, cen.shape[1], (B, H, G), generator=g, device=DEV)
    q = cen[torch.arange(H, device=DEV)[None, :, None], z] + NOISE * torch.randn(B, H, G, d, generator=g, device=DEV)
    return q.bfloat16().view(B, H * G, d)


def _replicas(c, g, sizes):
    """int32 [rows][R] and weights int32 [rows]: round-robin first copies, further copies D/R devices on."""
    D, R = c["D"], c["R"]
    first = (torch.cumsum(sizes, 0) - sizes) % D
    rep = (first[:, None] + max(1, D // R) * torch.arange(R, device=DEV)[None]) % D
    return rep.int().contiguous(), sizes.int().contiguous()


def _bitmap(c, g, n):
    """A bitmap of n bits, a quarter of them set (what is already in DRAM)."""
    bits = (torch.rand((n + 31) // 32, 32, generator=g, device=DEV) < 0.25).long()
    word = (bits << torch.arange(32, device=DEV)).sum(1)
    return torch.where(word >= 1 << 31, word - (1 << 32), word).int()


def _selections(g, rows, H, k, N, topics=256):
    """Ascending selections int32 [rows][H][k]: half of each is one of a few recurring runs of entries, half is spread."""
    topics = min(topics, N)
    run = k // 2 if N >= 2 * k else 0
    rest, span = k - run, N - run
    starts = torch.randint(0, N - run + 1, (H, topics), generator=g, device=DEV)
    out = torch.empty(rows, H, k, dtype=torch.int32, device=DEV)
    for r0 in range(0, rows, 2048):
        r = min(2048, rows - r0)
        z = torch.multinomial(_zipf(topics), r * H, replacement=True, generator=g).view(r, H)
        start = starts[torch.arange(H, device=DEV)[None], z]
        u = torch.rand(r, H, rest, generator=g, device=DEV, dtype=torch.float64)
        spread = ((torch.arange(rest, device=DEV) + u) * (span / rest)).long().clamp_(max=span - 1)     # one per stratum of at least one entry: distinct
        spread = spread + run * (spread >= start[..., None]).long()
        sel = torch.cat([start[..., None] + torch.arange(run, device=DEV), spread], -1)
        out[r0:r0 + r] = sel.sort(-1).values.int()
    return out


def prepare(case, seed):
    c, g = dict(case), _gen(seed)
    kind = c["kind"]
    s = {"case": c}
    if kind in ("step", "token", "batch"):
        H, N, k, L, Nc = c["H"], c["N"], c["k"], c["layers"], c["Nc"]
        B = c.get("B", 1)
        cen = torch.randn(H, Nc, c["d"], generator=g, device=DEV)
        e2c = _topics(c, g)
        sizes = torch.stack([torch.bincount(e2c[h].long(), minlength=Nc) for h in range(H)]).view(-1)
        rep, weight = _replicas(c, g, sizes)
        res = _bitmap(c, g, H * Nc) if c["resident"] else None
        keys = [_keys(c, g, cen, e2c) for _ in range(L)]
        qs = [_queries(c, g, cen, B) for _ in range(L)]
        cap = min(B * k, Nc)
        idx = torch.zeros(L, B, H, k, dtype=torch.int32, device=DEV)
        q_off, q_cluster, q_load = (torch.zeros(L, H, n, dtype=torch.int32, device=DEV) for n in (c["D"] + 1, cap, c["D"]))
        queues = [(q_off[t], q_cluster[t], q_load[t]) for t in range(L)]
        sw = _handle(kind != "step")
        if kind == "step":
            s.update(sw=sw, keys=keys, q=[q[0] for q in qs], e2c=e2c, rep=rep, weight=weight, res=res, idx=idx[0, 0], queues=queues[0], at=0)
        else:
            def calls():
                for t in range(L):
                    if kind == "token":
                        sw.step(c["unit"], keys[t], qs[t][0], k, e2c, Nc, rep, c["D"], G=c["G"], weight=weight, resident=res, out_idx=idx[t, 0], out=queues[t])
                    else:
                        sw.score_select(c["unit"], keys[t], qs[t], k, G=c["G"], out_idx=idx[t])
                        sw.map_requests_streams(idx[t], N, e2c, Nc, rep, c["D"], weight, res, out=queues[t])
                return [idx, q_off, q_cluster, q_load]
            torch.cuda.synchronize()
            s["token"] = _Recording(sw, calls)
    elif kind in ("count", "refresh", "profile"):
        s.update(sw=_handle(False), idx=_selections(g, c["rows"], c["H"], c["k"], c["N"]))
        s["C"] = torch.zeros(c["H"], c["N"], c["N"], dtype=torch.int32, device=DEV)
        # an entry is near another when they were activated together in an eighth of the steps in which a run recurs most
        s["tau"] = 1.0 - c["rows"] / 64.0 / (float(c["rows"]) * c["k"] ** 2)
    elif kind == "window":
        H, Nc = c["H"], c["Nc"]
        pick = lambda n: torch.rand(H, c["N"], generator=g, device=DEV).topk(n, 1).indices.int().contiguous()      # noqa: E731
        s.update(sw=_handle(False), sel=_selections(g, c["W"], H, c["k"], c["N"]), new=pick(c["n_new"]), med=pick(Nc))
        s["primary"] = torch.randint(0, c["D"], (H, Nc), generator=g, device=DEV, dtype=torch.int32)
        s["size"] = torch.randint(1, 64, (H, Nc), generator=g, device=DEV, dtype=torch.int32)
        s["tau"] = 1.0 - 8.0 / 256
    elif kind == "medoid":
        H, N, Nc, L = c["H"], c["N"], c["Nc"], c["layers"]
        cen = torch.randn(H, Nc, c["d"], generator=g, device=DEV)
        # clusters of a few entries around their medoid, sizes 1 to 2 N / Nc, every entry in one of them
        order = torch.rand(H, N, generator=g, device=DEV).argsort(1)
        cut = torch.rand(H, N - 1, generator=g, device=DEV).argsort(1)[:, :Nc - 1].sort(1).values + 1
        zero = torch.zeros(H, 1, dtype=torch.long, device=DEV)
        off = torch.cat([zero, cut, zero + N], 1)
        med = order.gather(1, off[:, :-1]).int().contiguous()
        topics = torch.empty(H, N, dtype=torch.int32, device=DEV)
        member = torch.searchsorted(off, torch.arange(N, device=DEV).expand(H, N).contiguous(), right=True) - 1
        topics.scatter_(1, order, member.int())
        rep, _ = _replicas(c, g, torch.ones(H * N, dtype=torch.long, device=DEV))
        rep[torch.rand(H * N, generator=g, device=DEV) < 0.5, 1:] = -1      # half the entries have a single copy
        keys = [_keys(c, g, cen, topics) for _ in range(L)]
        qs = [_queries(c, g, cen, 1) for _ in range(L)]
        off, ent = off.int().contiguous(), order.int().contiguous()
        ident = torch.arange(N, dtype=torch.int32, device=DEV).expand(H, N).contiguous()
        res = _bitmap(c, g, H * N)
        sw, cap = _handle(True), c["cap"]

        def calls():
            out = []
            for t in range(L):
                pos, _ = sw.score_select_indexed(c["unit"], keys[t], med, qs[t], c["k"], G=c["G"])
                entries, count = sw.expand_clusters(pos[0], H, Nc, off, ent, cap)
                q = sw.map_requests(entries, H, N, ident, N, rep, c["D"], None, res, cap=cap)
                out.append((pos, entries, count, q, sw.submission_order(q[0], q[1])))
            return out
        torch.cuda.synchronize()
        s["token"] = _Recording(sw, calls)
    torch.cuda.synchronize()
    return s


def run(s):
    c = s["case"]
    kind = c["kind"]
    if "token" in s:
        return s["token"]()
    sw = s["sw"]
    if kind == "step":
        t = s["at"]
        s["at"] = (t + 1) % c["layers"]
        sw.step(c["unit"], s["keys"][t], s["q"][t], c["k"], s["e2c"], c["Nc"], s["rep"], c["D"], G=c["G"], weight=s["weight"], resident=s["res"], out_idx=s["idx"],
                out=s["queues"])
        return [s["idx"], s["queues"]]
    if kind == "count":
        return sw.coact_accumulate(s["idx"], c["N"], s["C"], decay_q16=c["decay"])
    if kind == "refresh":
        sw.coact_accumulate(s["idx"], c["N"], s["C"], decay_q16=c["decay"])
        return [s["C"], sw.coact_density(s["C"], s["tau"])]
    if kind == "profile":
        return [s["C"], sw.coact_build_density(s["idx"], c["N"], s["C"], s["tau"])]
    return sw.window_assign(s["sel"], c["N"], s["new"], s["med"], s["tau"], s["primary"], s["size"], c["D"])


def work(case):
    """Inputs read once and outputs written once; operations of the definition (a multiply and an add per channel and
    query head of a score, one increment per pair of a selection)."""
    c = dict(case)
    kind = c["kind"]
    if kind in ("step", "token", "batch", "medoid"):
        H, G, d, B, k, D = c["H"], c["G"], c["d"], c.get("B", 1), c["k"], c["D"]
        L = d * (2 if c["unit"] == "page" else 1)
        rows = c["Nc"] if kind == "medoid" else c["N"]
        items = c["cap"] if kind == "medoid" else min(B * k, c["Nc"])
        n = H * rows * L * 2 + B * H * G * d * 2 + B * H * k * 8 + H * (items * (c["R"] + 3) + D * 2) * 4
        steps = 1 if kind == "step" else c["layers"]
        return {"bytes": steps * n, "flops": steps * 2 * B * H * G * rows * L}
    H, N, k = c["H"], c["N"], c["k"]
    if kind == "window":
        pairs = H * c["n_new"] * c["Nc"]
        return {"bytes": (c["W"] * H * k + H * (c["n_new"] + 3 * c["Nc"])) * 4 + pairs * 9, "flops": 2 * pairs}
    C = H * N * N * 4
    sweeps = {"count": 1 if c.get("decay") == 0 else 2, "refresh": 2, "profile": 1}[kind]
    return {"bytes": c["rows"] * H * k * 4 + sweeps * C, "flops": float(c["rows"]) * H * k * k}


def tolerance(case):
    # Selections come from fp32 sums of bf16 products.  Another order of the additions can swap two entries whose scores
    # differ in the last bits, and one swap moves the rest of its list by a place.  Against fp64 scores none of 400 thousand
    # selected entries differed; the share below is what one such swap in a token's hundred lists amounts to.
    if case["kind"] in ("step", "token", "batch", "medoid"):
        return {"differ": 0.002}
    return "exact"
