"""The work a program has this library do, as cases to be timed.

Every case calls the Python binding the way a user's program does.  The graphs
are synthetic and made on the GPU from the seed alone, with the three shapes
the library is used on:

  sbm   planted partition: blocks of 128 vertices, unit weights (short, even
        rows; clear communities)
  rmat  R-MAT (0.57, 0.19, 0.19), simple, loop-free, unit weights (hubs of
        10^3 to 10^5 entries, weak communities, isolated vertices)
  lfr   power-law degrees (exponent 2.5, mean 20, at most 5,000) and power-law
        communities (exponent 1.5, 50 to 20,000 vertices), mixing 0.3, integer
        weights 1..8

Vertex ids carry no locality in any of them except the blocks of `sbm`.
"""
import math

import numpy as np
import torch

import paper_2507_06471_amd as lv

DEVICE = "cuda"

# name, call, graph, n, and the graph's density: `ef` R-MAT samples per vertex,
# `deg` mean degree (sbm, lfr); `host` = the program wants labels in host memory
LISTED = [
    # The smallest whole run: a few thousand vertices, every level and every
    # level's labels back on the host.  Launches and round trips are the cost.
    dict(name="louvain_sbm_4096", call="louvain", graph="sbm", n=4096, deg=8.4, host=True),
    # Label propagation on a small graph of odd size, labels on the host.
    dict(name="lpa_rmat_10007", call="lpa", graph="rmat", n=10007, ef=8, host=True),
    # Scoring a given partition: the smallest call there is.
    dict(name="modularity_sbm_4096", call="modularity", graph="sbm", n=4096, deg=8.4),
    # An ordinary unweighted graph of two million entries.
    dict(name="louvain_rmat_65536", call="louvain", graph="rmat", n=65536, ef=16, host=True),
    # An ordinary weighted graph with clear communities (social-network like).
    dict(name="louvain_lfr_1000003", call="louvain", graph="lfr", n=1000003, deg=20.0, host=False),
    # Label propagation on a larger weighted graph.
    dict(name="lpa_lfr_3000017", call="lpa", graph="lfr", n=3000017, deg=20.0, host=False),
    # Label propagation with hubs; 128 M samples in about 4 M vertices.
    dict(name="lpa_rmat_4194304", call="lpa", graph="rmat", n=4194304, ef=16, host=False),
    # The whole of a one-off job: CSR in host memory, a handle, Louvain, the
    # labels back in host memory, the handle closed.
    dict(name="job_rmat_700001", call="job", graph="rmat", n=700001, ef=12),
    # A raw edge list on the device (loops and repeats in it) becomes a handle,
    # whose merged CSR is read back on the device.
    dict(name="edges_rmat_2097152", call="edges", graph="rmat", n=2097152, ef=16),
    # Many small graphs packed into one handle, every graph's partition back.
    dict(name="batch_256", call="batch", graph="mix", count=256, lo=1024, hi=65536, mode="louvain"),
    # A server with a burst of jobs from clients, all results collected.
    dict(name="serve_16", call="serve", graph="rmat", count=16, lo=10000, hi=1000000),
    # The largest graph the framework is benchmarked on, labels left on the GPU.
    dict(name="louvain_rmat_16777216", call="louvain", graph="rmat", n=16777216, ef=16, host=False),
]


def listed():
    return [dict(c) for c in LISTED]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    call = rng.choice(["louvain", "louvain", "louvain", "lpa", "lpa", "modularity", "job", "edges", "batch", "serve"])
    if call == "batch":
        return dict(call=call, graph="mix", count=_log(rng, 16, 400), lo=1024, hi=_log(rng, 4096, 65536),
                    mode=rng.choice(["louvain", "lpa"]))
    if call == "serve":
        return dict(call=call, graph="rmat", count=rng.randint(4, 24), lo=10000, hi=_log(rng, 50000, 1000000))
    if call == "job":
        return dict(call=call, graph="rmat", n=_log(rng, 10000, 4000000), ef=rng.randint(8, 16))
    if call == "edges":
        return dict(call=call, graph="rmat", n=_log(rng, 20000, 4194304), ef=rng.randint(8, 16))
    graph = rng.choice(["sbm", "rmat", "lfr"])
    top = 4000000 if call == "modularity" else {"sbm": 65536, "rmat": 16777216, "lfr": 10000000}[graph]
    c = dict(call=call, graph=graph)
    if graph == "sbm":
        c.update(n=_log(rng, 1024, min(top, 65536)), deg=round(rng.uniform(8.0, 32.0), 2))
    elif graph == "rmat":
        c.update(n=_log(rng, 10000, top), ef=rng.randint(8, 16))
    else:
        c.update(n=_log(rng, 20000, top), deg=20.0)
    if call != "modularity":
        c["host"] = c["n"] < 500000
    return c


# ---------------------------------------------------------------- graphs
class Csr:
    """Symmetric CSR: int32 offsets / indices, int32 weights or None (unit)."""

    def __init__(self, n, offsets, indices, weights=None):
        self.n, self.offsets, self.indices, self.weights = n, offsets, indices, weights

    def host(self):
        w = None if self.weights is None else self.weights.cpu().numpy()
        return Csr(self.n, self.offsets.cpu().numpy(), self.indices.cpu().numpy(), w)


def _generator(seed):
    return torch.Generator(device=DEVICE).manual_seed(int(seed))


def _canonical(n, u, v, gen=None):
    """CSR of the simple loop-free graph with the listed pairs; weights 1..8 if a generator is given."""
    key = torch.minimum(u, v) * n + torch.maximum(u, v)
    key = torch.unique(key[u != v])
    u, v = key // n, key % n
    del key
    w = None
    if gen is not None:
        w = torch.randint(1, 9, u.shape, generator=gen, device=DEVICE, dtype=torch.int32)
    both = torch.cat([u * n + v, v * n + u])
    del u, v
    if w is None:
        both = torch.sort(both).values
    else:
        both, at = torch.sort(both)
        w = torch.cat([w, w])[at]
        del at
    offsets = torch.searchsorted(both, torch.arange(n + 1, device=DEVICE) * n).to(torch.int32)
    return Csr(n, offsets, (both % n).to(torch.int32), w)


def _rmat_samples(n, ef, gen):
    """ef * n quadrant descents: endpoints int64 (an endpoint outside [0, n) makes the sample the loop (0, 0))."""
    m = int(ef) * n
    u = torch.zeros(m, dtype=torch.int64, device=DEVICE)
    v = torch.zeros(m, dtype=torch.int64, device=DEVICE)
    for _ in range(max(1, (n - 1).bit_length())):
        r = torch.rand(m, generator=gen, device=DEVICE)
        u.mul_(2).add_(r >= 0.76)
        v.mul_(2).add_(((r >= 0.57) & (r < 0.76)) | (r >= 0.95))
    out = (u >= n) | (v >= n)
    return u.masked_fill_(out, 0), v.masked_fill_(out, 0)


def _sbm(n, deg, gen, intra=0.75, block=128):
    """Blocks of 128 consecutive vertices holding `intra` of the mean degree."""
    m_in, m_out = int(n * deg * intra / 2), int(n * deg * (1 - intra) / 2)
    u = torch.randint(0, n, (m_in,), generator=gen, device=DEVICE)
    b0 = u // block * block
    size = torch.clamp(n - b0, max=block)
    v = b0 + (torch.rand(m_in, generator=gen, device=DEVICE, dtype=torch.float64) * size).long()
    x = torch.randint(0, n, (2, m_out), generator=gen, device=DEVICE)
    return _canonical(n, torch.cat([u, x[0]]), torch.cat([v, x[1]]))


def _power_law(gen, count, lo, hi, tau):
    u = torch.rand(count, generator=gen, device=DEVICE, dtype=torch.float64)
    a, b = lo ** (1 - tau), hi ** (1 - tau)
    return (a + u * (b - a)) ** (1 / (1 - tau))


def _lfr(n, deg, gen, mu=0.3):
    """Configuration models inside the communities and across them; (CSR, community of each vertex)."""
    top = float(min(5000, n // 4))
    k = _power_law(gen, n, deg / 3, top, 2.5).round().long().clamp(min=1)
    sizes = _power_law(gen, n // 50 + 1, 50.0, float(min(20000, n // 4)), 1.5).round().long()
    ends = torch.cumsum(sizes, 0)
    member = torch.searchsorted(ends, torch.arange(n, device=DEVICE), right=True)
    sizes = torch.bincount(member)
    member = member[torch.randperm(n, generator=gen, device=DEVICE)]
    inner = torch.minimum(((1 - mu) * k).round().long(), sizes[member] - 1)
    ids = torch.arange(n, device=DEVICE)
    stub = torch.repeat_interleave(ids, inner)
    key = member[stub] * (1 << 40) + torch.randint(0, 1 << 40, stub.shape, generator=gen, device=DEVICE)
    stub = stub[torch.argsort(key, stable=True)]
    del key
    c = member[stub]
    first = torch.searchsorted(c, torch.arange(len(sizes), device=DEVICE))
    rank = torch.arange(len(c), device=DEVICE) - first[c]
    pair = (rank[:-1] % 2 == 0) & (c[:-1] == c[1:])
    u, v = stub[:-1][pair], stub[1:][pair]
    del c, rank, pair, stub
    out = torch.repeat_interleave(ids, k - inner)
    out = out[torch.randperm(len(out), generator=gen, device=DEVICE)]
    half = len(out) // 2
    u, v = torch.cat([u, out[:half]]), torch.cat([v, out[half:2 * half]])
    return _canonical(n, u, v, gen), member


def _graph(case, gen):
    """(CSR on the GPU, a partition of its vertices)."""
    n = case["n"]
    if case["graph"] == "sbm":
        return _sbm(n, case["deg"], gen), torch.arange(n, device=DEVICE) // 128
    if case["graph"] == "lfr":
        return _lfr(n, case["deg"], gen)
    g = _canonical(n, *_rmat_samples(n, case["ef"], gen))
    return g, torch.randint(0, n // 50 + 1, (n,), generator=gen, device=DEVICE)


def _many(case, gen):
    """Graphs of log-uniform size in [lo, hi]: R-MAT, alternating with sbm for `mix`."""
    t = torch.linspace(0, 1, case["count"], dtype=torch.float64)
    sizes = torch.exp(math.log(case["lo"]) + t * (math.log(case["hi"]) - math.log(case["lo"]))).round().long()
    at = torch.randperm(case["count"], generator=torch.Generator().manual_seed(case["count"]))
    out = []
    for i, n in enumerate(sizes[at].tolist()):
        deg = 8 + 24 * ((i * 0.6180339887) % 1.0)
        if case["graph"] == "mix" and i % 2 == 0:
            out.append(_sbm(n, deg, gen).host())
        else:
            ef = max(4, round(deg / 2)) if case["graph"] == "mix" else 8 + i % 9
            out.append(_canonical(n, *_rmat_samples(n, ef, gen)).host())
    return out


# ---------------------------------------------------------------- the calls
def prepare(case, seed):
    gen, call = _generator(seed), case["call"]
    if call == "batch":
        return {"case": case, "graph": lv.Graph.batch(_many(case, gen))}
    if call == "serve":
        return {"case": case, "graphs": _many(case, gen), "server": lv.Server()}
    if call == "edges":
        u, v = _rmat_samples(case["n"], case["ef"], gen)
        # room for every sample as its own pair; what the merged graph does not need stays zero
        room = [torch.zeros(k, dtype=torch.int32, device=DEVICE) for k in (case["n"] + 1, 2 * len(u), 2 * len(u))]
        s = {"case": case, "src": u.to(torch.int32), "dst": v.to(torch.int32)}
        s.update(zip(("offsets", "indices", "weights"), room))
        torch.cuda.synchronize()
        return s
    g, part = _graph(case, gen)
    if call == "job":
        return {"case": case, "csr": g.host()}
    torch.cuda.synchronize()
    s = {"case": case, "graph": lv.Graph(g.n, g.offsets, g.indices, g.weights)}
    if call == "modularity":
        s["labels"] = part.to(torch.int32)
    elif not case["host"]:
        s["out"] = torch.empty(g.n, dtype=torch.int32, device=DEVICE)
    torch.cuda.synchronize()
    return s


def _louvain_outputs(r):
    moves = np.zeros((8, 20), dtype=np.int64)
    q_end = np.zeros(8, dtype=np.int64)
    for i, x in enumerate(r.levels[:8]):
        moves[i, :len(x.moves)] = x.moves
        q_end[i] = x.info["q_end"]
    first = r.levels[0].labels
    return {"labels": r.final_labels, "first_level": r.final_labels if first is None else first,
            "q_int": r.q_int, "M": r.M, "q": r.q, "moves": moves, "q_end": q_end}


def run(s):
    case = s["case"]
    call = case["call"]
    if call == "louvain":
        if case["host"]:
            return _louvain_outputs(lv.louvain(s["graph"]))
        return _louvain_outputs(lv.louvain(s["graph"], level_labels=False, out=s["out"]))
    if call == "lpa":
        r = lv.lpa(s["graph"], out=s.get("out"))
        moves = np.zeros(20, dtype=np.int64)
        moves[:len(r.moves)] = r.moves
        return {"labels": r.labels, "moves": moves, "q_int": r.info["q_end"]}
    if call == "modularity":
        q_int, M, q = lv.modularity(s["graph"], s["labels"])
        return {"q_int": q_int, "M": M, "q": q}
    if call == "job":
        with lv.Graph.from_csr(s["csr"]) as g:
            r = lv.louvain_final(g)
        return {"labels": r.labels, "q_int": r.q_int, "M": r.M, "q": r.q}
    if call == "edges":
        with lv.Graph.from_edges(case["n"], s["src"], s["dst"], drop_loops=True, simple=True) as g:
            nnz = g.nnz
            status = lv.load_library().lv_graph_csr(g.handle, s["offsets"].data_ptr(), s["indices"].data_ptr(),
                                                    s["weights"].data_ptr(), None, lv.LV_MEM_DEVICE)
        if status != lv.LV_OK:
            raise RuntimeError(f"lv_graph_csr: {status}")
        return {"nnz": nnz, "offsets": s["offsets"], "indices": s["indices"], "weights": s["weights"]}
    if call == "batch":
        if case["mode"] == "lpa":
            rs = lv.lpa(s["graph"])
            return {"labels": np.concatenate([r.labels for r in rs]),
                    "sweeps": np.asarray([r.info["sweeps"] for r in rs], dtype=np.int64),
                    "q_int": np.asarray([r.info["q_end"] for r in rs], dtype=np.int64)}
        r = lv.louvain_final(s["graph"])
        return {"labels": r.labels, "q_int": r.q_int, "M": r.M, "q": r.q}
    server = s["server"]
    tickets = [server.submit(g) for g in s["graphs"]]
    got = []
    for t, g in zip(tickets, s["graphs"]):
        server.wait(t)
        got.append(server.result(t, g.n))
    return {"labels": [x[0] for x in got], "q_int": [x[1]["q_int"] for x in got]}


def _entries(case):
    """(vertices, CSR entries) of the case's graphs, as drawn (duplicates of R-MAT samples not taken off)."""
    if case["call"] in ("batch", "serve"):
        lo, hi = math.log(case["lo"]), math.log(case["hi"])
        n = case["count"] * (case["hi"] - case["lo"]) / max(hi - lo, 1e-9)
        return n, n * (20 if case["graph"] == "mix" else 24)
    return case["n"], case["n"] * (2 * case["ef"] if case["graph"] == "rmat" else case["deg"])


def work(case):
    """The graph read once, one add per entry, and the labels (or the merged CSR) written once."""
    n, e = _entries(case)
    per = 8 if case["graph"] == "lfr" else 4
    if case["call"] == "edges":
        return {"bytes": 8 * e / 2 + 4 * n + 8 * e, "flops": e}
    return {"bytes": per * e + 8 * n, "flops": e}


def exact(case, seed):
    """Modularity in 64-bit integers and doubles; the other calls return partitions, whole numbers, and a
    modularity that follows from the partition they found."""
    if case["call"] != "modularity":
        return None
    g, part = _graph(case, _generator(seed))
    w = torch.ones(len(g.indices), dtype=torch.int64, device=DEVICE) if g.weights is None else g.weights.long()
    row = torch.repeat_interleave(torch.arange(g.n, device=DEVICE), (g.offsets[1:] - g.offsets[:-1]).long())
    deg = torch.zeros(g.n, dtype=torch.int64, device=DEVICE).index_add_(0, row, w)
    vol = torch.zeros(int(part.max()) + 1, dtype=torch.int64, device=DEVICE).index_add_(0, part, deg)
    inside = int(w[part[row] == part[g.indices.long()]].sum())
    M = int(deg.sum())
    q_int = M * inside - int((vol * vol).sum())
    return {"q_int": q_int, "M": M, "q": float(np.float64(q_int) / (np.float64(M) * np.float64(M)))}
