"""What this index is used for, as cases that can be timed: searches over the data shapes and batch sizes the
benchmark's configurations name, over every kind of list (floats, halves, bytes, product-quantiser codes), and
indexes that are created, loaded and fed by an insert stream.

A case is a dict of plain values:
  op        "search": one batch against an index that is already loaded
            "stream": a fresh index takes `n` vectors in one add, then `batches` insertion batches of `batch`
                      vectors, is rearranged where a list exceeds `threshold`, and answers one batch of queries
  data      "gauss", "bytes", "unit" or "zipf": the mixtures of paper_2408_02937_amd/synth.py, drawn on the GPU
  d, n, nlist, block_vecs, metric, storage, pq_m: the index; nprobe, k, nq: the request.
"""
import math

import torch

from paper_2408_02937_amd import rtams

DEV = "cuda:0"
CHUNK_ELEMS = 1 << 29  # coordinates of the base set that are drawn at a time


def _search(name, data, d, n, nlist, block_vecs, metric, nprobe, k, nq, storage="f32", pq_m=0):
    return {"name": name, "op": "search", "data": data, "d": d, "n": n, "nlist": nlist, "block_vecs": block_vecs,
            "metric": metric, "nprobe": nprobe, "k": k, "nq": nq, "storage": storage, "pq_m": pq_m,
            "batch": 0, "batches": 0, "threshold": 0}


def _stream(name, data, d, n, nlist, block_vecs, metric, nprobe, k, nq, batch, batches, threshold, storage="f32", pq_m=0):
    c = _search(name, data, d, n, nlist, block_vecs, metric, nprobe, k, nq, storage, pq_m)
    return {**c, "op": "stream", "batch": batch, "batches": batches, "threshold": threshold}


def listed():
    return [
        # the smallest index and the paper's own serving batch (at most 10 queries): five short launches
        _search("tiny_batch10", "gauss", 32, 10_000, 64, 64, "l2", 8, 10, 10),
        # one interactive query against a million byte-valued vectors: a chain of latencies
        _search("bytes_batch1", "bytes", 128, 1_000_000, 1024, 128, "l2", 32, 100, 1),
        # a serving batch of ordinary size on the same index
        _search("bytes_batch32", "bytes", 128, 1_000_000, 1024, 128, "l2", 32, 100, 32),
        # throughput on the same index: every list is probed by several queries of the batch
        _search("bytes_batch256", "bytes", 128, 1_000_000, 1024, 128, "l2", 32, 100, 256),
        # ten million deep embeddings by inner product
        _search("unit96_batch128", "unit", 96, 10_000_000, 4096, 256, "ip", 64, 10, 128),
        # retrieval over wide text embeddings; pairs spread thinly over many lists
        _search("unit768_batch64", "unit", 768, 5_000_000, 8192, 128, "ip", 32, 10, 64),
        # the benchmark's workload: skewed growth, hot lists of millions of vectors that most queries probe
        _search("zipf256_batch256", "zipf", 256, 20_000_000, 16384, 256, "l2", 64, 50, 256),
        # lists of product-quantiser codes, sixteen bytes a vector
        _search("pq16_batch256", "bytes", 128, 1_000_000, 1024, 128, "l2", 32, 100, 256, pq_m=16),
        # lists that keep bytes instead of floats: a quarter of the memory, the same answers
        _search("u8_batch256", "bytes", 128, 1_000_000, 1024, 128, "l2", 32, 100, 256, storage="u8"),
        # real-time insertion in small batches into an index of ordinary size
        _stream("insert64", "bytes", 128, 65_536, 1024, 128, "l2", 32, 100, 32, 64, 256, 0),
        # a fast insert stream of larger batches from a skewed law, hot lists rearranged afterwards
        _stream("insert1024_zipf", "zipf", 256, 65_536, 16384, 256, "l2", 64, 50, 256, 1024, 64, 10_000),
        # bulk load: the coarse quantizer over 8,192 centroids of wide vectors
        _stream("load_unit768", "unit", 768, 500_000, 8192, 128, "ip", 32, 10, 64, 0, 0, 0),
    ]


def _log(rng, lo, hi):
    """A whole number between lo and hi, spread over its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    data = rng.choice(["gauss", "bytes", "unit", "zipf"])
    metric = {"gauss": "l2", "bytes": "l2", "unit": "ip", "zipf": "l2"}[data]
    kind = rng.choice(["f32", "f32", "f32", "f32", "f16", "u8", "pq"])
    if kind == "u8" and data != "bytes":
        kind = "f32"
    step = {"f32": 4, "f16": 8, "u8": 16, "pq": 8}[kind]
    d = max(step, _log(rng, 24, 768 if data == "unit" else 256) // step * step)
    pq_m = 0
    if kind == "pq":
        pq_m = rng.choice([m for m in (4, 8, 12, 16, 24, 32, 48, 64) if d % m == 0 and m <= d])
    nlist = _log(rng, 64, 16384)
    op = rng.choice(["search", "search", "search", "search", "stream"])
    n = max(_log(rng, 10_000, min(5_000_000, 1_000_000_000 // d)), 8 * nlist)
    nprobe = _log(rng, 1, min(64, nlist))
    k = _log(rng, 1, 128)
    nq = _log(rng, 1, 256)
    block_vecs = rng.choice([64, 128, 256])
    storage = kind if kind in ("f16", "u8") else "f32"
    if op == "search":
        c = _search("", data, d, n, nlist, block_vecs, metric, nprobe, k, nq, storage, pq_m)
    else:
        n = max(8 * 64, min(n, 500_000_000 // d // 8, 2_000_000_000 // nlist))
        nlist = min(nlist, n // 8)
        batch = _log(rng, 8, 4096)
        batches = max(1, min(256, 200_000 // batch, 500_000_000 // (batch * nlist)))
        c = _stream("", data, d, n, nlist, block_vecs, metric, min(nprobe, nlist), k, nq, batch, batches,
                    rng.choice([0, 0, 10_000]), storage, pq_m)
    del c["name"]
    return c


# ------------------------------------------------------------------ inputs
def _gen(seed, stream):
    g = torch.Generator(device=DEV)
    g.manual_seed((int(seed) * 1_000_003 + stream) & 0x7FFFFFFFFFFF)
    return g


class _Data:
    """The mixture of a case: centres drawn once, rows drawn on demand from a generator of their own."""

    def __init__(self, case, seed):
        self.case, self.seed = case, seed
        d, data = case["d"], case["data"]
        g = _gen(seed, 0)
        if data == "zipf":
            self.sigma = 0.1
            self.centres = torch.randn(case["nlist"], d, generator=g, device=DEV)
            w = 1.0 / torch.arange(1, case["nlist"] + 1, dtype=torch.float64, device=DEV) ** 1.1
            self.cdf = torch.cumsum(w / w.sum(), 0)
            self.ranking = torch.randperm(case["nlist"], generator=g, device=DEV)
        else:
            # clusters: a few hundred vectors to one, as many as the set has lists or a few times that
            count = {"gauss": 100, "bytes": 1000, "unit": 10_000}[data]
            count = max(16, min(count, case["n"] // 100))
            if data == "bytes":
                self.sigma, self.centres = 20.0, torch.rand(count, d, generator=g, device=DEV) * 128.0
            else:
                self.sigma, self.centres = 0.1, torch.randn(count, d, generator=g, device=DEV)

    def rows(self, stream, n):
        g, data = _gen(self.seed, stream), self.case["data"]
        x = torch.randn(n, self.case["d"], generator=g, device=DEV)
        if data == "zipf":
            u = torch.rand(n, generator=g, device=DEV, dtype=torch.float64)
            at = self.ranking[torch.searchsorted(self.cdf, u).clamp_(max=self.case["nlist"] - 1)]
        else:
            at = torch.randint(self.centres.shape[0], (n,), generator=g, device=DEV)
        x.mul_(self.sigma).add_(self.centres[at])
        if data == "bytes":
            x.round_().clamp_(0.0, 255.0)
        if data == "unit":
            x.div_(x.norm(dim=1, keepdim=True))
        return x

    def base(self):
        """The base set, piece by piece."""
        per = max(1, min(self.case["n"], CHUNK_ELEMS // self.case["d"]))
        for i, lo in enumerate(range(0, self.case["n"], per)):
            yield self.rows(1000 + i, min(per, self.case["n"] - lo))

    def centroids(self):
        if self.case["data"] == "zipf":
            return self.centres.clone()
        return self.rows(2, self.case["nlist"])

    def queries(self):
        return self.rows(3, self.case["nq"])

    def inserts(self):
        return [self.rows(4, self.case["batch"] * self.case["batches"])] if self.case["batches"] else []

    def codebooks(self):
        d, m = self.case["d"], self.case["pq_m"]
        r = self.rows(5, 256 * 4).view(4, 256, m, d // m)  # 256 distinct sub-vectors for every sub-space
        return torch.stack([r[s % 4, :, s, :] for s in range(m)]).contiguous()


def _candidates(case):
    """Room for the candidates of a query: a few times the average, under the skewed law a quarter of everything."""
    n_all = case["n"] + case["batch"] * case["batches"]
    avg = case["n"] // case["nlist"]
    cand = max(65_536, 4 * case["nprobe"] * (avg + case["block_vecs"]))
    if case["data"] == "zipf":
        cand = max(cand, n_all // 4)
    return min(cand, n_all)


def _index(case, resources):
    n_all = case["n"] + case["batch"] * case["batches"]
    return rtams.Index(case["d"], case["nlist"], case["metric"], case["block_vecs"],
                       pool_blocks=n_all // case["block_vecs"] + 3 * case["nlist"] + 1024,
                       rearrange_threshold=case["threshold"], n_resources=resources, max_batch=256, max_k=128,
                       max_nprobe=min(64, case["nlist"]), max_add_batch=65536, candidates_per_query=_candidates(case),
                       storage=case["storage"], pq_m=case["pq_m"])


def prepare(case, seed):
    data = _Data(case, seed)
    state = {"case": case, "queries": data.queries(), "centroids": data.centroids(),
             "codebooks": data.codebooks() if case["pq_m"] else None}
    if case["op"] == "stream":
        (state["base"],) = data.base() if case["n"] * case["d"] <= CHUNK_ELEMS else [torch.cat(list(data.base()))]
        flat = data.inserts()
        state["inserts"] = list(flat[0].split(case["batch"])) if flat else []
        return state
    depth = 8 if _candidates(case) <= 500_000 else 2  # requests in flight; gigabytes of candidate room to each of the largest
    ix = _index(case, depth)
    ix.set_centroids(state["centroids"])
    if case["pq_m"]:
        ix.set_codebooks(state["codebooks"])
    for piece in data.base():
        ix.add(piece)
    torch.cuda.synchronize()
    # a program that keeps several requests in flight waits for the oldest before it submits the next
    state.update(index=ix, depth=depth, events=[], turn=0)
    return state


def _run_search(s):
    case, depth = s["case"], s["depth"]
    at = s["turn"] % depth
    if s["turn"] >= depth:
        s["events"][at].synchronize()
    else:
        s["events"].append(torch.cuda.Event())
    s["turn"] += 1
    dist, ids = s["index"].search(s["queries"], case["k"], case["nprobe"])
    s["events"][at].record()
    return {"dist": dist, "ids": ids}


def _run_stream(s):
    case = s["case"]
    ix = _index(case, 2)
    ix.set_centroids(s["centroids"])
    if case["pq_m"]:
        ix.set_codebooks(s["codebooks"])
    ix.add(s["base"])
    for b in s["inserts"]:
        ix.add(b)
    if case["threshold"]:
        torch.cuda.current_stream().synchronize()  # the host learns through pinned memory which lists exceed
        ix.rearrange(-1)
    dist, ids = ix.search(s["queries"], case["k"], case["nprobe"])
    sizes = ix.list_sizes()
    ix.close()
    return {"dist": dist, "ids": ids, "list_sizes": sizes}


def run(state):
    return _run_search(state) if state["case"]["op"] == "search" else _run_stream(state)


# ------------------------------------------------------------------ what a pass cannot do without
def work(case):
    d, n, nlist, nq, nprobe = case["d"], case["n"], case["nlist"], case["nq"], case["nprobe"]
    elem = {"f32": 4, "f16": 2, "u8": 1}[case["storage"]]
    stored = case["pq_m"] if case["pq_m"] else d * elem
    n_all = n + case["batch"] * case["batches"]
    per_query = n_all * nprobe / nlist
    if case["data"] == "zipf":  # a query's own list holds a vector with the probability a vector is drawn for it
        w = [1.0 / r ** 1.1 for r in range(1, nlist + 1)]
        per_query += n_all * sum(x * x for x in w) / sum(w) ** 2
    per_query = min(per_query, n_all)
    probed = 1.0 - (1.0 - nprobe / nlist) ** nq  # share of the lists some query of the batch probes
    per_pair = case["pq_m"] if case["pq_m"] else 2.0 * d  # additions of table entries, or multiply-adds
    out = {"bytes": n_all * stored * probed + nlist * d * 4 + nq * d * 4 + nq * case["k"] * 12,
           "flops": 2.0 * nq * nlist * d + per_pair * nq * per_query}
    if case["op"] == "stream":  # every vector is read once, written once with its id, and compared with the centroids
        out["bytes"] += n_all * (d * 4 + stored + 8)
        out["flops"] += 2.0 * n_all * nlist * d + (2.0 * 256 * d * n_all if case["pq_m"] else 0.0)
    return out


def tolerance(case):
    # byte values: every score is a whole number below 2^24, held exactly in 32 bits
    if case["data"] == "bytes" and not case["pq_m"]:
        return "exact"
    # sums of d (or pq_m) products in 32 bits: the same requests with the sums in another order differ by up to 2.5e-7
    # (norm), 1.1e-6 (one value) and 5e-4 (ids of neighbours whose scores agree to that), against 64 bits by 3.6e-7
    return {"rel": 1.4e-6, "max": 5e-6, "differ": 0.002}


# ------------------------------------------------------------------ the same in 64 bits, in plain torch
def _stored(case, x):
    if case["storage"] == "f16":
        return x.half().double()
    if case["storage"] == "u8":
        return x.round().clamp(0.0, 255.0).double()
    return x.double()


def _coarse(metric, y, c):
    """Scores [len(y)][len(c)] of rows against centroids; smaller is better."""
    p = y @ c.t()
    return p.neg_() if metric == "ip" else p.mul_(-2.0).add_((c * c).sum(1))


def exact(case, seed):
    data = _Data(case, seed)
    metric, k = case["metric"], case["k"]
    cents = data.centroids().double()
    q = data.queries().double()
    order = torch.sort(_coarse(metric, q, cents), dim=1, stable=True).indices[:, :case["nprobe"]]
    probed = torch.zeros(case["nq"], case["nlist"], dtype=torch.bool, device=DEV).scatter_(1, order, True)
    books = lut = None
    if case["pq_m"]:
        m, ds = case["pq_m"], case["d"] // case["pq_m"]
        books = data.codebooks().double()
        sub = q.view(-1, m, 1, ds)
        lut = ((sub - books) ** 2).sum(3) if metric == "l2" else (sub * books).sum(3)  # [nq][m][256]
    worst = math.inf if metric == "l2" else -math.inf
    best = torch.full((case["nq"], k), worst, dtype=torch.float64, device=DEV)
    sizes = torch.zeros(case["nlist"], dtype=torch.int64, device=DEV)
    rows = max(256, min((1 << 28) // max(case["nlist"], case["nq"]), (1 << 28) // case["d"]))
    for piece in [*([] if case["op"] == "search" else data.inserts())] + [None]:
        for big in ([piece] if piece is not None else data.base()):
            for x32 in big.split(rows):
                x = x32.double()
                lists = _coarse(metric, x, cents).argmin(1)
                sizes += torch.bincount(lists, minlength=case["nlist"])
                if case["pq_m"]:
                    s = torch.zeros(case["nq"], len(x), dtype=torch.float64, device=DEV)
                    for j in range(m):
                        xs = x[:, j * ds:(j + 1) * ds]
                        code = ((books[j] ** 2).sum(1) - 2.0 * xs @ books[j].t()).argmin(1)
                        s += lut[:, j, :][:, code]
                else:
                    x = _stored(case, x32)
                    s = q @ x.t()
                    if metric == "l2":
                        s = s.mul_(-2.0).add_((q * q).sum(1, keepdim=True)).add_((x * x).sum(1))
                s.masked_fill_(~probed[:, lists], worst)
                top = torch.topk(s, min(k, s.shape[1]), dim=1, largest=metric == "ip").values
                best = torch.topk(torch.cat([best, top], 1), k, dim=1, largest=metric == "ip").values
    if metric == "l2":
        best = best.clamp_(min=0.0)
    out = {"dist": best, "ids": None}
    if case["op"] == "stream":
        out["list_sizes"] = None
    return out
