"""The work that a user of this library has it do, as cases that can be timed and compared.

A case is one call, or one round of calls, of the public Python entry points
(`paper_2602_21477_amd.binding`) on inputs that are already on the GPU: searches from one query on
a small memory up to batches of 1024 over ten million vectors, the rounds of a memory that changes
between searches, a call that serves many agents, the build of an index and the training of its
centroids.  The shapes are those of `paper_2602_21477_amd.workload` and of the tests; the data are
the same seeded Gaussian mixtures (drawn on the GPU, normalised last), with centroids from a few
Lloyd iterations on a sample or, for the skewed memory, the means of the mixture's components.
"""
import math

import torch

from paper_2602_21477_amd import binding as B

SIGMA, QNOISE = 0.3, 0.05
ROOM = 65536  # vectors that an index which takes inserts has room for beyond those it is built from


# ------------------------------------------------------------------------------------------ cases

def _search(name, n, d, nlist, nprobe, k, nq, metric="ip", storage="f32", zipf=0.0, page=0, replaced=0, probed=0.0):
    """`replaced`: memories deleted and inserted again with new contents before the search.
    `probed`: share of the rows in lists that at least one query probes, where the lists are so uneven that the
    count of a fair spread says little (0: the fair spread)."""
    return {"name": name, "kind": "search", "n": n, "d": d, "nlist": nlist, "nprobe": nprobe, "k": k, "nq": nq,
            "metric": metric, "storage": storage, "zipf": zipf, "page": page, "replaced": replaced, "probed": probed}


def listed():
    return [
        # One question of one small agent: what a single call costs when there is next to nothing to read.
        _search("one_query_small", 20_000, 128, 64, 8, 10, 1),
        # The same memory under a full batch (the tiny workload of the benchmark).
        _search("batch_256_small", 20_000, 128, 64, 8, 10, 256),
        # A memory with no round number anywhere: rows that are padded, half-filled pages, few queries, long results.
        _search("ragged_l2_f16", 123_457, 411, 333, 19, 77, 37, "l2", "f16", page=96),
        # One agent over a million embeddings, answering a handful of requests at a time (the batch size that
        # query throughput is usually quoted at) ...
        _search("agent_8_queries", 1_000_000, 768, 1024, 32, 10, 8),
        # ... and a fuller batch in which 8 memories have been rewritten since the last one (update = delete + insert).
        _search("agent_64_queries_8_new", 1_000_000, 768, 1024, 32, 10, 64, replaced=8),
        # Sixteen agents with memories of their own, 32 queries each, in one call.
        {"name": "sixteen_agents", "kind": "multi", "agents": 16, "n": 0, "n_lo": 100_000, "n_hi": 500_000, "d": 1024,
         "nlist": 512, "nprobe": 16, "k": 20, "nq": 32, "metric": "ip", "storage": "f32"},
        # The benchmark's own workload: ten million half-precision rows, 1024 queries, both metrics.  (Under L2 the
        # merged clusters that Lloyd leaves behind draw most probes: fewer rows, many queries on each.)
        _search("large_ip_f16", 10_000_000, 768, 4096, 64, 100, 1024, "ip", "f16"),
        _search("large_l2_f16", 10_000_000, 768, 4096, 64, 100, 1024, "l2", "f16", probed=0.35),
        # A skewed memory (cluster sizes by Zipf's law, wide rows) that is written to before every small batch.
        _search("skewed_16_queries_1_new", 2_000_000, 1536, 2048, 48, 10, 16, zipf=1.2, replaced=1, probed=0.5),
        # A memory that is brought up to date in bulk: two thousand rows replaced, and a look at the result.
        _search("replace_2000", 300_000, 1024, 512, 16, 20, 4, replaced=2000),
        # An agent's memory is loaded: the index is built over its vectors and asked for the first time.
        {"name": "build_300k", "kind": "build", "n": 300_000, "d": 1024, "nlist": 512, "nprobe": 16, "k": 20, "nq": 32,
         "metric": "ip", "storage": "f32"},
        # The centroids of the ten-million-vector memory are trained, an iteration at a time (several in a row are not
        # comparable: a near-tied row that changes sides changes every later iteration).
        {"name": "kmeans_4096", "kind": "kmeans", "n": 262_144, "d": 768, "nlist": 4096, "iters": 1},
    ]


def draw(rng):
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["search"] * 6 + ["replace"] * 2 + ["multi", "build", "kmeans"])
    d = log(48, 1536)
    if rng.random() < 0.4:  # embedding widths are round more often than not
        d = max(64, d // 64 * 64)
    nlist = log(40, 2048)
    n = min(log(max(10_000, 24 * nlist), 1_500_000), 1_200_000_000 // d)
    nprobe = min(nlist, log(4, 64))
    case = {"n": n, "d": d, "nlist": nlist, "nprobe": nprobe, "k": log(1, 100), "nq": log(1, 1024),
            "metric": rng.choice(["ip", "l2"]), "storage": rng.choice(["f32", "f32", "f16"])}
    if kind == "kmeans":
        return {"kind": "kmeans", "n": min(n, 262_144), "d": d, "nlist": nlist, "iters": 1}
    if kind == "multi":
        agents = rng.randint(2, 16)
        hi = max(2 * 24 * nlist, n // agents)
        return dict(case, kind="multi", agents=agents, n=0, n_lo=hi // 3, n_hi=hi, nq=log(1, 64))
    if kind == "build":
        return dict(case, kind="build", nq=log(1, 64))
    return dict(case, kind="search", zipf=0.0, page=rng.choice([0, 0, 0, 64, 256]), probed=0.0,
                replaced=log(1, 2000) if kind == "replace" else 0)


# ------------------------------------------------------------------------------------------ inputs

def _gen(seed, stream):
    return torch.Generator(device="cuda").manual_seed((int(seed) * 1009 + stream) % (1 << 62))


def _weights(ncomp, zipf):
    w = torch.arange(1, ncomp + 1, dtype=torch.float64, device="cuda") ** (-zipf)
    return torch.cumsum(w / w.sum(), 0)


def _mixture(g, mu, cdf, m, noise, f16):
    """m rows of the mixture, float32; for half-precision memories already rounded to what is stored."""
    x = torch.empty((m, mu.shape[1]), dtype=torch.float32, device="cuda")
    for a in range(0, m, 1 << 19):
        b = min(m, a + (1 << 19))
        comp = torch.searchsorted(cdf, torch.rand(b - a, dtype=torch.float64, device="cuda", generator=g)).clamp_(max=len(cdf) - 1)
        t = torch.randn((b - a, mu.shape[1]), device="cuda", generator=g).mul_(noise).add_(mu[comp])
        t /= t.norm(dim=1, keepdim=True).clamp_(min=1e-30)
        x[a:b] = t.half() if f16 else t
    return x


def _lloyd(g, x, nlist, iters):
    """A few Lloyd iterations under L2 on a sample; sums in whole numbers, so that they come out the same every time."""
    rows = x if len(x) <= 64 * nlist else x[torch.randint(len(x), (64 * nlist,), device="cuda", generator=g)]
    cent = rows[torch.randperm(len(rows), device="cuda", generator=g)[:nlist]].clone()
    fixed = (rows.double() * 2.0 ** 40).long()
    for _ in range(iters):
        cn = cent.square().sum(1)
        assign = torch.cat([(cn - 2 * (rows[a:a + 65536] @ cent.T)).argmin(1) for a in range(0, len(rows), 65536)])
        total = torch.zeros(cent.shape, dtype=torch.int64, device="cuda").index_add_(0, assign, fixed)
        count = torch.bincount(assign, minlength=nlist)[:, None]
        cent = torch.where(count > 0, (total.double() / 2.0 ** 40 / count.clamp(min=1)).float(), cent)
    return cent


def _memory(case, seed, agent, n):
    """(rows, centroids, a source of queries, a source of new rows) of one memory."""
    d, nlist, f16, zipf = case["d"], case["nlist"], case["storage"] == "f16", case.get("zipf", 0.0)
    g = _gen(seed, 1 + agent)
    mu = torch.randn((nlist, d), device="cuda", generator=g)
    cdf = _weights(nlist, zipf)
    x = _mixture(g, mu, cdf, n, SIGMA, f16)
    if zipf > 0:
        cent = torch.stack([(t / t.norm(dim=1, keepdim=True)).mean(0) for t in
                            (m + SIGMA * torch.randn((32, d), device="cuda", generator=g) for m in mu)])
    else:
        cent = _lloyd(g, x, nlist, 6)

    def queries(m):
        return _mixture(g, mu, cdf, m, math.hypot(SIGMA, QNOISE), False)

    def new_rows(m):  # a skewed memory is written where it is largest
        top = max(1, nlist // 20) if zipf > 0 else nlist
        return _mixture(g, mu[:top], _weights(top, 0.0), m, SIGMA, f16)

    return x, cent, queries, new_rows, g


def _inputs(case, seed):
    """Everything a case is given: per agent its rows and centroids, then queries and replacements."""
    sizes = [case["n"]]
    if case["kind"] == "multi":
        t = torch.Generator().manual_seed(int(seed) % (1 << 62))
        sizes = torch.randint(case["n_lo"], case["n_hi"] + 1, (case["agents"],), generator=t).tolist()
    for agent, n in enumerate(sizes):
        x, cent, queries, new_rows, g = _memory(case, seed, agent, n)
        q = queries(case["nq"])
        m = case.get("replaced", 0)
        ids = torch.randperm(n, device="cuda", generator=g)[:m].contiguous() if m else None
        yield x, cent, q, ids, new_rows(m) if m else None


def _training(case, seed):
    g = _gen(seed, 1)
    mu = torch.randn((case["nlist"], case["d"]), device="cuda", generator=g)
    x = _mixture(g, mu, _weights(case["nlist"], 0.0), case["n"], SIGMA, False)
    return x, x[torch.randperm(case["n"], device="cuda", generator=g)[:case["nlist"]]].clone()


def _index(case, x, cent):
    return B.Index(cent, x, metric=B.PK_METRIC_L2 if case["metric"] == "l2" else B.PK_METRIC_IP,
                   storage=B.PK_F16 if case["storage"] == "f16" else B.PK_F32, page_vecs=case.get("page", 0),
                   insert_reserve=ROOM if case.get("replaced", 0) else 0)


def prepare(case, seed):
    state = {"case": case}
    if case["kind"] == "kmeans":
        state["x"], state["first"] = _training(case, seed)
        return state
    if case["kind"] == "build":
        (state["x"], state["cent"], state["q"], _, _), = _inputs(case, seed)
        return state
    # what a serving program keeps: its indexes, with the search workspace sized once
    state["index"], state["q"] = [], []
    for x, cent, q, ids, new in _inputs(case, seed):
        state["index"].append(_index(case, x, cent))
        state["q"].append(q)
        state["ids"], state["new"] = ids, new
        del x
    nq = case["nq"] * len(state["q"])
    B.pk_workspace_reserve([ix.handle for ix in state["index"]], max(nq, case.get("replaced", 0)), case["k"], case["nprobe"], 0)
    state["at"] = [case["nq"] * a for a in range(len(state["q"]) + 1)]
    state["q"] = torch.cat(state["q"])
    return state


def run(state):
    case = state["case"]
    if case["kind"] == "kmeans":
        cent = state["first"].clone()
        assign = torch.empty(case["n"], dtype=torch.int32, device="cuda")
        inertia = B.pk_kmeans(state["x"], cent, case["iters"], assign)
        return {"centroids": cent, "assign": assign, "inertia": inertia}
    if case["kind"] == "build":
        ix = _index(case, state["x"], state["cent"])
        ids, dist = ix.search(state["q"], case["k"], case["nprobe"])
        lengths = ix.list_lengths()
        ix.close()
        return {"ids": ids, "dist": dist, "lengths": lengths}
    if case["kind"] == "multi":
        ids, dist = B.search_multi(state["index"], state["at"], state["q"], case["k"], case["nprobe"])
        return {"ids": ids, "dist": dist}
    ix, out = state["index"][0], {}
    if case["replaced"]:
        out["removed"] = ix.delete(state["ids"])
        out["lists"] = ix.insert(state["new"], state["ids"], want_lists=True)
    out["ids"], out["dist"] = ix.search(state["q"], case["k"], case["nprobe"])
    return out


# ------------------------------------------------------------------------------------------ floors

def work(case):
    d, nlist = case["d"], case["nlist"]
    if case["kind"] == "kmeans":
        n, it = case["n"], case["iters"]
        return {"bytes": it * n * d * 4.0 + n * 4 + 2 * nlist * d * 4, "flops": 2.0 * it * n * nlist * d}
    size = 2 if case["storage"] == "f16" else 4
    nq, nprobe, k, m = case["nq"], case["nprobe"], case["k"], case.get("replaced", 0)
    agents = case.get("agents", 1)
    n = case["n"] if agents == 1 else (case["n_lo"] + case["n_hi"]) / 2
    share = case.get("probed", 0.0) or 1.0 - (1.0 - nprobe / nlist) ** nq
    # the probed rows once, the centroid table, the queries, the results; coarse and fine products
    nbytes = share * n * d * size + nlist * d * 4.0 + nq * d * 4 + nq * k * 12
    flops = 2.0 * d * (nq * nprobe * n / nlist + nq * nlist)
    if m:  # the ids of the memory, the new rows in and out, their assignment
        nbytes += n * 8.0 + m * d * (4 + size)
        flops += 2.0 * m * nlist * d
    if case["kind"] == "build":
        nbytes += n * d * (4.0 + size) + n * 8.0
        flops += 2.0 * n * nlist * d
    return {"bytes": agents * nbytes, "flops": agents * flops}


# ------------------------------------------------------------------------------------------ outputs

def tolerance(case):
    if case["kind"] == "kmeans":  # a near-tied row or two on the other side, each felt in two clusters of a few dozen rows
        return {"rel": 1e-3, "max": 0.5, "differ": 0.001}
    if case["storage"] == "f16":  # (the queries meet half-precision rows rounded to half precision themselves)
        return {"rel": 2e-4, "max": 2e-3, "differ": 0.01}
    return {"rel": 1e-5, "max": 1e-4, "differ": 0.01}


def _nearness(x, c, l2):
    """Larger is nearer; in 64 bits."""
    s = x @ c.T
    return 2 * s - c.square().sum(1) if l2 else s


def _exact_search(case, x, cent, q):
    l2 = case["metric"] == "l2"
    c, q = cent.double(), q.double()
    nq, k = len(q), case["k"]
    near = _nearness(q, c, l2).topk(case["nprobe"], 1).indices
    probed = torch.zeros((nq, len(c)), dtype=torch.bool, device="cuda").scatter_(1, near, True)
    best = torch.full((nq, k), -math.inf, dtype=torch.float64, device="cuda")
    ids = torch.full((nq, k), -1, dtype=torch.int64, device="cuda")
    lengths = torch.zeros(len(c), dtype=torch.int64, device="cuda")
    step = max(4096, min(131_072, (1 << 28) // max(nq, len(c))))
    for a in range(0, len(x), step):
        rows = x[a:a + step].double()
        assign = _nearness(rows, c, l2).argmax(1)
        lengths += torch.bincount(assign, minlength=len(c))
        v = q @ rows.T
        if l2:
            v = 2 * v - rows.square().sum(1) - q.square().sum(1)[:, None]
        v.masked_fill_(~probed[:, assign], -math.inf)
        v, at = v.topk(min(k, v.shape[1]), 1)
        best, pick = torch.cat([best, v], 1).topk(k, 1)
        ids = torch.cat([ids, at + a], 1).gather(1, pick)
    ids.masked_fill_(best == -math.inf, -1)
    return ids, (-best if l2 else best), lengths


def exact(case, seed):
    if case["kind"] == "kmeans":
        x, cent = _training(case, seed)
        # One near-tied row that goes to the other cluster moves a centroid by far more than any rounding does, so that
        # no 64-bit value stands for it; the sum of the distances is what a tie does not move.
        far = 0.0
        for a in range(0, len(x), 32768):
            rows = x[a:a + 32768].double()
            far += float((rows.square().sum(1) - _nearness(rows, cent.double(), True).amax(1)).sum())
        return {"centroids": None, "assign": None, "inertia": [far]}
    ids, dist, out = [], [], {}
    for x, cent, q, at, new in _inputs(case, seed):
        if at is not None:
            x[at] = new
            out["removed"] = len(at)
            out["lists"] = _nearness(new.double(), cent.double(), case["metric"] == "l2").argmax(1).int()
        i, v, lengths = _exact_search(case, x, cent, q)
        ids.append(i)
        dist.append(v)
    out["ids"], out["dist"] = torch.cat(ids), torch.cat(dist)
    if case["kind"] == "build":
        out["lengths"] = lengths
    return out
