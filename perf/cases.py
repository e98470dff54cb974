"""Timed cases of the similarity join: the calls that programs make, over the sizes they make them at.

A case is a plain dict.  ``profile`` names the shape of the corpus (dimensions, components per vector,
popularity exponent: those of the five workloads in synth/corpus.py), ``n`` its vectors, ``t`` the threshold,
and ``kind`` the call that one pass makes:

* ``join``      self-join of a resident index into device buffers (``entry``: plain, graph replay, or the
                allocation-free call); ``head`` > 0 builds the index with the bf16 head screen
* ``query``     external query rows against a resident index, rows and pairs on the host or on the device
* ``serve``     a burst of requests of uneven size through the continuous-batching server
* ``build``     building an index from rows on the device, and reading its ingredients
* ``dedupe``    one-shot use: rows on the host, index, join, pairs on the host, index freed

Corpora are drawn on the GPU from the seed: Zipf popularity without repeats in a row, lognormal weights,
unit rows in float32.
"""
import math

import numpy as np
import torch

import paper_1402_3010_amd as apss

# m dimensions, components per vector (uniform lo..hi, or lognormal of a mean and sigma clipped to lo..hi),
# popularity exponent s
PROFILES = {
    "short": dict(m=10_000, mean=35.0, sigma=0.0, lo=10, hi=60, s=1.0),
    "text": dict(m=200_000, mean=80.0, sigma=1.0, lo=5, hi=2000, s=1.1),
    "heavy": dict(m=1_000_000, mean=120.0, sigma=1.2, lo=5, hi=5000, s=1.0),
    "flat": dict(m=500_000, mean=150.0, sigma=1.0, lo=5, hi=2000, s=0.9),
    "serve": dict(m=1_000_000, mean=100.0, sigma=1.0, lo=5, hi=2000, s=1.0),
}


def listed():
    return [
        # a small collection joined again and again: launches and waits count
        dict(name="join_2k", kind="join", entry="plain", profile="short", n=2_000, t=0.5, head=0),
        # the same, replayed as a captured graph on the program's own stream
        dict(name="join_graph_3k", kind="join", entry="graph", profile="text", n=3_001, t=0.6, head=0),
        # a join inside a loop that may not allocate, odd size
        dict(name="join_noalloc_20k", kind="join", entry="noalloc", profile="text", n=20_011, t=0.7, head=0),
        # near-duplicate search at a low threshold: many pairs come out
        dict(name="join_100k", kind="join", entry="plain", profile="text", n=100_000, t=0.5, head=0),
        # the large join: heavy-tailed rows over a million dimensions
        dict(name="join_500k", kind="join", entry="plain", profile="heavy", n=500_000, t=0.7, head=0),
        # flat popularity, so a wide dense head: the screened join with its tuned geometry
        dict(name="screened_200k", kind="join", entry="plain", profile="flat", n=200_000, t=0.8, head=4096),
        # one lookup against a resident corpus: latency
        dict(name="query_1", kind="query", profile="serve", n=500_000, t_build=0.5, t=0.7, nq=1, device=False),
        # a small batch with its own threshold per row, device to device
        dict(name="query_64", kind="query", profile="serve", n=500_000, t_build=0.5, t=0.0, nq=64, device=True),
        # the largest request of a server
        dict(name="query_4096", kind="query", profile="serve", n=1_000_000, t_build=0.5, t=0.0, nq=4096, device=False),
        # uneven requests that arrive together
        dict(name="serve_burst", kind="serve", profile="serve", n=500_000, t_build=0.5, requests=20, largest=512,
             slots=2),
        # a new corpus on the device is indexed
        dict(name="build_500k", kind="build", profile="heavy", n=500_000, t=0.7),
        # a small batch of host rows is deduplicated once
        dict(name="dedupe_5k", kind="dedupe", profile="text", n=5_003, t=0.8),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["join", "join", "join", "query", "query", "serve", "build", "dedupe"])
    if kind == "join":
        profile = rng.choice(["short", "text", "heavy", "flat"])
        entry = rng.choice(["plain", "plain", "graph", "noalloc"])
        t = round(rng.uniform(0.5, 0.95), 3)
        head = 4096 if profile == "flat" and entry == "plain" and rng.random() < 0.5 else 0
        # the allocation-free call has room for about five million pairs
        top = 60_000 if entry == "noalloc" else 20_000 if profile == "short" else 150_000 if t < 0.65 else 300_000
        return dict(kind=kind, entry=entry, profile=profile, n=_log_int(rng, 1_500, top), t=t, head=head)
    if kind == "query":
        same_t = rng.random() < 0.5
        return dict(kind=kind, profile=rng.choice(["serve", "text"]), n=_log_int(rng, 20_000, 1_000_000), t_build=0.5,
                    t=round(rng.uniform(0.5, 0.95), 3) if same_t else 0.0, nq=_log_int(rng, 1, 4096),
                    device=rng.random() < 0.5)
    if kind == "serve":
        return dict(kind=kind, profile="serve", n=_log_int(rng, 50_000, 700_000), t_build=0.5,
                    requests=rng.randint(4, 40), largest=_log_int(rng, 16, 1024), slots=rng.randint(1, 3))
    if kind == "build":
        return dict(kind=kind, profile=rng.choice(["short", "text", "heavy", "flat"]), n=_log_int(rng, 1_000, 400_000),
                    t=round(rng.uniform(0.5, 0.95), 3))
    return dict(kind=kind, profile=rng.choice(["short", "text", "flat"]), n=_log_int(rng, 300, 20_000),
                t=round(rng.uniform(0.5, 0.95), 3))


# ---------------------------------------------------------------- inputs


def _rows(profile, n, seed, popularity_seed=None):
    """(row_ptr, col, val) on the GPU; the popularity order of the dimensions is drawn from popularity_seed."""
    p = PROFILES[profile]
    m = p["m"]
    g = torch.Generator(device="cuda").manual_seed(int(seed) * 2 + 1)
    f64 = dict(dtype=torch.float64, device="cuda")
    if p["sigma"] > 0:
        z = torch.randn(n, generator=g, **f64) * p["sigma"] + (math.log(p["mean"]) - p["sigma"] ** 2 / 2)
        want = torch.exp(z).round().clamp(p["lo"], p["hi"]).to(torch.int64)
    else:
        want = torch.randint(p["lo"], p["hi"] + 1, (n,), generator=g, device="cuda")
    cum = torch.cumsum(torch.arange(1, m + 1, **f64).cpu() ** -p["s"], 0).cuda()
    row_ids = torch.arange(n, device="cuda")
    keys = torch.empty(0, dtype=torch.int64, device="cuda")
    missing = want
    for _ in range(8):  # repeats inside a row are drawn again
        r = torch.repeat_interleave(row_ids, missing)
        if r.numel() == 0:
            break
        k = torch.searchsorted(cum, torch.rand(r.numel(), generator=g, **f64) * cum[-1]).clamp_(max=m - 1)
        keys = torch.unique(torch.cat([keys, r * m + k]))
        missing = want - torch.bincount(keys // m, minlength=n)
    row, k = keys // m, keys % m
    perm_g = torch.Generator(device="cuda").manual_seed(int(seed if popularity_seed is None else popularity_seed) * 2)
    col = torch.randperm(m, generator=perm_g, device="cuda")[k].to(torch.int32)
    rp = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    rp[1:] = torch.cumsum(torch.bincount(row, minlength=n), 0)
    w = torch.exp(torch.randn(keys.numel(), generator=g, **f64))
    sq = torch.zeros(keys.numel() + 1, dtype=torch.int64, device="cuda")  # exact sums, whatever their order
    sq[1:] = torch.cumsum((w * w * 2.0 ** 32).round().to(torch.int64), 0)
    norm = torch.sqrt((sq[rp[1:]] - sq[rp[:-1]]).to(torch.float64) * 2.0 ** -32)
    val = (w / norm[row]).to(torch.float32)
    return rp, col, val


def _queries(case, seed, corpus):
    """Query rows: fresh ones of the corpus's shape, every tenth a perturbed copy of a corpus row."""
    rp, col, val = (x.cpu().numpy() for x in corpus)
    n, nq = case["n"], case["nq"]
    frp, fcol, fval = (x.cpu().numpy() for x in _rows(case["profile"], nq, seed + 7919, seed))
    rng = np.random.default_rng(seed)
    cols, vals, lens = [], [], []
    for q in range(nq):
        if rng.random() < 0.1 or nq == 1:
            r = int(rng.integers(0, n))
            c, v = col[rp[r]:rp[r + 1]], val[rp[r]:rp[r + 1]].astype(np.float64)
            v = v * rng.lognormal(0.0, 0.05, size=len(v))
            v = (v / math.sqrt(float(v @ v))).astype(np.float32)
        else:
            c, v = fcol[frp[q]:frp[q + 1]], fval[frp[q]:frp[q + 1]]
        cols.append(c)
        vals.append(v)
        lens.append(len(c))
    qrp = np.zeros(nq + 1, np.int64)
    np.cumsum(lens, out=qrp[1:])
    tq = None if case["t"] > 0 else rng.uniform(case["t_build"], 0.95, size=nq).astype(np.float32)
    return qrp, np.concatenate(cols), np.concatenate(vals), tq


def _request_sizes(case):
    rng = np.random.default_rng(case["requests"] * 1009 + case["largest"])
    return [int(round(math.exp(rng.uniform(0.0, math.log(case["largest"]))))) for _ in range(case["requests"])]


def _serve_queries(case, seed, corpus):
    sizes = _request_sizes(case)
    qrp, qc, qv, _ = _queries(dict(case, nq=sum(sizes), t=1.0), seed, corpus)
    rng = np.random.default_rng(seed + 23)
    reqs, q = [], 0
    for k in sizes:
        a, b = qrp[q], qrp[q + k]
        reqs.append((k, qrp[q:q + k + 1] - a, qc[a:b], qv[a:b], float(np.float32(rng.uniform(case["t_build"], 0.95)))))
        q += k
    return reqs


def _pair_room(case):
    """Pairs that the program's result buffers hold."""
    kind, n = case["kind"], case["n"]
    nq = sum(_request_sizes(case)) if kind == "serve" else case["nq"] if kind == "query" else n / 2
    t = case["t"] if case.get("t", 0.0) > 0 else case["t_build"]
    room = int(nq + 2e-3 * 10.0 ** (-3.2 * (t - 0.5)) * n * nq + 65_536)
    return min(room, 5_000_000) if case.get("entry") == "noalloc" else room


def _buffers(case):
    """A program's own result arrays (i, j, sim), on the device or the host, zero past the pairs it has."""
    room = _pair_room(case)
    if case["kind"] == "join" or case.get("device"):
        return [torch.zeros(room, dtype=d, device="cuda") for d in (torch.int32, torch.int32, torch.float32)]
    return [np.zeros(room, d) for d in (np.uint32, np.uint32, np.float32)]


def _keep(out, pairs):
    for o, p in zip(out, pairs):
        o[:len(p)] = p
    return out


def prepare(case, seed):
    kind, n = case["kind"], case["n"]
    m = PROFILES[case["profile"]]["m"]
    corpus = _rows(case["profile"], n, seed)
    if kind == "build":
        return dict(case=case, corpus=(n, m) + corpus)
    if kind == "dedupe":
        rp, col, val = (x.cpu().numpy() for x in corpus)
        return dict(case=case, rows=(n, m, rp, col, val), out=_buffers(case))
    if kind == "join":
        opts = {}
        if case["head"]:
            opts = dict(screen_dims=case["head"], variant=2, range_rows=8192, range_group=8)
        if case["entry"] == "graph":
            stream = torch.cuda.Stream()
            torch.cuda.synchronize()
            index = apss.Index.build((n, m) + corpus, case["t"], stream=stream.cuda_stream, graph=True, **opts)
        else:
            stream, index = None, apss.Index.build((n, m) + corpus, case["t"], **opts)
        return dict(case=case, index=index, stream=stream, out=_buffers(case))
    index = apss.Index.build((n, m) + corpus, case["t_build"])
    if kind == "serve":
        server = apss.Server(index, slots=case["slots"], max_batch_queries=4096)
        return dict(case=case, server=server, requests=_serve_queries(case, seed, corpus), out=_buffers(case))
    qrp, qc, qv, tq = _queries(case, seed, corpus)
    if case["device"]:
        qrp, qc, qv = (torch.from_numpy(x).cuda() for x in (qrp, qc, qv))
    return dict(case=case, index=index, q=(qrp, qc, qv), tq=tq, out=_buffers(case))


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "join":
        call = state["index"].join_device_noalloc if case["entry"] == "noalloc" else state["index"].join_device
        return [call(case["t"], *state["out"])] + state["out"]
    if kind == "query":
        h, nq = state["index"].handle, case["nq"]
        if case["device"]:
            return [apss.query_device(h, nq, *state["q"], *state["out"], case["t"], state["tq"])] + state["out"]
        pairs = apss.query(h, nq, *state["q"], case["t"], state["tq"])
        return [len(pairs[0])] + _keep(state["out"], pairs)
    if kind == "serve":
        h = state["server"].handle
        ids = [apss.submit(h, k, rp, col, val, t) for k, rp, col, val, t in state["requests"]]
        got = [apss.poll(h, r) for r in ids]
        return [np.array([len(g[0]) for g in got])] + _keep(state["out"],
                                                            [np.concatenate([g[k] for g in got]) for k in range(3)])
    if kind == "build":
        index = apss.Index.build(state["corpus"], case["t"])
        rank, maxweight, cut = index.export()
        postings = index.sizes()["postings"]
        index.close()
        return dict(rank=rank, maxweight=maxweight, cut=cut, postings=postings)
    n, m, rp, col, val = state["rows"]
    index = apss.Index.build((n, m, torch.from_numpy(rp), torch.from_numpy(col), torch.from_numpy(val)), case["t"])
    pairs = index.join(case["t"])
    index.close()
    return [len(pairs[0])] + _keep(state["out"], pairs)


# ---------------------------------------------------------------- least work and reference values


def _popularity(profile):
    """Expected share of vectors that hold the dimension of each popularity, most popular first."""
    p = PROFILES[profile]
    k = np.arange(1, p["m"] + 1, dtype=np.float64) ** -p["s"]
    lo, hi = 0.0, 1e7
    for _ in range(60):
        mid = (lo + hi) / 2
        lo, hi = (mid, hi) if (1.0 - np.exp(-mid * k)).sum() < p["mean"] else (lo, mid)
    return 1.0 - np.exp(-lo * k)


def work(case):
    """Rows read once and results written once; multiply-adds over the dimensions that a pair of vectors
    shares past the leading part whose norm is below the threshold (the part that no index needs)."""
    p = PROFILES[case["profile"]]
    kind, n, mean = case["kind"], case["n"], p["mean"]
    rows_bytes = n * (8.0 * mean + 8.0)
    if kind == "build":
        return dict(bytes=2.0 * rows_bytes + 12.0 * p["m"], flops=2.0 * n * mean)
    share = _popularity(case["profile"])
    if kind == "serve":
        nq, t = float(sum(_request_sizes(case))), (case["t_build"] + 0.95) / 2
    elif kind == "query":
        nq, t = float(case["nq"]), case["t"] if case["t"] > 0 else (case["t_build"] + 0.95) / 2
    else:
        nq, t = float(n) / 2, case["t"]
    needed = share[np.cumsum(share) > t * t * mean]
    flops = 2.0 * nq * n * float((needed * needed).sum())
    if kind in ("query", "serve"):
        # the lists of the query's own dimensions
        rows_bytes = nq * (8.0 * mean + 8.0) + min(rows_bytes, 8.0 * nq * n * float((needed * needed).sum()))
    return dict(bytes=rows_bytes * (2.0 if kind == "dedupe" else 1.0), flops=flops)


def _all_pairs64(rp, col, val, n, m, t):
    """Pairs i < j with a float64 dot product of at least t, sorted, by dense panels of dimensions."""
    used, col = torch.unique(col.to(torch.int64), return_inverse=True)
    row = torch.repeat_interleave(torch.arange(n, device="cuda"), rp[1:] - rp[:-1])
    sims = torch.zeros(n, n, dtype=torch.float64, device="cuda")
    step = 16_384
    for d0 in range(0, used.numel(), step):
        sel = (col >= d0) & (col < d0 + step)
        panel = torch.zeros(n, step, dtype=torch.float64, device="cuda")
        panel[row[sel], col[sel] - d0] = val[sel].to(torch.float64)
        sims.addmm_(panel, panel.t().contiguous())
    i, j = torch.nonzero(torch.triu(sims >= float(np.float32(t)), diagonal=1), as_tuple=True)
    return i, j, sims[i, j]


def _padded(case, i, j, sims):
    room = _pair_room(case)
    out = [torch.zeros(room, dtype=d, device="cuda") for d in (torch.int64, torch.int64, torch.float64)]
    return [i.numel()] + _keep(out, (i, j, sims))


def exact(case, seed):
    kind, n = case["kind"], case["n"]
    m = PROFILES[case["profile"]]["m"]
    if kind == "serve" or (kind in ("join", "dedupe") and n > 24_000):
        return None
    if kind == "query" and float(case["nq"]) * n > 4e7:
        return None
    rp, col, val = _rows(case["profile"], n, seed)
    if kind == "build":
        mw = torch.zeros(m, dtype=torch.float64, device="cuda")
        mw.scatter_reduce_(0, col.to(torch.int64), val.to(torch.float64), "amax")
        return dict(rank=None, maxweight=mw, cut=None, postings=None)
    if kind in ("join", "dedupe"):
        return _padded(case, *_all_pairs64(rp, col, val, n, m, case["t"]))
    qrp, qc, qv, tq = _queries(case, seed, (rp, col, val))
    nq = case["nq"]
    row = torch.repeat_interleave(torch.arange(n, device="cuda"), rp[1:] - rp[:-1])
    sims = torch.zeros(nq, n, dtype=torch.float64, device="cuda")
    for q in range(nq):
        dense = torch.zeros(m, dtype=torch.float64, device="cuda")
        a, b = int(qrp[q]), int(qrp[q + 1])
        dense[torch.from_numpy(qc[a:b].astype(np.int64)).cuda()] = torch.from_numpy(qv[a:b].astype(np.float64)).cuda()
        sims[q].index_add_(0, row, dense[col.to(torch.int64)] * val)
    limit = np.full(nq, np.float32(case["t"]), np.float32) if tq is None else tq
    i, j = torch.nonzero(sims >= torch.from_numpy(limit.astype(np.float64)).cuda()[:, None], as_tuple=True)
    return _padded(case, i, j, sims[i, j])
