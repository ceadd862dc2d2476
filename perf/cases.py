"""Performance cases: the calls a retrieval service makes of this library, from one request to its largest batches.

A case is a plain dict.  ``op`` says which public entry points one pass goes through:

  search   IvfIndex.search: coarse step, grouping, list scan, merge (the whole retrieval of a batch)
  static   hr_ivf_search_static: the same for a caller that cannot allocate (small batches of a serving loop)
  coarse   IvfIndex.coarse: the nprobe closest centroids alone
  reuse    the next hop of multi-hop requests: coarse step, the cached rows of the previous hop rescored, their lists
           looked up, the probe lists reordered, then the lists searched in sub-stages with a carried result
  swap     partial residency: counters read, lists swapped out and in, the new rows' derived data refreshed, the
           probes split, the lists in place searched

The index of every case is what the paper's corpora look like to the library: unit vectors (inner product) or raw ones
(squared L2) scattered around the centroids of their lists, list sizes uniform or Zipf, the queries drawn near
centroids that are chosen uniformly, by popularity (Zipf) or by list size; labels are a permutation.  Everything is
made on the GPU from the seed alone.
"""
import numpy as np
import torch

import paper_2507_09138_amd as hr

DTYPE = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
NOISE, DRIFT = 0.3, 0.05          # spread of vectors around their centroid, step of a query from one hop to the next
CARRIED = 20                      # entries a multi-hop request carries and caches
STAGES = 4                        # sub-stages of its search


def _case(name, op, N, d, nlist, zipf, storage, metric, nq, pick, nprobe, k, tables=False):
    c = dict(op=op, N=N, d=d, nlist=nlist, zipf=zipf, storage=storage, metric=metric, nq=nq, pick=pick, nprobe=nprobe, k=k,
             tables=tables)
    return dict(c, name=name) if name else c


def listed():
    return [
        # one user's question against a small corpus, from a loop that cannot allocate: latency and launches
        _case("one request", "static", 65536, 768, 256, 1.0, "f32", "ip", 1, "uniform", 16, 10),
        # a small batch against the same corpus
        _case("small batch", "search", 65536, 768, 256, 1.0, "f32", "ip", 64, "uniform", 16, 10),
        # odd sizes throughout, short vectors, few neighbours
        _case("ragged d128", "search", 1000003, 128, 1000, 0.8, "f16", "l2", 777, "size", 33, 7),
        # uncompressed vectors of a mid-sized corpus, plain and with the row tables that the loader offers
        _case("f32 lists", "search", 1048576, 768, 1024, 0.0, "f32", "ip", 1024, "uniform", 32, 10),
        _case("f32 lists, tables", "search", 1048576, 768, 1024, 0.0, "f32", "ip", 1024, "uniform", 32, 10, True),
        # the benchmark's own batch: skewed lists, skewed popularity
        _case("popular lists", "search", 4194304, 768, 4096, 1.1, "f16", "ip", 4096, "zipf", 64, 10),
        # one hop of multi-hop requests: few queries per list
        _case("one hop", "search", 4194304, 768, 4096, 1.1, "f16", "ip", 512, "uniform", 32, 10),
        # the next hop of the same requests, searched in sub-stages from the cached rows of the hop before
        _case("next hop, sub-stages", "reuse", 4194304, 768, 4096, 1.1, "f16", "ip", 512, "uniform", 32, 10),
        # the largest batch: 16.8 M bfloat16 vectors, squared L2, 100 neighbours
        _case("large batch, k 100", "search", 16777216, 768, 16384, 1.05, "bf16", "l2", 8192, "size", 128, 100),
        # a passage corpus of 1024-dimensional embeddings, the best passage of each request, many lists probed
        _case("passages d1024", "search", 12582912, 1024, 4096, 0.5, "f16", "ip", 256, "size", 128, 1),
        # routing only: the closest of many centroids for an odd number of queries
        _case("centroids only", "coarse", 1048576, 768, 16384, 1.05, "bf16", "l2", 3001, "size", 128, 1),
        # hot lists in place, some swapped in between two batches (bfloat16 with its binary16 row table)
        _case("swap lists in", "swap", 2097152, 512, 2048, 1.0, "bf16", "ip", 256, "zipf", 24, 20, True),
    ]


def _spread(rng, lo, hi):
    """A whole number whose logarithm is uniform between those of lo and hi."""
    return int(round(float(np.exp(rng.uniform(np.log(lo), np.log(hi))))))


def draw(rng):
    op = rng.choice(["search"] * 6 + ["static", "coarse", "reuse", "swap"])
    storage = rng.choice(["f16", "bf16", "f32"])
    d = rng.choice([64, 128, 256, 512, 768, 768, 1024])
    row = d * (4 if storage == "f32" else 2)
    nlist = _spread(rng, 64, 16384)
    N = max(nlist * 40, min(_spread(rng, 60e6, 9e9) // row, nlist * 3000))
    tables = storage != "f16" and rng.random() < 0.3
    metric = rng.choice(["ip", "l2"])
    zipf = rng.choice([0.0, 0.5, 0.8, 1.0, 1.1])
    pick = rng.choice(["uniform", "zipf", "size"])
    nq, nprobe, k = _spread(rng, 1, 8192), _spread(rng, 4, min(512, nlist // 2)), _spread(rng, 1, 128)
    if op == "static":
        nq, nprobe, k, nlist = min(nq, 1 + nq % 64), min(nprobe, 32), min(k, 20), min(nlist, 4096)
        N = min(N, nlist * 3000)
    if op == "reuse":
        nprobe, k, nq = max(STAGES, nprobe // STAGES * STAGES), min(k, CARRIED), min(nq, 2048)
    if op == "swap":
        nq = min(nq, 2048)
    c = _case("", op, N, d, nlist, zipf, storage, metric, nq, pick, nprobe, k, tables)
    while work(c)["flops"] > 2.0e12:
        c["nq"] = max(1, c["nq"] // 2 - 1)
    return c


# ---- what a pass cannot do without


def _sizes(case):
    """List sizes by rank, largest first: they sum to N and none is empty."""
    n, w = case["nlist"], np.arange(1, case["nlist"] + 1, dtype=np.float64) ** -case["zipf"]
    sizes = 1 + np.floor((case["N"] - n) * w / w.sum()).astype(np.int64)
    sizes[0] += case["N"] - sizes.sum()
    return sizes


def _chance(case, sizes):
    """Probability by rank that a query's own cluster is that list."""
    w = {"uniform": np.ones(len(sizes)), "size": sizes.astype(np.float64), "zipf": np.arange(1, len(sizes) + 1) ** -max(case["zipf"], 0.5)}[case["pick"]]
    return w / w.sum()


def _scan_work(case, nprobe, own=True):
    """(bytes of the rows of all lists that somebody probes, flops) with the own cluster among the probed lists or not;
    the other lists of a query are as good as random."""
    sizes, nq, d = _sizes(case), case["nq"], case["d"]
    p = _chance(case, sizes) if own else np.zeros(len(sizes))
    others = (nprobe - (1 if own else 0)) / case["nlist"]
    rows = float((sizes * (1 - (1 - p) ** nq * (1 - others) ** nq)).sum())
    pairs = nq * (float((sizes * p).sum()) + others * case["N"])
    es = 4 if case["storage"] == "f32" else 2
    return rows * (d * es + (4 if case["metric"] == "l2" else 0)), 2.0 * d * pairs


def work(case):
    nq, d, k, nlist, nprobe = (case[x] for x in ("nq", "d", "k", "nlist", "nprobe"))
    es = 4 if case["storage"] == "f32" else 2
    b, f = nq * d * 4.0 + nlist * d * 4.0, 2.0 * nq * nlist * d             # queries and centroids, coarse scores
    if case["op"] == "coarse":
        return {"bytes": b + nq * nprobe * 8, "flops": f}
    if case["op"] == "reuse":
        b, f = b + nq * CARRIED * (d * es + 4 * 16.0) + nq * nprobe * 12, f + 2.0 * nq * CARRIED * d
        for s in range(STAGES):
            sb, sf = _scan_work(case, nprobe // STAGES, own=s == 0)
            b, f = b + sb + nq * CARRIED * 32, f + sf
        return {"bytes": b, "flops": f}
    sb, sf = _scan_work(case, nprobe)
    if case["op"] == "swap":
        part = int(_sizes(case)[_moved(case)].sum())
        share = 1.0 - _cold(case) / nlist                                   # (the cold lists are the shortest: close to all rows)
        b += part * d * es * (2 if case["tables"] else 1) + part * 4 + nlist * 24 + nq * nprobe * 12
        sb, sf = sb * share, sf * share
    return {"bytes": b + sb + nq * k * 12, "flops": f + sf}


def tolerance(case):
    # Products of the operands as the storage type rounds them, summed in float32 in some order.  Measured against 64-bit
    # sums of the same operands, and against the same search with the dimensions permuted: inner product 2e-7 (largest
    # 8e-7), squared L2 1.3e-6 (largest 8e-6: a difference of terms near 1); neighbours closer than that trade places,
    # 7e-4 of the ids for 10 or 20 of them and 5e-3 for 100.
    rel, most = (1e-6, 4e-6) if case["metric"] == "ip" else (5e-6, 4e-5)
    return {"rel": rel, "max": most, "differ": min(1e-2, 3e-3 + 1e-4 * case["k"])}


# ---- inputs


def _arrays(case, g):
    dev, N, d, nlist = g.device, case["N"], case["d"], case["nlist"]
    unit = case["metric"] == "ip"
    cent = torch.nn.functional.normalize(torch.randn(nlist, d, generator=g, device=dev), dim=1)
    sizes = _sizes(case)
    rank_to_list = torch.randperm(nlist, generator=g, device=dev)
    by_list = torch.empty(nlist, dtype=torch.int64, device=dev)
    by_list[rank_to_list] = torch.from_numpy(sizes).to(dev)
    offsets = torch.zeros(nlist + 1, dtype=torch.int64, device=dev)
    offsets[1:] = torch.cumsum(by_list, 0)
    row_list = torch.repeat_interleave(torch.arange(nlist, device=dev), by_list, output_size=N)
    vectors = torch.empty(N, d, dtype=DTYPE[case["storage"]], device=dev)
    step = max(1, (1 << 28) // d)
    for r in range(0, N, step):
        x = torch.randn(min(step, N - r), d, generator=g, device=dev).mul_(NOISE / d ** 0.5).add_(cent[row_list[r:r + step]])
        vectors[r:r + step] = torch.nn.functional.normalize(x, dim=1) if unit else x
    ids = torch.randperm(N, generator=g, device=dev)
    return cent, offsets, vectors, ids, rank_to_list, torch.from_numpy(_chance(case, sizes)).to(dev)


def _queries(case, cent, rank_to_list, chance, g):
    """The batch of queries and, for multi-hop requests, those of the hop after it (else None)."""
    own = rank_to_list[torch.multinomial(chance, case["nq"], replacement=True, generator=g)]

    def near(x, spread):
        y = x + torch.randn(x.shape, generator=g, device=g.device) * (spread / case["d"] ** 0.5)
        return torch.nn.functional.normalize(y, dim=1) if case["metric"] == "ip" else y

    q = near(cent[own], NOISE)
    return q, near(q, DRIFT) if case["op"] == "reuse" else None


def _cold(case):
    return case["nlist"] // 4             # lists that are not in place (the shortest)


def _moved(case):
    """Ranks of the lists that are swapped in: up to eight from the middle of the size ranking."""
    n = case["nlist"]
    return slice(n // 2, n // 2 + max(1, min(8, n // 16)))


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def prepare(case, seed):
    g = _generator(seed)
    cent, offsets, vectors, ids, rank_to_list, chance = _arrays(case, g)
    index = hr.IvfIndex(cent, offsets.cpu(), vectors, ids, row_tables=case["tables"])
    nq, k, nlist = case["nq"], case["k"], case["nlist"]
    queries, after = _queries(case, cent, rank_to_list, chance, g)
    s = dict(case=case, index=index, queries=queries)
    if case["op"] == "static":
        s["ids"] = torch.empty(nq, k, dtype=torch.int64, device=g.device)
        s["scores"] = torch.empty(nq, k, dtype=torch.float32, device=g.device)
    if case["op"] == "reuse":
        # the hop before this one: its probe lists and its carried result
        s["probed"], _ = index.coarse(s["queries"], case["nprobe"], case["metric"])
        state = index.new_state_rows(nq, CARRIED)
        index.scan_step_rows(s["queries"], s["probed"], state, case["metric"])
        s["cached_rows"] = state[2]
        s["queries"] = after
    if case["op"] == "swap":
        s["into"] = rank_to_list[_moved(case)].to(torch.int32)
        s["out"] = rank_to_list[nlist - _cold(case):].to(torch.int32)
        host = offsets.cpu()
        s["ranges"] = sorted((int(host[x]), int(host[x + 1])) for x in s["into"].cpu().tolist())
        index.set_resident(s["out"], False)
        _swap_batch(s)                    # (one batch has been counted when a pass reads the counters)
    return s


def _swap_batch(s):
    case, index = s["case"], s["index"]
    probe, _ = index.coarse(s["queries"], case["nprobe"], case["metric"])
    here, missing = index.split_probes(probe)
    return (here, missing) + index.scan(s["queries"], here, case["k"], case["metric"])


# ---- one pass


def run(s):
    case, index, q = s["case"], s["index"], s["queries"]
    if case["op"] == "search":
        return index.search(q, case["nprobe"], case["k"], case["metric"])
    if case["op"] == "static":
        metric = hr.HR_METRIC_IP if case["metric"] == "ip" else hr.HR_METRIC_L2
        hr.hr_ivf_search_static(index.handle, q, case["nq"], case["nprobe"], case["k"], metric, s["ids"], s["scores"])
        return s["ids"], s["scores"]
    if case["op"] == "coarse":
        return index.coarse(q, case["nprobe"], case["metric"])
    if case["op"] == "reuse":
        probe, _ = index.coarse(q, case["nprobe"], case["metric"])
        hot = index.lists_of_rows(s["cached_rows"][:, :case["k"]])
        order = hr.reorder_probes(probe, s["probed"], hot)
        state = index.rescore(q, s["cached_rows"], CARRIED, case["metric"])
        per = case["nprobe"] // STAGES
        for j in range(STAGES):
            index.scan_step_rows(q, order[:, j * per:(j + 1) * per].contiguous(), state, case["metric"])
        return probe, order, state
    hot = index.hot_lists(case["nlist"] // 2)
    hits = index.list_hits(reset=True)
    index.set_resident(s["out"], False)
    index.set_resident(s["into"], True)
    for a, b in s["ranges"]:
        index.refresh_rows(a, b)
    return (hot, hits) + _swap_batch(s)


# ---- the same outputs in 64 bits


def _operand(case, q):
    """Queries as the list scan multiplies them: rounded to binary16 with binary16 rows, bfloat16 pairs with bfloat16 ones."""
    if case["storage"] == "f16" or (case["storage"] == "bf16" and case["tables"]):
        return q.half().double()
    if case["storage"] == "bf16":
        hi = q.bfloat16().float()
        return hi.double() + (q - hi).bfloat16().double()
    return q.double()


def _keys(case, q, rows):
    """Larger is better: inner products, or minus the squared distances; both arguments in 64 bits."""
    dots = q @ rows.T
    return dots if case["metric"] == "ip" else 2 * dots - (q * q).sum(1)[:, None] - (rows * rows).sum(1)


def _closest(case, cent, q):
    key, probe = torch.topk(_keys(case, q.double(), cent.double()), case["nprobe"], dim=1)
    return probe, key if case["metric"] == "ip" else -key


def _best(case, offsets, vectors, ids, q, probe, k):
    """The k best rows of every query's probed lists (a probe of -1 is none): labels, scores, row numbers."""
    nq, nprobe = probe.shape
    op, host = _operand(case, q), offsets.tolist()
    key = torch.full((nq * nprobe, k), -float("inf"), dtype=torch.float64, device=q.device)
    row = torch.full((nq * nprobe, k), -1, dtype=torch.int64, device=q.device)
    by_list, pair = torch.sort(probe.reshape(-1), stable=True)
    ends = torch.searchsorted(by_list, torch.arange(-1, case["nlist"], device=q.device), right=True).tolist()
    for x in range(case["nlist"]):
        at = pair[ends[x]:ends[x + 1]]
        a, b = host[x], host[x + 1]
        for part in torch.split(at, max(1, (1 << 28) // (b - a))) if len(at) else ():
            top = torch.topk(_keys(case, op[part // nprobe], vectors[a:b].double()), min(k, b - a), dim=1)
            key[part, :min(k, b - a)] = top.values
            row[part, :min(k, b - a)] = torch.where(top.values > -float("inf"), top.indices + a, -1)
    key, at = torch.topk(key.view(nq, nprobe * k), k, dim=1)
    row = row.view(nq, nprobe * k).gather(1, at)
    return torch.where(row >= 0, ids[row.clamp(min=0)], -1), key if case["metric"] == "ip" else -key, row


def exact(case, seed):
    g = _generator(seed)
    cent, offsets, vectors, ids, rank_to_list, chance = _arrays(case, g)
    q, after = _queries(case, cent, rank_to_list, chance, g)
    if case["op"] == "reuse":
        # (a row that the hop before returned is a candidate whether its list is probed again or not)
        cached = _best(case, offsets, vectors, ids, q, _closest(case, cent, q)[0], CARRIED)[2]
        found = _best(case, offsets, vectors, ids, after, _closest(case, cent, after)[0], CARRIED)[2]
        row = torch.cat([found, torch.where((cached[:, :, None] == found[:, None, :]).any(2), -1, cached)], 1)
        op = _operand(case, after)
        key = torch.stack([_keys(case, op[i:i + 1], vectors[row[i].clamp(min=0)].double())[0] for i in range(case["nq"])])
        key = torch.topk(torch.where(row >= 0, key, -float("inf")), CARRIED, dim=1).values
        return None, None, (None, key if case["metric"] == "ip" else -key, None)
    probe, score = _closest(case, cent, q)
    if case["op"] == "coarse":
        return probe.int(), score
    if case["op"] == "swap":
        cold = torch.zeros(case["nlist"], dtype=torch.bool, device=q.device)
        cold[rank_to_list[case["nlist"] - _cold(case):]] = True
        cold[rank_to_list[_moved(case)]] = False
        probe = torch.where(cold[probe], -1, probe)
        return (None,) * 4 + _best(case, offsets, vectors, ids, q, probe, case["k"])[:2]
    return _best(case, offsets, vectors, ids, q, probe, case["k"])[:2]
