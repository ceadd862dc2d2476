"""Sizes at which the kernels around the list scan change their way: edges of samples, buffers and tiles, the smallest
and the largest of each range, against float64 arithmetic of the same operands."""
import threading

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _hr():
    import paper_2507_09138_amd as hr
    return hr


def _index(N, d, nlist, dtype, seed, tables=False, zipf=0.0):
    """An index of random vectors and the arrays it was made from."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    cent = torch.randn(nlist, d, generator=g, device="cuda")
    w = torch.arange(1, nlist + 1, dtype=torch.float64) ** -zipf
    sizes = torch.floor((N - nlist) * w / w.sum()).long() + 1
    sizes[0] += N - int(sizes.sum())
    off = torch.zeros(nlist + 1, dtype=torch.int64)
    off[1:] = torch.cumsum(sizes, 0)
    vec = torch.randn(N, d, generator=g, device="cuda").to(dtype)
    ids = torch.randperm(N, generator=g, device="cuda")
    return _hr().IvfIndex(cent, off, vec, ids, row_tables=tables), cent, off, vec, ids, g


def _keys(q, x, metric):
    dots = q @ x.T
    return dots if metric == "ip" else 2 * dots - (x * x).sum(1)


@pytest.mark.parametrize("nlist,nprobe,nq", [(256, 64, 3), (257, 1, 5), (257, 256, 5), (1024, 32, 9), (1025, 512, 9), (4096, 1, 65), (4097, 64, 65),
                                             (16384, 512, 70), (16387, 3, 1), (16384, 128, 300)])
@pytest.mark.parametrize("metric", ["ip", "l2"])
def test_coarse_takes_the_closest_centroids(nlist, nprobe, nq, metric):
    """Probe lists against float64 at sizes on both sides of every sample size, with centroids that occur twice."""
    g = torch.Generator(device="cuda")
    g.manual_seed(nlist + nprobe)
    cent = torch.randn(nlist, 64, generator=g, device="cuda")
    cent[nlist // 2:nlist // 2 + nlist // 8] = cent[:nlist // 8]
    off = torch.arange(nlist + 1, dtype=torch.int64)
    vec = torch.randn(nlist, 64, generator=g, device="cuda").half()
    ix = _hr().IvfIndex(cent, off, vec, torch.arange(nlist, device="cuda"))
    q = torch.randn(nq, 64, generator=g, device="cuda")
    probe, _ = ix.coarse(q, nprobe, metric)
    key = _keys(q.double(), cent.double(), metric)
    best = torch.topk(key, nprobe, dim=1).values
    got = key.gather(1, probe.long())
    # float32 sums of 64 products of values near 1, the norms among them: a few 2^-24 of |q|^2 + |x|^2 (below 400)
    assert float((got - best).abs().max()) < 4e-5
    assert all(len(set(p)) == nprobe for p in probe.cpu().tolist())
    # equal centroids: the lower index first (equal scores may be keys that |q|^2 - key rounds to the same value)
    p = probe.cpu().numpy()
    twin = (np.abs(p[:, 1:] - p[:, :-1]) == nlist // 2) & (np.minimum(p[:, 1:], p[:, :-1]) < nlist // 8)
    assert np.all(p[:, 1:][twin] > p[:, :-1][twin])
    _lower_twins_are_there(p, nlist)
    ix.close()


def _lower_twins_are_there(p, nlist):
    """Of two equal centroids (index i and i + nlist/2) the lower one is taken first, at the last place as well."""
    taken = np.zeros((len(p), nlist), dtype=bool)
    np.put_along_axis(taken, p.astype(np.int64), True, axis=1)
    low = np.arange(nlist // 8)
    assert not np.any(taken[:, low + nlist // 2] & ~taken[:, low])


@pytest.mark.parametrize("d", [128, 512, 768, 1024])
@pytest.mark.parametrize("nlist,nprobe,nq", [(64, 17, 300), (100, 33, 1000), (300, 300, 129), (777, 100, 200), (1500, 16, 65), (4099, 128, 700), (2048, 32, 8200)])
def test_coarse_at_the_edges_of_tiles_and_segments(nlist, nprobe, nq, d):
    """Longer vectors: their fragments are addressed and grouped differently, and the work items of the scoring differ in
    rows and queries; odd numbers of lists and queries leave the last of both unfilled."""
    g = torch.Generator(device="cuda")
    g.manual_seed(nlist + nq + d)
    cent = torch.randn(nlist, d, generator=g, device="cuda")
    cent[nlist // 2:nlist // 2 + nlist // 8] = cent[:nlist // 8]
    vec = torch.zeros(nlist, d, dtype=torch.float16, device="cuda")
    ix = _hr().IvfIndex(cent, torch.arange(nlist + 1), vec, torch.arange(nlist, device="cuda"))
    q = torch.randn(nq, d, generator=g, device="cuda")
    probe, score = ix.coarse(q, nprobe, "ip")
    key = _keys(q.double(), cent.double(), "ip")
    best = torch.topk(key, nprobe, dim=1).values
    # float32 sums of d products, |q||x| below 1.5 d: 2^-24 of that for each of a few roundings
    tol = 1.5 * d * 2.0 ** -24 * 8
    assert float((key.gather(1, probe.long()) - best).abs().max()) <= 2 * tol
    assert float((score.double() - key.gather(1, probe.long())).abs().max()) <= tol
    p = probe.cpu().numpy()
    assert all(len(set(r)) == nprobe for r in p.tolist())
    _lower_twins_are_there(p, nlist)
    ix.close()


def _operand(q, storage):
    """The query as the list scan multiplies it (float32 lists: as it is)."""
    if storage == "bf16":
        hi = q.bfloat16().float()
        return hi.double() + (q - hi).bfloat16().double()
    return q.half().double() if storage == "f16" else q.double()


@pytest.mark.parametrize("storage,tables", [("bf16", False), ("f32", True), ("f32", False), ("f16", False)])
@pytest.mark.parametrize("d", [64, 128, 256, 512, 768, 1024])
@pytest.mark.parametrize("nq,k,metric", [(1, 1, "ip"), (15, 100, "l2"), (17, 10, "ip"), (64, 10, "l2"), (65, 128, "ip"), (128, 3, "l2"), (129, 24, "ip"),
                                         (257, 100, "l2")])
def test_scan_finds_the_best_rows_at_the_edges_of_query_tiles(storage, tables, d, nq, k, metric):
    """Every query probes every list, so the buckets are as wide as the batch: on both sides of a wave's columns and of
    a tile's; the lists end in the middle of a block of rows."""
    dtype = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}[storage]
    ix, cent, off, vec, ids, g = _index(2000 + nq, d, 5, dtype, nq + d, tables=tables, zipf=0.7)
    q = torch.randn(nq, d, generator=g, device="cuda")
    found, score = ix.search(q, 5, k, metric)
    op = _operand(q, storage)
    key = _keys(op, vec.double(), metric)
    best = torch.topk(key, k, dim=1).values
    row = torch.empty_like(ids)
    row[ids] = torch.arange(len(ids), device="cuda")
    got = key.gather(1, row[found])
    # sums of d products (and norms) of values near 1 in float32, in chains of at most d/32 steps: 2^-24 of the
    # magnitudes, |q||x| + |x|^2 below 3 d, with room for the steps of a chain
    tol = 3 * d * 2.0 ** -24 * 8
    assert float((got - best).abs().max()) <= 2 * tol
    want = best if metric == "ip" else (op * op).sum(1, keepdim=True) - best
    assert float((score.double() - want).abs().max()) <= 2 * tol
    assert all(len(set(r)) == k for r in found.cpu().tolist())
    ix.close()


@pytest.mark.parametrize("storage,tables", [("bf16", False), ("f32", True), ("f32", False), ("f16", False)])
@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("nq,k,metric", [(3, 5, "l2"), (40, 20, "ip"), (150, 100, "l2")])
def test_scan_of_lists_that_end_around_the_edges_of_blocks(storage, tables, d, nq, k, metric):
    """Short vectors go in blocks of 16 .. 64 rows: lists of one row, and on both sides of every such block and of a few
    of them, the last ones right at the end of the tables."""
    dtype = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}[storage]
    g = torch.Generator(device="cuda")
    g.manual_seed(d + nq)
    sizes = torch.tensor([1, 15, 16, 17, 31, 32, 33, 47, 63, 64, 65, 95, 96, 97, 127, 128, 129, 255, 256, 257, 300, 1])
    nlist, N = len(sizes), int(sizes.sum())
    off = torch.zeros(nlist + 1, dtype=torch.int64)
    off[1:] = torch.cumsum(sizes, 0)
    cent = torch.randn(nlist, d, generator=g, device="cuda")
    vec = torch.randn(N, d, generator=g, device="cuda").to(dtype)
    ix = _hr().IvfIndex(cent, off, vec, torch.arange(N, device="cuda"), row_tables=tables)
    q = torch.randn(nq, d, generator=g, device="cuda")
    op = q.half().double() if storage == "bf16" and tables else _operand(q, storage)
    key = _keys(op, vec.double(), metric)
    for probe in (torch.arange(nlist), torch.tensor([0, 21, 9])):
        rows = torch.cat([torch.arange(int(off[x]), int(off[x + 1])) for x in probe.tolist()]).cuda()
        kk = min(k, len(rows))
        found, score = ix.scan(q, probe.int().cuda().repeat(nq, 1), kk, metric)
        best = torch.topk(key[:, rows], kk, dim=1).values
        got = key.gather(1, found)
        # (as above: sums of d products and norms of values near 1, in chains of at most d / 32 steps)
        tol = 3 * d * 2.0 ** -24 * 8
        assert float((got - best).abs().max()) <= 2 * tol
        assert all(len(set(r)) == kk for r in found.cpu().tolist())
    ix.close()


@pytest.mark.parametrize("nlist,nq,nprobe,N", [(1, 1, 1, 5000), (3, 1, 3, 2000000), (3, 1365, 3, 60000), (256, 64, 16, 65536), (1000, 241, 17, 100000),
                                               (1024, 4096, 1, 40000), (1025, 1, 512, 60000), (4096, 128, 32, 100000), (4097, 128, 32, 100000),
                                               (4095, 9, 455, 50000), (64, 129, 32, 30000), (64, 3000, 48, 30000), (300, 1000, 24, 30000), (16384, 520, 510, 40000)])
def test_grouping_keeps_every_pair_whatever_the_batch(nlist, nq, nprobe, N):
    """Around the largest batch that one workgroup groups alone (4096 pairs, 4096 lists), then with many pairs per list, up to
    the most lists that are counted in LDS; lists that are not in place, probes of nothing, and one list of most of the
    rows; then the counters of the probes."""
    ix, cent, off, vec, ids, g = _index(N, 64, nlist, torch.float16, nlist + nq, zipf=1.3)
    q = torch.randn(nq, 64, generator=g, device="cuda")
    probe = torch.rand(nq, nlist, generator=g, device="cuda").topk(nprobe, dim=1).indices.int()
    away = torch.arange(1, nlist, 7, dtype=torch.int32, device="cuda")
    none = torch.rand(nq, nprobe, generator=g, device="cuda") < 0.1
    probe[none] = -1
    if len(away):
        ix.set_resident(away, False)
    ix.list_hits(reset=True)
    k = 7
    found, score = ix.scan(q, probe, k, "ip")
    hits = torch.bincount(probe[probe >= 0].long(), minlength=nlist)
    assert torch.equal(ix.list_hits().cuda(), hits)
    allowed = torch.zeros(nq, nlist + 1, dtype=torch.bool, device="cuda")
    allowed.scatter_(1, torch.where(probe < 0, nlist, probe.long()), True)
    allowed[:, away.long()] = False
    of_row = torch.repeat_interleave(torch.arange(nlist), off[1:] - off[:-1]).cuda()
    op, row = q.half().float(), torch.empty_like(ids)
    row[ids] = torch.arange(N, device="cuda")
    for i in range(0, nq, 256):
        key = torch.where(allowed[i:i + 256][:, of_row], op[i:i + 256].double() @ vec.double().T, -float("inf"))
        best = torch.topk(key, k, dim=1).values
        f = found[i:i + 256]
        got = torch.where(f >= 0, key.gather(1, row[f.clamp(min=0)]), -float("inf"))
        assert torch.equal(f >= 0, best > -float("inf"))
        ok = f >= 0
        # float32 sums of 64 products of values near 1, |q||x| below 200: 2^-24 of that for each of a few roundings
        assert float((got[ok] - best[ok]).abs().max() if ok.any() else 0.0) < 1e-4
        assert float((score[i:i + 256][ok].double() - best[ok]).abs().max() if ok.any() else 0.0) < 1e-4
    ix.close()


@pytest.mark.parametrize("sizes,nq,nprobe", [([0, 0, 700, 0, 5, 0, 1, 300, 0], 9, 9), ([0] * 5 + [2000] + [0] * 4000, 30, 130), ([3, 0] * 2048, 8, 512),
                                             ([0, 1, 0, 600] * 1100, 8, 512), ([1000] + [0] * 99, 1, 100), ([0] * 64, 5, 64)])
@pytest.mark.parametrize("metric", ["ip", "l2"])
def test_grouping_with_lists_without_rows(sizes, nq, nprobe, metric):
    """Empty lists, at the ends and in rows of them, in batches that one launch groups and (the fourth) that five do: they
    have no work items and share the place of the next list that has."""
    g = torch.Generator(device="cuda")
    g.manual_seed(len(sizes) + nq)
    nlist, N, d, k = len(sizes), sum(sizes), 64, 6
    off = torch.zeros(nlist + 1, dtype=torch.int64)
    off[1:] = torch.cumsum(torch.tensor(sizes), 0)
    cent = torch.randn(nlist, d, generator=g, device="cuda")
    vec = torch.randn(N, d, generator=g, device="cuda").half()
    ix = _hr().IvfIndex(cent, off, vec, torch.arange(N, device="cuda"))
    q = torch.randn(nq, d, generator=g, device="cuda")
    probe = torch.rand(nq, nlist, generator=g, device="cuda").topk(nprobe, dim=1).indices.int()
    found, score = ix.scan(q, probe, k, metric)
    allowed = torch.zeros(nq, nlist, dtype=torch.bool, device="cuda")
    allowed.scatter_(1, probe.long(), True)
    op = q.half().double()
    of_row = torch.repeat_interleave(torch.arange(nlist), off[1:] - off[:-1]).cuda()
    key = torch.cat([torch.where(allowed[:, of_row], _keys(op, vec.double(), metric), -float("inf")),
                     torch.full((nq, k), -float("inf"), device="cuda", dtype=torch.float64)], 1)
    best = torch.topk(key, k, dim=1).values
    assert torch.equal(found >= 0, best > -float("inf"))
    ok = found >= 0
    got = key.gather(1, found.clamp(min=0))
    # float32 sums of 64 products (and norms) of values near 1, |q||x| + |x|^2 below 300: a few 2^-24 of that
    assert float((got - best)[ok].abs().max() if ok.any() else 0.0) < 2e-4
    ix.close()


@pytest.mark.parametrize("order", ["random", "sampled high", "sampled low", "rising", "falling", "equal", "two values"])
@pytest.mark.parametrize("nlist,nprobe", [(300, 100), (300, 300), (512, 512), (777, 300), (1024, 300), (1024, 512), (1025, 512), (2048, 512), (4099, 300),
                                          (16384, 128), (16384, 512), (65536, 16)])
def test_coarse_is_exact_in_whatever_order_the_scores_come(nlist, nprobe, order):
    """Scores that are whole numbers, so every key is exact: in random order, and in orders in which the keys that the
    selection samples (evenly spread places) are all the best or all the worst, or in which many are equal.  The probe
    list is the oracle's, ties included: lower index first."""
    rng = np.random.default_rng(nlist + nprobe)
    value = rng.permutation(nlist)
    size = 1024 if nlist > 4096 else (512 if nlist > 1024 else 256)
    if order.startswith("sampled"):
        at = np.unique(np.arange(size) * nlist // size)
        rest = rng.permutation(np.setdiff1d(np.arange(nlist), at))
        value = np.empty(nlist, dtype=np.int64)
        value[np.concatenate([rest, at] if order.endswith("high") else [at, rest])] = np.arange(nlist)
    elif order in ("rising", "falling"):
        value = np.arange(nlist) if order == "rising" else np.arange(nlist)[::-1]
    elif order == "equal":
        value = np.zeros(nlist, dtype=np.int64)
    elif order == "two values":
        value = (rng.random(nlist) < 0.3).astype(np.int64)
    # (whole numbers below 2^16: a binary16 part and a scaled rest hold 22 bits of a value)
    cent = torch.zeros(nlist, 64, device="cuda")
    cent[:, 0] = torch.from_numpy(np.ascontiguousarray(value)).float().cuda() / 16
    vec = torch.zeros(nlist, 64, dtype=torch.float16, device="cuda")
    ix = _hr().IvfIndex(cent, torch.arange(nlist + 1), vec, torch.arange(nlist, device="cuda"))
    q = torch.zeros(3, 64, device="cuda")
    q[:, 0] = torch.tensor([1.0, -1.0, 2.0])
    probe, score = ix.coarse(q, nprobe, "ip")
    for i, sign in enumerate((1, -1, 2)):
        best = np.lexsort((np.arange(nlist), -sign * value))[:nprobe]
        assert np.array_equal(probe[i].cpu().numpy(), best)
        assert np.array_equal(score[i].cpu().numpy(), (sign * value[best] / 16).astype(np.float32))
    ix.close()


@pytest.mark.parametrize("storage,tables,d,nq,want", [("bf16", False, 64, 128, 512), ("f32", True, 64, 128, 512), ("bf16", False, 64, 64, 256), ("f16", False, 64, 128, 256),
                                                      ("bf16", True, 64, 128, 256), ("bf16", False, 1024, 128, 512), ("bf16", False, 64, 512, 1024)])
def test_segments_are_as_long_as_what_an_item_costs(storage, tables, d, nq, want):
    """Rows per work item where the batch makes about a thousand of them: rows x tiles / 1024, tiles of 64 queries where an
    item multiplies two operands per query, of 128 otherwise."""
    dtype = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}[storage]
    N = 1 << 18
    ix, cent, off, vec, ids, g = _index(N, d, 4, dtype, nq + d, tables=tables)
    q = torch.randn(nq, d, generator=g, device="cuda")
    ix.search(q, 4, 10, "ip")
    torch.cuda.synchronize()
    ws = ix.workspace(nq, 4, 10)
    assert _hr().hr_ivf_stats(ix.handle, ws, ws.numel(), nq, 4, 10)["seg_rows"] == want
    ix.close()


@pytest.mark.parametrize("storage,tables,d,nlist,nq,nprobe,k", [("bf16", False, 64, 64, 256, 48, 100), ("bf16", False, 128, 64, 300, 40, 100), ("f32", True, 64, 64, 200, 64, 128),
                                                                ("bf16", False, 64, 256, 200, 128, 100), ("bf16", False, 64, 256, 192, 128, 128), ("f32", True, 64, 256, 192, 128, 128), ("f16", False, 64, 5000, 700, 20, 5)])
def test_static_search_beyond_the_first_plan(storage, tables, d, nlist, nq, nprobe, k):
    """Batches whose 256 work items do not fit the static array with whole selection buffers: with shorter ones, and, the
    next two, with half the items; then one whose coarse step goes in chunks of an odd number of half tiles.  The same
    results as a search that has a workspace of its own."""
    dtype = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}[storage]
    ix, cent, off, vec, ids, g = _index(100000, d, nlist, dtype, nq, tables=tables, zipf=0.6)
    q = torch.randn(nq, d, generator=g, device="cuda")
    want, ws = ix.search(q, nprobe, k, "ip")
    got = torch.full_like(want, -7)
    score = torch.zeros_like(ws)
    _hr().hr_ivf_search_static(ix.handle, q, nq, nprobe, k, _hr().HR_METRIC_IP, got, score)
    assert torch.equal(got, want) and torch.equal(score, ws)
    ix.close()


@pytest.mark.parametrize("nq", [100, 500, 1024, 1025, 1100, 2100])
@pytest.mark.parametrize("nlist", [4100, 16385])
def test_tiles_of_the_coarse_step_in_groups(nlist, nq):
    """Long items of the scoring, one to eight tiles of queries in a group, groups of unequal size, and, with the static
    array, chunks of queries; every query against float64."""
    d, nprobe = 1024, 24
    ix, cent, off, vec, ids, g = _index(nlist, d, nlist, torch.float16, nq)
    q = torch.randn(nq, d, generator=g, device="cuda")
    probe, score = ix.coarse(q, nprobe, "ip")
    key = q.double() @ cent.double().T
    # float32 sums of d products of values near 1: |q||x| below 1.5 d, a few 2^-24 of that
    tol = 1.5 * d * 2.0 ** -24 * 8
    best = torch.topk(key, nprobe, dim=1).values
    assert float((key.gather(1, probe.long()) - best).abs().max()) <= 2 * tol
    assert float((score.double() - best).abs().max()) <= tol
    want = ix.search(q, nprobe, 4, "ip")
    got = torch.empty_like(want[0]), torch.empty_like(want[1])
    _hr().hr_ivf_search_static(ix.handle, q, nq, nprobe, 4, _hr().HR_METRIC_IP, got[0], got[1])
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    ix.close()


def test_workspace_of_a_small_batch_is_small():
    """Result slots are bounded by the segments that the longest list has, not by the largest batch's alone."""
    ix, *_ = _index(65536, 64, 256, torch.bfloat16, 1)
    assert _hr().hr_ivf_workspace_bytes(ix.handle, 1, 16, 10) < 8 << 20
    sizes = [_hr().hr_ivf_workspace_bytes(ix.handle, n, 16, 10) for n in (1, 2, 63, 64, 65, 128, 1000, 5000)]
    assert sizes == sorted(sizes)                       # (what is enough for a batch is enough for a smaller one)
    ix.close()


@pytest.mark.parametrize("dtype,d,N", [(torch.float16, 768, 65536), (torch.float32, 512, 20000), (torch.bfloat16, 64, 65536)])
def test_workspace_for_many_neighbours_is_enough_for_few(dtype, d, N):
    """Also where few neighbours go in shorter segments: sizes along k, and calls with the workspace of the largest k."""
    hr = _hr()
    ix, cent, off, vec, ids, g = _index(N, d, 64, dtype, d, zipf=1.0)
    for nq, nprobe in ((1, 16), (3, 8), (40, 60)):
        sizes = [hr.hr_ivf_workspace_bytes(ix.handle, nq, nprobe, k) for k in range(1, hr.HR_K_MAX + 1)]
        assert sizes == sorted(sizes)
        q = torch.randn(nq, d, generator=g, device="cuda")
        ws = torch.empty(sizes[24], dtype=torch.uint8, device="cuda")            # (of k = 25)
        for k in (1, 10, 24):
            want = ix.search(q, nprobe, k, "ip")
            got = torch.empty_like(want[0]), torch.empty_like(want[1])
            hr.hr_ivf_search(ix.handle, q, nq, nprobe, k, hr.HR_METRIC_IP, got[0], got[1], ws, ws.numel())
            assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
        probe = torch.empty(nq, nprobe, dtype=torch.int32, device="cuda")
        hr.hr_ivf_coarse(ix.handle, q, nq, nprobe, hr.HR_METRIC_IP, probe, None, ws, ws.numel())
        assert torch.equal(probe, ix.coarse(q, nprobe, "ip")[0])
    ix.close()


@pytest.mark.parametrize("nlist", [1, 15, 16, 17, 1023, 1024, 1025, 2049, 3000])
def test_hot_lists_at_the_edges_of_tiles(nlist):
    """Equal counts on both sides of every tile of counters, and lists that nobody probed."""
    ix, *_ = _index(nlist * 2, 64, nlist, torch.float16, nlist)
    rng = np.random.default_rng(nlist)
    probe = torch.from_numpy(rng.integers(0, max(1, nlist - nlist // 5), (40, min(nlist, 60)))).int().cuda()
    ix.scan(torch.zeros(40, 64, device="cuda"), probe, 1)
    hits = torch.bincount(probe.reshape(-1).long(), minlength=nlist).cpu()
    for gc in {1, (nlist + 1) // 2, nlist}:
        assert torch.equal(ix.hot_lists(gc).cpu(), torch.sort(hits, descending=True, stable=True).indices[:gc].int())
    ix.close()


@pytest.mark.parametrize("k", [1, 20, 64, 65, 128])
@pytest.mark.parametrize("metric", ["ip", "l2"])
def test_merge_by_one_wave_and_by_four(k, metric):
    """1025 queries are merged by a wave each, 1024 by four: the same results, with rows that occur twice (equal keys,
    lower label first), many segments per list, and a carried result with rows that are found again."""
    ix, cent, off, vec, ids, g = _index(60000, 64, 7, torch.float16, k, zipf=0.8)
    vec[30000:] = vec[:30000]
    ix.refresh_rows(0, 60000)
    q = torch.randn(1025, 64, generator=g, device="cuda")
    a, sa = ix.search(q, 7, k, metric)
    b, sb = ix.search(q[:1024], 7, k, metric)
    assert torch.equal(a[:1024], b) and torch.equal(sa[:1024], sb)
    op = q.half().double()
    for i in range(0, 1025, 205):
        best = torch.topk(_keys(op[i:i + 205], vec.double(), metric), k, dim=1).values
        want = best if metric == "ip" else (op[i:i + 205] ** 2).sum(1, keepdim=True) - best
        # float32 sums of 64 products (and norms) of values near 1, |q||x| + |x|^2 below 300: a few 2^-24 of that
        assert float((sa[i:i + 205].double() - want).abs().max()) < 2e-4
    probe = torch.rand(1025, 7, generator=g, device="cuda").topk(6, dim=1).indices.int()
    out = []
    for n in (1025, 1024):
        state = ix.new_state_rows(n, k)
        for part in (probe[:n, :3], probe[:n, 2:]):
            ix.scan_step_rows(q[:n], part.contiguous(), state, metric)
        out.append(state)
    assert all(torch.equal(x[:1024], y) for x, y in zip(*out))
    ix.close()


@pytest.mark.parametrize("m", [1, 3, 4, 5, 16, 17, 64, 65, 128])
@pytest.mark.parametrize("nq,d", [(5, 64), (5, 768), (1024, 128), (1025, 1024)])
@pytest.mark.parametrize("storage,metric", [("f16", "ip"), ("bf16", "l2"), ("f32", "l2")])
def test_rescore_whatever_the_number_of_rows(m, nq, d, storage, metric):
    """Up to four waves per query and one, rows that are listed twice or do not exist, fewer and more places than rows."""
    dtype = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}[storage]
    N, k = 3000, 20
    ix, cent, off, vec, ids, g = _index(N, d, 5, dtype, m + d)
    q = torch.randn(nq, d, generator=g, device="cuda")
    rows = torch.randint(-1, N + 2, (nq, m), generator=g, device="cuda").int()
    if m > 2:
        rows[:, m // 2] = rows[:, 0]
    found, score, at = ix.rescore(q, rows, k, metric)
    op = _operand(q, storage)
    r = rows.long()
    ok = (r >= 0) & (r < N)
    first = torch.tril((r[:, :, None] == r[:, None, :]), -1).any(2)
    ok &= ~first
    x = vec[r.clamp(0, N - 1)].double()
    key = (x * op[:, None, :]).sum(2)
    if metric == "l2":
        key = 2 * key - (x * x).sum(2)
    key = torch.cat([torch.where(ok, key, -float("inf")), torch.full((nq, k), -float("inf"), device="cuda", dtype=torch.float64)], 1)
    best = torch.topk(key, k, dim=1).values
    assert torch.equal(found >= 0, best > -float("inf")) and torch.equal(found >= 0, at >= 0)
    assert torch.equal(torch.where(at >= 0, ids[at.clamp(min=0).long()], -1), found)
    want = best if metric == "ip" else (op * op).sum(1, keepdim=True) - best
    # sums of d products (and norms) of values near 1 in float32, d / 16 of them in a chain: |q||x| + |x|^2 below 3 d
    have = found >= 0
    assert float((score.double() - want)[have].abs().max() if have.any() else 0.0) <= 3 * d * 2.0 ** -24 * 16
    ix.close()


@pytest.mark.parametrize("storage", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("d,nq,nprobe,k", [(512, 1, 7, 10), (768, 1, 40, 24), (768, 1, 3, 25), (1024, 3, 40, 1), (768, 2, 1, 10), (1024, 1, 40, 10)])
def test_small_batches_go_in_shorter_segments(storage, d, nq, nprobe, k):
    """Segments of a few requests: down to 128 KB of rows where every workgroup has one item at most, 256 rows beyond, for
    short vectors and many neighbours; the best rows against float64."""
    dtype = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}[storage]
    ix, cent, off, vec, ids, g = _index(30000, d, 40, dtype, nq + d, zipf=1.0)
    q = torch.randn(nq, d, generator=g, device="cuda")
    probe = torch.rand(nq, 40, generator=g, device="cuda").topk(nprobe, dim=1).indices.int()
    found, score = ix.scan(q, probe, k, "ip")
    torch.cuda.synchronize()
    ws = ix.workspace(nq, nprobe, k)
    seg = _hr().hr_ivf_stats(ix.handle, ws, ws.numel(), nq, nprobe, k)["seg_rows"]
    least = max(64, ((128 << 10) // (d * (4 if storage == "f32" else 2)) + 15) // 16 * 16)
    assert seg >= (least if k <= 24 else 256) and seg % 16 == 0 and (nq * nprobe > 7 or k > 24 or seg < 256)
    of_row = torch.repeat_interleave(torch.arange(40), off[1:] - off[:-1]).cuda()
    allowed = torch.zeros(nq, 40, dtype=torch.bool, device="cuda").scatter_(1, probe.long(), True)
    key = torch.where(allowed[:, of_row], _keys(_operand(q, storage), vec.double(), "ip"), -float("inf"))
    row = torch.empty_like(ids)
    row[ids] = torch.arange(len(ids), device="cuda")
    best = torch.topk(key, k, dim=1).values
    # float32 sums of d products of values near 1 in chains of at most d / 32 steps: |q||x| below 1.5 d
    assert float((key.gather(1, row[found]) - best).abs().max()) <= 1.5 * d * 2.0 ** -24 * 16
    assert float((score.double() - best).abs().max()) <= 1.5 * d * 2.0 ** -24 * 16
    ix.close()


@pytest.mark.parametrize("storage", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("d,nq", [(64, 1), (512, 3), (768, 16), (768, 17), (768, 300), (1024, 20), (128, 3000)])
@pytest.mark.parametrize("metric", ["ip", "l2"])
def test_queries_prepared_with_the_selection_or_before_the_scoring(storage, d, nq, metric):
    """Queries at a 16-byte address and behind one (which the scoring does not load by itself): the same bits, from the
    coarse step alone and from the whole search."""
    dtype = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}[storage]
    ix, cent, off, vec, ids, g = _index(4000, d, 70, dtype, nq + d)
    flat = torch.zeros(nq * d + 8, device="cuda")
    flat[:nq * d] = torch.randn(nq * d, generator=g, device="cuda")
    q = flat[:nq * d].view(nq, d).clone()
    flat[1:nq * d + 1] = q.reshape(-1)
    behind = flat[1:nq * d + 1].view(nq, d)
    assert q.data_ptr() % 16 == 0 and behind.data_ptr() % 16 == 4 and behind.is_contiguous()
    for run in (lambda x: ix.coarse(x, 9, metric), lambda x: ix.search(x, 9, 12, metric)):
        for a, b in zip(run(q), run(behind)):
            assert torch.equal(a, b)
    probe, score = ix.coarse(q, 9, metric)
    key = _keys(q.double(), cent.double(), metric)
    best = torch.topk(key, 9, dim=1).values
    want = best if metric == "ip" else (q.double() ** 2).sum(1, keepdim=True) - best
    # float32 sums of d products and norms of values near 1: |q||x| + |x|^2 + |q|^2 below 4.5 d, a few 2^-24 of that
    assert float((score.double() - want).abs().max()) <= 4.5 * d * 2.0 ** -24 * 8
    ix.close()


@pytest.mark.parametrize("storage,tables", [("f16", False), ("bf16", True), ("f32", False)])
@pytest.mark.parametrize("d,nq,nprobe,k,metric", [(64, 300, 4, 10, "l2"), (128, 257, 3, 24, "ip"), (256, 300, 4, 1, "l2"), (64, 300, 4, 25, "ip")])
def test_full_tiles_of_short_vectors(storage, tables, d, nq, nprobe, k, metric):
    """Batches that put two workgroups on a compute unit (binary16 all but the last, float32 of d = 128), lists that end
    inside a block and a segment."""
    dtype = {"f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}[storage]
    N, nlist = 180011, 4
    ix, cent, off, vec, ids, g = _index(N, d, nlist, dtype, nq + d, tables=tables, zipf=0.4)
    q = torch.randn(nq, d, generator=g, device="cuda")
    probe = torch.rand(nq, nlist, generator=g, device="cuda").topk(nprobe, dim=1).indices.int()
    found, score = ix.scan(q, probe, k, metric)
    allowed = torch.zeros(nq, nlist, dtype=torch.bool, device="cuda").scatter_(1, probe.long(), True)
    of_row = torch.repeat_interleave(torch.arange(nlist), off[1:] - off[:-1]).cuda()
    op, row = (q if storage == "f32" else q.half()).double(), torch.empty_like(ids)
    row[ids] = torch.arange(N, device="cuda")
    for i in range(0, nq, 100):
        key = torch.where(allowed[i:i + 100][:, of_row], _keys(op[i:i + 100], vec.double(), metric), -float("inf"))
        best = torch.topk(key, k, dim=1).values
        # float32 sums of d products (and norms) of values near 1: |q||x| + |x|^2 below 3 d, a few 2^-24 of that
        tol = 3 * d * 2.0 ** -24 * 8
        assert float((key.gather(1, row[found[i:i + 100]]) - best).abs().max()) <= 2 * tol
        want = best if metric == "ip" else (op[i:i + 100] ** 2).sum(1, keepdim=True) - best
        assert float((score[i:i + 100].double() - want).abs().max()) <= 2 * tol
    ix.close()


@pytest.mark.parametrize("storage,tables", [("bf16", True), ("bf16", False), ("f32", True), ("f16", False)])
@pytest.mark.parametrize("d,rows", [(64, 777), (256, 1), (512, 64), (768, 1001), (1024, 3)])
def test_refreshed_rows_are_as_freshly_loaded(storage, tables, d, rows):
    """Squared L2, which reads the norms that the refresh derives again (and the tables): the same bits as from an index
    that is loaded with the new rows, for rows of one to four steps of a wave."""
    dtype = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}[storage]
    ix, cent, off, vec, ids, g = _index(5000, d, 9, dtype, d + rows, tables=tables)
    q = torch.randn(33, d, generator=g, device="cuda")
    before = ix.search(q, 9, 20, "l2")
    vec[1500:1500 + rows] = (0.5 * torch.randn(rows, d, generator=g, device="cuda")).to(dtype)        # (nearer than the others)
    ix.refresh_rows(1500, 1500 + rows)
    got = ix.search(q, 9, 20, "l2")
    fresh = _hr().IvfIndex(cent, off, vec, ids, row_tables=tables)
    want = fresh.search(q, 9, 20, "l2")
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1]) and not torch.equal(got[0], before[0])
    ix.close()
    fresh.close()


@pytest.mark.parametrize("threads", [2, 8, 80])
def test_refreshes_at_the_same_time_report_their_own_rows(threads):
    """bfloat16 rows with a binary16 table, every thread with rows of its own, on several streams: a value beyond binary16 is
    reported by the call that refreshed its row, every time, and by no other (more threads than there are report words, too)."""
    N, each = 16000, 200
    ix, cent, off, vec, ids, g = _index(N, 64, 8, torch.bfloat16, threads, tables=True)
    streams = [torch.cuda.Stream() for _ in range(4)]
    for t in range(1, threads, 2):
        vec[t * each + 7 * t % each, t % 64] = 1.0e6
    torch.cuda.synchronize()
    start, wrong = threading.Barrier(threads), []

    def work(t):
        with torch.cuda.stream(streams[t % len(streams)]):
            start.wait()
            for i in range(40):
                try:
                    ix.refresh_rows(t * each, (t + 1) * each)
                    code = 0
                except _hr().HrError as e:
                    code = e.code
                if code != (-5 if t % 2 else 0):
                    wrong.append((t, i, code))

    pool = [threading.Thread(target=work, args=(t,)) for t in range(threads)]
    for p in pool:
        p.start()
    for p in pool:
        p.join()
    assert not wrong
    ix.close()


@pytest.mark.parametrize("storage", ["f16", "f32"])
@pytest.mark.parametrize("rows,nlist,nq,nprobe", [(4, 300, 2400, 60), (33, 200, 2700, 60), (80, 50, 4000, 30)])
def test_full_tiles_of_short_lists(storage, rows, nlist, nq, nprobe):
    """Two workgroups on a compute unit and lists that are shorter than a block, or end in their second or third one."""
    dtype, d, k = {"f16": torch.float16, "f32": torch.float32}[storage], 128, 9
    ix, cent, off, vec, ids, g = _index(rows * nlist, d, nlist, dtype, nq + rows, zipf=0.3)
    q = torch.randn(nq, d, generator=g, device="cuda")
    probe = torch.rand(nq, nlist, generator=g, device="cuda").topk(nprobe, dim=1).indices.int()
    found, score = ix.scan(q, probe, k, "l2")
    allowed = torch.zeros(nq, nlist, dtype=torch.bool, device="cuda").scatter_(1, probe.long(), True)
    of_row = torch.repeat_interleave(torch.arange(nlist), off[1:] - off[:-1]).cuda()
    op, row = (q if storage == "f32" else q.half()).double(), torch.empty_like(ids)
    row[ids] = torch.arange(len(ids), device="cuda")
    key = torch.where(allowed[:, of_row], _keys(op, vec.double(), "l2"), -float("inf"))
    best = torch.topk(key, k, dim=1).values
    # float32 sums of d products and norms of values near 1: |q||x| + |x|^2 below 3 d, a few 2^-24 of that
    tol = 3 * d * 2.0 ** -24 * 8
    assert float((key.gather(1, row[found]) - best).abs().max()) <= 2 * tol
    assert float((score.double() - ((op ** 2).sum(1, keepdim=True) - best)).abs().max()) <= 2 * tol
    ix.close()


@pytest.mark.parametrize("tables", [False, True])
@pytest.mark.parametrize("d,N,nlist,nq,k,metric", [(64, 900, 3, 3, 1, "ip"), (768, 4000, 4, 5, 10, "l2"), (1024, 3000, 2, 130, 24, "ip"), (512, 2500, 5, 33, 25, "l2"),
                                                   (128, 6000, 2, 40, 64, "ip"), (256, 5000, 2, 20, 100, "l2"), (64, 1500, 4, 1100, 128, "ip"), (768, 700, 3, 1030, 37, "l2"),
                                                   (1024, 300, 6, 1024, 12, "ip"), (768, 90, 2, 7, 128, "l2")])
@pytest.mark.parametrize("spread,scale", [(1e-5, 1.0), (1e-2, 1.0), (1.0, 1e-6), (1e-5, 1e-12)])
def test_float32_rows_that_binary16_cannot_tell_apart(tables, d, N, nlist, nq, k, metric, spread, scale):
    """Rows so close to each other, or so small, that all of them, or many, lie within what rounding to binary16 may have taken:
    selection buffers overflow with them in the scan and in the merge (one wave and four).  As many rows as there are, each once, with
    the scores that float64 gives them, at a spread of 1e-2 and more those of its best (closer rows are as good as equal in float32:
    test_rows_that_differ_by_less_than_binary16_rounds plants what tells them apart).  The queries start at an odd address; a
    carried result goes on being merged exactly."""
    hr = _hr()
    g = torch.Generator(device="cuda")
    g.manual_seed(N + k)
    cent = torch.randn(nlist, d, generator=g, device="cuda") * scale
    off = torch.linspace(0, N, nlist + 1).long()
    base = torch.randn(1, d, generator=g, device="cuda")
    vec = ((base + spread * torch.randn(N, d, generator=g, device="cuda")) * scale).contiguous()
    ids = torch.randperm(N, generator=g, device="cuda")
    ix = hr.IvfIndex(cent, off, vec, ids, row_tables=tables)
    q = (torch.randn(nq * d + 1, generator=g, device="cuda") * scale)[1:].view(nq, d)
    probe = torch.arange(nlist, dtype=torch.int32, device="cuda").repeat(nq, 1)
    found, score = ix.scan(q, probe, k, metric)
    key = _keys(q.double(), vec.double(), metric)
    n = min(k, N)
    best = torch.topk(key, n, dim=1).values
    row = torch.empty_like(ids)
    row[ids] = torch.arange(N, device="cuda")
    assert bool((found[:, :n] >= 0).all()) and bool((found[:, n:] == -1).all())
    # float32 sums of d products in chains of at most d/64 + 6 steps: 2^-24 of |q||x| (+ |x|^2) for each
    size = q.double().norm(dim=1, keepdim=True) * vec.double().norm(dim=1).max() * 2 + (vec.double().norm(dim=1).max() ** 2 if metric == "l2" else 0)
    tol = size * 2.0 ** -24 * 24
    got = key.gather(1, row[found[:, :n]])
    assert bool(((got - best).abs() <= 2 * tol).all())
    qq = (q.double() ** 2).sum(1, keepdim=True)
    want = best if metric == "ip" else (qq - best).clamp(min=0)
    assert bool(((score[:, :n].double() - want).abs() <= 2 * tol + qq * 2.0 ** -22).all())
    assert all(len(set(r)) == n for r in found[:, :n].cpu().tolist())
    # list by list with a carried result
    state = ix.new_state_rows(nq, k)
    for x in range(nlist):
        ix.scan_step_rows(q, probe[:, x:x + 1].contiguous(), state, metric)
    got = key.gather(1, row[state[0][:, :n]])
    assert bool(((got - best).abs() <= 2 * tol + qq * 2.0 ** -22).all())
    ix.close()


@pytest.mark.parametrize("tables", [False, True])
def test_bounds_of_replaced_float32_rows(tables):
    """Rows ten times as long in place of others, in the middle of a list and over the edge of the next: found with the inner
    product, which reads no norms but the bounds."""
    d, N = 256, 4000
    ix, cent, off, vec, ids, g = _index(N, d, 7, torch.float32, 5, tables=tables)
    q = torch.randn(40, d, generator=g, device="cuda")
    for a, b in ((100, 101), (int(off[2]) - 20, int(off[2]) + 3)):
        vec[a:b] = 10 * torch.randn(b - a, d, generator=g, device="cuda")
        ix.refresh_rows(a, b)
        found, score = ix.search(q, 7, 30, "ip")
        best = torch.topk(q.double() @ vec.double().T, 30, dim=1).values
        # 2^-24 of |q||x| below 16 * 160 * 1.3, with room for the steps of the sums
        assert float((score.double() - best).abs().max()) <= 2600 * 2.0 ** -24 * 16
    ix.close()


@pytest.mark.parametrize("storage,d", [("f16", 64), ("bf16", 768), ("f32", 1024)])
@pytest.mark.parametrize("nq,nprobe,nlist", [(1, 1, 7), (1024, 4, 64), (1023, 4, 4096), (8, 512, 512), (1024, 4, 4097), (9, 456, 4096), (1025, 4, 16), (9, 456, 4097)])
def test_seeding_and_grouping_in_one_launch_or_in_two(storage, d, nq, nprobe, nlist):
    """The largest batch that takes the one launch and smaller ones, one more pair, query or list than that, some lists out of
    place: the results of the same queries as part of a larger batch."""
    dtype = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}[storage]
    ix, cent, off, vec, ids, g = _index(9000, d, nlist, dtype, nq + d, zipf=0.6)
    q = torch.randn(nq + 1100, d, generator=g, device="cuda")
    ix.set_resident(torch.arange(0, nlist, 5, dtype=torch.int32, device="cuda"), False)
    probe = torch.rand(nq + 1100, nlist, generator=g, device="cuda").topk(nprobe, dim=1).indices.int()
    probe[::3, 0] = -1
    few = ix.scan(q[:nq], probe[:nq].contiguous(), 10, "l2")
    many = ix.scan(q, probe, 10, "l2")
    assert torch.equal(few[0], many[0][:nq]) and torch.equal(few[1], many[1][:nq])
    ix.close()


def _replaced(N, d, nlist, rows, seed, tables):
    """An index of float32 lists loaded with rows that differ, all of which are replaced afterwards."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    cent = torch.randn(nlist, d, generator=g, device="cuda")
    off = torch.linspace(0, N, nlist + 1).long()
    vec = torch.randn(N, d, generator=g, device="cuda")
    ids = torch.randperm(N, generator=g, device="cuda")
    ix = _hr().IvfIndex(cent, off, vec, ids, row_tables=tables)
    vec.copy_(rows(g))
    ix.refresh_rows(0, N)
    return ix, vec, ids, g


@pytest.mark.parametrize("tables", [False, True])
@pytest.mark.parametrize("d,k,metric", [(64, 10, "ip"), (256, 20, "l2"), (512, 10, "l2"), (768, 10, "ip"), (768, 1, "l2"), (1024, 24, "ip"), (1024, 10, "l2")])
@pytest.mark.parametrize("spread", [1e-5, 1e-4])
@pytest.mark.parametrize("share", [1, 3])
def test_close_float32_rows_are_the_same_bits_in_every_call(tables, d, k, metric, spread, share):
    """Rows so close that buffers overflow with rows whose bounds say nothing, all rows of a list (both parts are multiplied then) or the
    third of it that the queries are closest to: ids and scores must not depend on the batch around a query, on the plan (segments and
    buffers of the static scratch) or on which lists are searched together."""
    hr = _hr()
    nlist, nq = 6, 250
    N = nlist * 1500

    def rows(g):
        base = torch.randn(1, d, generator=g, device="cuda")
        close = base + spread * torch.randn(N, d, generator=g, device="cuda")
        far = torch.randn(N, d, generator=g, device="cuda") - (0.5 if metric == "ip" else 0.0) * base
        return torch.where((torch.arange(N, device="cuda") % 1500 < 1500 // share)[:, None], close, far)

    ix, vec, ids, g = _replaced(N, d, nlist, rows, d + k, tables)
    q = torch.randn(1100, d, generator=g, device="cuda")
    if share > 1:
        q = q + vec[0]
    alone = ix.search(q[:nq], nlist, k, metric)
    for _ in range(3):
        again = ix.search(q[:nq], nlist, k, metric)
        assert torch.equal(again[0], alone[0]) and torch.equal(again[1], alone[1])
    larger = ix.search(q, nlist, k, metric)
    assert torch.equal(larger[0][:nq], alone[0]) and torch.equal(larger[1][:nq], alone[1])
    fixed = torch.empty_like(alone[0]), torch.empty_like(alone[1])
    hr.hr_ivf_search_static(ix.handle, q[:nq], nq, nlist, k, hr.HR_METRIC_IP if metric == "ip" else hr.HR_METRIC_L2, *fixed)
    assert torch.equal(fixed[0], alone[0]) and torch.equal(fixed[1], alone[1])
    if metric == "ip":                                 # (equal scores may be different keys with the other metric)
        found, score = zip(*(ix.scan(q[:nq], torch.full((nq, 1), x, dtype=torch.int32, device="cuda"), k, metric) for x in range(nlist)))
        found, score = torch.cat(found, 1).cpu().numpy(), torch.cat(score, 1).cpu().numpy()
        order = np.lexsort((found, -score), axis=1)[:, :k]
        assert np.array_equal(np.take_along_axis(found, order, 1), alone[0].cpu().numpy())
        assert np.array_equal(np.take_along_axis(score, order, 1), alone[1].cpu().numpy())
    ix.close()


@pytest.mark.parametrize("tables", [False, True])
@pytest.mark.parametrize("d", [64, 768, 1024])
@pytest.mark.parametrize("metric", ["ip", "l2"])
def test_a_long_row_does_not_hide_a_short_one(tables, d, metric):
    """A query's first list holds a long row that is nearly orthogonal to it, so sums of its products differ by more than all that
    bounds the short row of the other list: of the two, searched together, the one with the better score alone is found."""
    nq = 300
    g = torch.Generator(device="cuda")
    g.manual_seed(d)
    q = torch.randn(nq, d, generator=g, device="cuda")
    long = torch.randn(nq, d, generator=g, device="cuda").double() * 2e4
    long = (long - (long * q.double()).sum(1, keepdim=True) / (q.double() ** 2).sum(1, keepdim=True) * q.double()).float()
    size = q.double().norm(dim=1) * long.double().norm(dim=1)
    key = (long.double() * q.double()).sum(1) * (1 if metric == "ip" else 2) - (0 if metric == "ip" else 1) * (long.double() ** 2).sum(1)
    gap = size * torch.tensor([0.0, 1e-9, 4e-9, 1.6e-8, 6.4e-8], dtype=torch.float64, device="cuda").repeat(nq // 5)
    # short row: along the query for the inner product; for the distance as far from it as the long one
    along = ((key + gap) / (q.double() ** 2).sum(1))[:, None] * q.double()
    if metric == "l2":
        far = torch.roll(long.double(), 1, 0)
        far = far - (far * q.double()).sum(1, keepdim=True) / (q.double() ** 2).sum(1, keepdim=True) * q.double()
        along = far / far.norm(dim=1, keepdim=True) * (-key - gap).clamp(min=0).sqrt()[:, None]
    vec = torch.stack([long, along.float()], 1).reshape(2 * nq, d).contiguous()
    ids = torch.randperm(2 * nq, generator=g, device="cuda")
    ix = _hr().IvfIndex(vec, torch.arange(2 * nq + 1), vec, ids, row_tables=tables)
    both = torch.arange(2 * nq, dtype=torch.int32, device="cuda").view(nq, 2)
    single = [ix.scan(q, both[:, x:x + 1].contiguous(), 1, metric) for x in (0, 1)]
    found, score = ix.scan(q, both, 1, metric)
    best = torch.maximum(single[0][1], single[1][1]) if metric == "ip" else torch.minimum(single[0][1], single[1][1])
    assert torch.equal(score, best)
    won = torch.where(single[0][1] == best, single[0][0], single[1][0])
    tie = single[0][1] == single[1][1]
    assert bool((tie | (found == won)).all())
    assert metric == "l2" or bool(((found == single[0][0]).any() and (found == single[1][0]).any()))
    ix.close()


@pytest.mark.parametrize("dtype,d", [(torch.float32, 64), (torch.float32, 1024), (torch.bfloat16, 64)])
@pytest.mark.parametrize("nlist,N,zipf", [(1024, 300000, 0.8), (300, 30000, 0.0), (4096, 300000, 0.3)])
def test_workspace_never_says_less_for_more(dtype, d, nlist, N, zipf):
    """More neighbours, more queries and more probes, also where the tiles of queries change their width; a search of fewer with
    that workspace is not refused."""
    hr = _hr()
    ix, cent, off, vec, ids, g = _index(N, d, nlist, dtype, d, zipf=zipf)
    size = lambda nq, nprobe, k: hr.hr_ivf_workspace_bytes(ix.handle, nq, nprobe, k)
    for nq, nprobe in ((1, 16), (100, 33), (1024, 32), (3000, 64)):
        sizes = [size(nq, nprobe, k) for k in range(1, hr.HR_K_MAX + 1)]
        assert sizes == sorted(sizes)
    for k in (10, 13, 20, 30, 100):
        for nprobe in (1, 16, 128):
            edge = 48 * nlist // nprobe
            sizes = [size(nq, nprobe, k) for nq in (edge // 2, edge - 1, edge, edge + 1, edge + 2, edge + edge // 3, 2 * edge)]
            assert sizes == sorted(sizes)
        for nq in (500, 48 * nlist // 64):
            sizes = [size(nq, nprobe, k) for nprobe in (1, 2, 16, 63, 64, 65, 100, 128, 256)]
            assert sizes == sorted(sizes)
    # (the coarse step takes the plan of one neighbour: it must stay inside the regions of any other)
    assert len({tuple(map(tuple, hr.hr_ivf_workspace_layout(ix.handle, 1024, 32, k)[:-2])) for k in (1, 12, 13, 30, 100)}) == 1
    q = torch.randn(1024, d, generator=g, device="cuda")
    ws = torch.empty(size(1024, 32, 20), dtype=torch.uint8, device="cuda")
    for nq, k in ((1024, 10), (1024, 13), (700, 20)):
        out = torch.empty(nq, k, dtype=torch.int64, device="cuda"), torch.empty(nq, k, device="cuda")
        hr.hr_ivf_search(ix.handle, q[:nq], nq, 32, k, hr.HR_METRIC_IP, *out, ws, ws.numel())
        want = ix.search(q[:nq], 32, k, "ip")
        assert torch.equal(out[0], want[0]) and torch.equal(out[1], want[1])
    ix.close()


@pytest.mark.parametrize("nq", [1, 8, 60])
def test_small_batches_never_go_in_longer_segments(nq):
    """Float32 rows of d = 1024, many neighbours: the segments of a small batch are no longer than those of a large one."""
    ix, cent, off, vec, ids, g = _index(48000, 1024, 60, torch.float32, 3)
    rows = []
    for n in (nq, 700):
        q = torch.randn(n, 1024, generator=g, device="cuda")
        ix.search(q, 8, 30, "ip")
        torch.cuda.synchronize()
        ws = ix.workspace(n, 8, 30)
        rows.append(_hr().hr_ivf_stats(ix.handle, ws, ws.numel(), n, 8, 30)["seg_rows"])
    assert rows[0] <= rows[1]
    ix.close()


@pytest.mark.parametrize("tables", [False, True])
def test_a_replaced_long_row_does_not_slow_its_list_for_good(tables):
    """Every list once held a row a thousand times as long: once all its rows are replaced, searches take as long as before, and the
    lists at the edges of a range and the empty ones keep bounds that hold."""
    d, nlist, N = 128, 64, 64000
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    cent = torch.randn(nlist, d, generator=g, device="cuda")
    off = torch.linspace(0, N, nlist + 1).long()
    off[7:10] = off[7]                                  # two lists without rows
    good = torch.randn(N, d, generator=g, device="cuda")
    vec = good.clone()
    ix = _hr().IvfIndex(cent, off, vec, torch.arange(N, device="cuda"), row_tables=tables)
    q = torch.randn(512, d, generator=g, device="cuda")

    def took():
        spans = []
        for _ in range(7):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(5):
                out = ix.search(q, 32, 10, "ip")
            b.record()
            b.synchronize()
            spans.append(a.elapsed_time(b))
        return min(spans), out

    before, want = took()
    vec[::500] *= 1000
    ix.refresh_rows(0, N)
    took()
    vec.copy_(good)
    ix.refresh_rows(0, N)
    after, got = took()
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    assert after < 2 * before
    # parts of lists at both ends of the range, each of which has held longer rows
    for a, b in ((int(off[3]) + 5, int(off[11]) - 5), (int(off[6]), int(off[10])), (int(off[7]), int(off[7]) + 1)):
        vec[a:b] = 30 * torch.randn(b - a, d, generator=g, device="cuda")
        ix.refresh_rows(a, b)
        found, score = ix.search(q, 64, 20, "ip")
        best = torch.topk(q.double() @ vec.double().T, 20, dim=1).values
        # |q||x| below 16 * 16 * 30 * 1.4, a few 2^-24 of it
        assert float((score.double() - best).abs().max()) <= 11000 * 2.0 ** -24 * 16
    ix.close()


def _split_and_not(N, d, nlist, seed, tables, zipf=0.0, scale=1.0, hole=None):
    """Two indexes of the same float32 rows: one that was loaded with them, and one that was loaded with rows which differ by less than
    rounding takes from them and has had no list replaced in one call since, so that it multiplies both parts of the rows."""
    hr = _hr()
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    cent = torch.randn(nlist, d, generator=g, device="cuda")
    w = torch.arange(1, nlist + 1, dtype=torch.float64) ** -zipf
    sizes = torch.floor((N - nlist) * w / w.sum()).long() + 1
    if hole is not None:
        sizes[hole] = 0
    sizes[0] += N - int(sizes.sum())
    off = torch.zeros(nlist + 1, dtype=torch.int64)
    off[1:] = torch.cumsum(sizes, 0)
    good = scale * torch.randn(N, d, generator=g, device="cuda")
    ids = torch.randperm(N, generator=g, device="cuda")
    vec = (1 + 1e-5 * torch.randn(N, d, generator=g, device="cuda")).contiguous()
    split = hr.IvfIndex(cent, off, vec, ids, row_tables=tables)
    vec.copy_(good)
    ends = [0, *((off[:-1] + off[1:]) // 2).tolist(), N]
    for at, end in zip(ends[:-1], ends[1:]):
        split.refresh_rows(at, end)
    torch.cuda.synchronize()
    return hr.IvfIndex(cent, off, good, ids, row_tables=tables), split, off, good, ids, g


@pytest.mark.parametrize("d", [64, 128, 256, 512, 768, 1024])
@pytest.mark.parametrize("N,nlist,nq,nprobe,k,zipf,scale", [(9000, 40, 1, 7, 10, 1.0, 1.0), (20011, 37, 333, 11, 1, 0.7, 1.0), (3000, 300, 65, 40, 100, 0.3, 100.0), (40000, 20, 1030, 9, 24, 0.5, 1.0),
                                                            (15000, 25, 129, 25, 13, 1.2, 1e-3), (700, 9, 17, 5, 128, 0.9, 1e-6), (5000, 60, 2000, 8, 50, 0.4, 1.0)])
@pytest.mark.parametrize("metric", ["ip", "l2"])
def test_both_parts_of_float32_rows_give_the_same_bits(d, N, nlist, nq, nprobe, k, zipf, scale, metric):
    """Every call that scans float32 lists, by their high parts or by both: odd sizes, empty lists, lists out of place, probes that are
    none, carried results, the static scratch; the best rows against float64."""
    hr = _hr()
    a, b, off, vec, ids, g = _split_and_not(N, d, nlist, N + d, nq % 2 == 0, zipf, scale, hole=nlist // 2)
    q = scale * torch.randn(nq, d, generator=g, device="cuda")
    out = torch.tensor([1, nlist - 2], dtype=torch.int32, device="cuda")
    probe = torch.rand(nq, nlist, generator=g, device="cuda").topk(nprobe, dim=1).indices.int()
    probe[::5, 1] = -1
    for x in (a, b):
        x.set_resident(out, False)
    results = []
    for x in (a, b):
        state = x.new_state_rows(nq, k)
        for part in (probe[:, :2], probe[:, 2:]):
            x.scan_step_rows(q, part.contiguous(), state, metric)
        fixed = torch.empty(min(nq, 40), k, dtype=torch.int64, device="cuda"), torch.empty(min(nq, 40), k, device="cuda")
        hr.hr_ivf_search_static(x.handle, q[:40].contiguous(), min(nq, 40), nprobe, k, hr.HR_METRIC_IP if metric == "ip" else hr.HR_METRIC_L2, *fixed)
        results.append([*x.search(q, nprobe, k, metric), *x.scan(q, probe, k, metric), *state, *fixed])
    for u, v in zip(*results):
        assert torch.equal(u, v)
    found, score = results[0][2:4]
    allowed = torch.zeros(nq, nlist + 1, dtype=torch.bool, device="cuda").scatter_(1, torch.where(probe < 0, nlist, probe).long(), True)[:, :nlist]
    allowed[:, out.long()] = False
    of_row = torch.repeat_interleave(torch.arange(nlist), off[1:] - off[:-1]).cuda()
    key = torch.where(allowed[:, of_row], _keys(q.double(), vec.double(), metric), -float("inf"))
    best = torch.topk(key, min(k, N), dim=1).values
    got = found[:, :best.shape[1]]
    assert torch.equal(got >= 0, best > -float("inf"))
    row = torch.empty_like(ids)
    row[ids] = torch.arange(N, device="cuda")
    mine = torch.where(got >= 0, key.gather(1, row[got.clamp(min=0)]), best)
    # float32 sums of d products in chains of at most d/64 + 6 steps and a norm: 2^-24 of |q||x| (+ |x|^2) for each
    size = q.double().norm(dim=1, keepdim=True) * vec.double().norm(dim=1).max() * 2 + (vec.double().norm(dim=1).max() ** 2 if metric == "l2" else 0)
    assert bool(((mine - best).abs().nan_to_num(0.0) <= size * 2.0 ** -24 * 24).all())
    a.close()
    b.close()


def test_both_parts_are_multiplied_where_bounds_tell_little():
    """What the loader and hr_ivf_refresh_rows make of rows, read from the number of work items: at d = 1024 a tile holds 128 queries, of
    which both parts are multiplied 64."""
    hr = _hr()
    d, N, nq = 1024, 600, 128
    g = torch.Generator(device="cuda")
    g.manual_seed(4)
    base, noise = torch.randn(1, d, generator=g, device="cuda"), torch.randn(N, d, generator=g, device="cuda")
    q = torch.randn(nq, d, generator=g, device="cuda")

    def tiles(ix, metric, rows=N):
        ix.scan(q, torch.zeros(nq, 1, dtype=torch.int32, device="cuda"), 10, metric)
        torch.cuda.synchronize()
        ws = ix.workspace(nq, 1, 10)
        s = hr.hr_ivf_stats(ix.handle, ws, ws.numel(), nq, 1, 10)
        return s["items"] // ((rows + s["seg_rows"] - 1) // s["seg_rows"])

    def load(rows, off=(0, N)):
        return hr.IvfIndex(base.expand(len(off) - 1, d).contiguous(), torch.tensor(off), rows.contiguous(), torch.arange(len(rows), device="cuda"))

    # windows of 0.02 and 0.03 deviations; 0.24 and 1.2; 3.6 and 270; an offset that all have; equal rows (both parts tell no more); rows of zeros
    for rows, ip, l2 in ((noise, 1, 1), (base + 0.15 * noise, 1, 2), (base + 0.01 * noise, 2, 2), (noise * 0.05 + 10, 2, 2), (base.expand(N, d), 1, 1), (0 * noise, 1, 1)):
        ix = load(rows)
        assert (tiles(ix, "ip"), tiles(ix, "l2")) == (ip, l2)
        ix.close()
    # a row a thousand times as long; rows that are replaced later, one of them or all
    long = noise.clone()
    long[7] *= 1000
    ix = load(long)
    assert (tiles(ix, "ip"), tiles(ix, "l2")) == (2, 2)
    ix.close()
    for before, a, b, rows, want in ((noise, 7, 8, long, 2), (noise, 0, N, base + 0.01 * noise, 2), (0 * noise, 0, N, noise, 1), (noise, 0, N, 2 * noise, 1)):
        vec = before.clone()
        ix = load(vec)
        vec[a:b] = rows[a:b]
        ix.refresh_rows(a, b)
        torch.cuda.synchronize()
        assert (tiles(ix, "ip"), tiles(ix, "l2")) == (want, want)
        ix.close()
    # lists that come and go: parts of them change nothing, nor fewer rows than a 64th
    def replaced(ix, vec, a, b, rows):
        vec[a:b] = rows[a:b]
        ix.refresh_rows(a, b)
        torch.cuda.synchronize()
        return tiles(ix, "ip"), tiles(ix, "l2")

    close = base + 0.01 * noise
    vec = close.clone()
    ix = load(vec)
    assert replaced(ix, vec, 0, N // 2, noise) == (2, 2) and replaced(ix, vec, N // 2, N, noise) == (2, 2)
    assert replaced(ix, vec, 0, N, noise) == (1, 1) and replaced(ix, vec, 0, N, close) == (2, 2) and replaced(ix, vec, 0, N, noise) == (1, 1)
    ix.close()
    # (a list of 600 rows, 400, 300 and the rest: 786 rows are a 64th)
    at = [0, N, N + 400, N + 700, 50300]
    many = torch.randn(at[-1], d, generator=g, device="cuda")
    near = base + 0.01 * many[:at[3]]
    vec = many.clone()
    ix = load(vec, at)
    assert replaced(ix, vec, 0, N, near) == (2, 2)
    assert replaced(ix, vec, 0, N, many) == (2, 2) and replaced(ix, vec, N, at[2], many) == (1, 1)
    assert replaced(ix, vec, 0, N, near) == (2, 2)
    assert replaced(ix, vec, 0, N, many) == (2, 2) and replaced(ix, vec, N, at[2], near) == (2, 2)
    assert replaced(ix, vec, N, at[2], many) == (2, 2) and replaced(ix, vec, at[2], at[3], many) == (2, 2) and replaced(ix, vec, 0, N, many) == (1, 1)
    ix.close()
    # rows as long as each other: one list in a hundred whose window is a little wide (1.0 deviations) does not count, one in fifty does; one
    # of 4 always
    for lists, step, want in ((100, 0.163, 1), (50, 0.163, 2), (100, 0.08, 2)):
        rows = torch.randn(64 * lists, d, generator=g, device="cuda")
        rows[-64:] = 32 * torch.nn.functional.normalize(base + step * rows[-64:], dim=1)
        ix = load(rows, list(range(0, 64 * lists + 1, 64)))
        assert tiles(ix, "ip", 64) == want
        ix.close()


@pytest.mark.parametrize("tables", [False, True])
@pytest.mark.parametrize("share", [1, 3])
@pytest.mark.parametrize("d,nq,k,metric", [(64, 3, 1, "ip"), (768, 5, 10, "l2"), (1024, 130, 24, "ip"), (512, 33, 25, "l2"), (128, 40, 64, "ip"), (256, 20, 100, "l2"), (768, 1100, 128, "ip"),
                                           (1024, 1030, 37, "l2")])
def test_rows_that_differ_by_less_than_binary16_rounds(tables, share, d, nq, k, metric):
    """Rows that are all the same in binary16 and differ along the queries by a thousand times what float32 sums may be off: the best of
    them are found, whether they are all of a list (both parts are multiplied) or the third of it that the queries are closest to
    (every one of them is within what the bounds leave, in the scan and in the merge); also list by list with a carried result."""
    hr = _hr()
    nlist, N = 4, 6000
    g = torch.Generator(device="cuda")
    g.manual_seed(d + k)
    base = (1.1 + 0.4 * torch.rand(1, d, generator=g, device="cuda")).half().float()        # (steps of 2^-10: rounding takes up to 2^-11)
    along = torch.randint(0, 2, (1, d), generator=g, device="cuda").float() * 2 - 1
    step = torch.rand(N, 1, generator=g, device="cuda") * 2.0 ** -11.5
    vec = base + step * along
    close = torch.arange(N, device="cuda") % (N // nlist) < N // nlist // share
    vec = torch.where(close[:, None], vec, -base + torch.randn(N, d, generator=g, device="cuda")).contiguous()
    assert torch.equal(vec[close].half().float(), base.expand(int(close.sum()), d))
    ids = torch.randperm(N, generator=g, device="cuda")
    ix = hr.IvfIndex(base.expand(nlist, d).contiguous(), torch.linspace(0, N, nlist + 1).long(), vec, ids, row_tables=tables)
    q = base + along * (0.5 + torch.rand(nq, 1, generator=g, device="cuda"))
    probe = torch.arange(nlist, dtype=torch.int32, device="cuda").repeat(nq, 1)
    key = _keys(q.double(), vec.double(), metric)
    best = torch.topk(key, k, dim=1).values
    row = torch.empty_like(ids)
    row[ids] = torch.arange(N, device="cuda")
    # float32 sums of d products in chains of at most d/64 + 6 steps, and a norm: 2^-24 of |q||x| (+ |x|^2) for each
    size = q.double().norm(dim=1, keepdim=True) * vec.double().norm(dim=1).max() * 2 + (vec.double().norm(dim=1).max() ** 2 if metric == "l2" else 0)
    tol = 2 * size * 2.0 ** -24 * (d / 64 + 6)
    some = key[:, close][:, torch.randint(0, int(close.sum()), (k,), generator=g, device="cuda")].sort(dim=1, descending=True).values
    assert bool(((some - best).abs().max(1, keepdim=True).values > 4 * tol).all())       # (any k of the close rows would not do)
    state = ix.new_state_rows(nq, k)
    for x in range(nlist):
        ix.scan_step_rows(q, probe[:, x:x + 1].contiguous(), state, metric)
    for found, score in (ix.search(q, nlist, k, metric), ix.scan(q, probe, k, metric), state[:2]):
        assert bool(((key.gather(1, row[found]) - best).abs() <= tol).all())
        want = best if metric == "ip" else (q.double() ** 2).sum(1, keepdim=True) - best
        assert bool(((score.double() - want).abs() <= 2 * tol).all())
        assert all(len(set(r)) == k for r in found.cpu().tolist())
    ix.close()
