"""Edges of single kernels and of the rules that choose between them: tile remainders, the smallest and
largest sizes of a path, and the sizes on both sides of a dispatch."""
import math
import time

import numpy as np
import pytest
import torch

from gpu_util import Pair, dev, make_pair, route
from paper_2602_21477_amd import binding as B
from paper_2602_21477_amd import workload as W

pytestmark = pytest.mark.gpu
IP, L2, F32, F16 = B.PK_METRIC_IP, B.PK_METRIC_L2, B.PK_F32, B.PK_F16


@pytest.mark.parametrize("storage,metric,d,page,k,nprobe,cap", [
    (F32, IP, 128, 0, 10, 8, 64), (F16, L2, 100, 96, 10, 16, 300), (F32, L2, 33, 32, 1, 3, 16), (F16, IP, 200, 128, 90, 64, 1000)])
def test_overflowed_queries_of_a_larger_batch_are_scored_again(gpu_device, storage, metric, d, page, k, nprobe, cap):
    """More than 128 queries: those whose region overflows are scored again under the threshold their kept
    keys give, as many as there are regions for; the others are rescored one by one.  Either way the rows equal
    those of regions that hold everything, bit for bit."""
    cfg = W.scaled(W.C1, n=9001, d=d)
    p, _ = make_pair(cfg, metric=metric, storage=storage, insert_reserve=512, page_vecs=page)
    try:
        p.gpu.insert(dev(W.inserts(cfg, 0, 200)))
        for nq in (129, 260):
            q = dev(W.queries(cfg, 30, nq))
            want_i, want_v = p.gpu.search(q, k, nprobe)
            for c in (cap, 16):
                B.pk_index_set_emit_cap(p.gpu.handle, c)
                B.pk_profile_begin(p.gpu.handle)
                got_i, got_v = p.gpu.search(q, k, nprobe)
                pr = B.pk_profile_end(p.gpu.handle)
                B.pk_index_set_emit_cap(p.gpu.handle, 0)
                assert pr.overflowed > 0 or k == 1
                assert torch.equal(got_i, want_i) and torch.equal(got_v, want_v)
        assert p.gpu.stats().device_error == 0
    finally:
        p.close()


def test_tie_groups_of_queries_that_are_scored_again(gpu_device):
    """Copies of one row under scrambled ids, fewer and more than a rescue region holds (4096)."""
    rng = np.random.default_rng(5)
    for copies in (600, 5000):
        x = rng.standard_normal((9000, 40)).astype(np.float32)
        x /= np.linalg.norm(x, axis=1, keepdims=True)
        dup = rng.permutation(len(x))[:copies]
        x[dup] = x[dup[0]]
        ids = rng.permutation(len(x)).astype(np.int64) + 9
        p = Pair(x, x[rng.permutation(len(x))[:8]].copy(), IP, F32, ids=ids)
        try:
            q = rng.standard_normal((150, 40)).astype(np.float32)
            q[::60] = x[dup[0]]
            B.pk_index_set_emit_cap(p.gpu.handle, 128)
            gi, gv = p.gpu.search(dev(q), 20, 8)
            assert gi[0].tolist() == sorted(ids[dup].tolist())[:20]
            B.pk_index_set_emit_cap(p.gpu.handle, 0)
            wi, wv = p.gpu.search(dev(q), 20, 8)
            assert torch.equal(gi, wi) and torch.equal(gv, wv)
        finally:
            p.close()


def rows_by_split_gemm(n, nlist):
    """How many of a build's rows the split GEMM takes: chunks of 16384 always fill 128 tiles of 128 x 128, a tail may not."""
    tail = n % 16384
    return n if tail == 0 or -(-tail // 128) * -(-nlist // 128) >= 128 else n - tail


@pytest.mark.parametrize("metric", [IP, L2])
@pytest.mark.parametrize("n,d,nlist,scale,gemm", [
    (1, 1, 1, 1.0, 0), (63, 64, 33, 1.0, 0), (65, 100, 64, 1e-9, 0), (257, 1536, 255, 1e12, 0),
    (4097, 33, 700, 1.0, 4097), (40000, 96, 513, 1e-20, 40000), (16384, 1, 1, 1.0, 16384), (16384 + 63, 64, 33, 1.0, 16384),
    (16384 + 65, 100, 64, 1e-9, 16384), (32768, 1536, 255, 1e12, 32768), (33000, 1500, 300, 1e-9, 32768), (5000, 70, 513, 1e12, 5000)])
def test_split_operand_assignment_is_within_fp32_of_64_bits(gpu_device, n, d, nlist, scale, gemm, metric):
    """Rows and centroids held as two halfs each, in the three tile sizes of the kernel, with remainders in every
    direction and rows whose scale is far from 1; tails too short for it go to the centroid kernel, which keeps the same
    bound.  A row may only go to a list whose score is as good as the best to fp32 rounding: the split's own error is
    below 2^-22 of |x||c|, the accumulation's below K * 2^-24 of it."""
    assert rows_by_split_gemm(n, nlist) == gemm
    rng = np.random.default_rng(n + d)
    x = (rng.standard_normal((n, d)) * np.exp(rng.standard_normal((n, 1)))).astype(np.float32)
    cent = rng.standard_normal((nlist, d)).astype(np.float32)
    x[:: 7, : d // 2] *= 1e-4  # elements that are tiny beside the row's largest
    x, cent = x * np.float32(scale), cent * np.float32(scale)
    ix = B.Index(dev(cent), dev(x), metric=metric)
    try:
        where = np.full(n, -1)
        for l, m in enumerate(ix.list_lengths()):
            if m:
                where[ix.list_ids(l).cpu().numpy()] = l
        assert (where >= 0).all()
        x64, c64 = x.astype(np.float64), cent.astype(np.float64)
        s = x64 @ c64.T
        if metric == L2:
            s = 2 * s - (c64 ** 2).sum(1)
        size = np.linalg.norm(x64, axis=1) * np.linalg.norm(c64, axis=1).max()
        if metric == L2:
            size = size + (x64 ** 2).sum(1) + (c64 ** 2).sum(1).max()
        gap = s.max(1) - s[np.arange(n), where]
        assert (gap <= (2.0 ** -21 + d * 2.0 ** -23) * size).all(), (gap / size).max()
    finally:
        ix.close()


def lists_of(ix, n):
    """The list of each of the ids 0 .. n - 1, every one of which is in exactly one list."""
    where, found = np.full(n, -1), 0
    for l in np.nonzero(ix.list_lengths())[0]:
        ids = ix.list_ids(int(l)).cpu().numpy()
        where[ids] = l
        found += len(ids)
    assert found == n and (where >= 0).all()
    return where


def by_first_halves(n, d, nlist):
    """Whether a build's (or k-means') assignment begins with the products of the first halves alone: many products, or
    chunks of large rows."""
    row = -(-d // 64) * 256
    return n * -(-nlist // 32) * 32 * (row // 4) >= 1.5e10 or min(n, 32768) * row > 64 << 20


@pytest.mark.parametrize("metric", [IP, L2])
@pytest.mark.parametrize("nlist,kind,d", [(33, "plain", 48), (200, "plain", 48), (513, "plain", 48), (33, "huge", 48), (513, "huge", 48), (65, "nan", 48),
                                          (1, "plain", 48), (33, "plain", 600), (513, "plain", 600), (513, "huge", 600), (65, "nan", 600)])
def test_rows_without_a_comparable_score_go_to_some_list(gpu_device, nlist, kind, d, metric):
    """Rows and centroids with NaN, infinities and values whose products overflow, in all three tile sizes of the
    assignment, with lists that do not fill their tiles: every row ends up in a list that exists, the rows beside it in
    their own.  (d = 600: by the first halves' products to begin with.)"""
    rng = np.random.default_rng(nlist)
    n = 32768 + 16384  # a chunk of each size: 256 x 256 (513 lists) or 128 x 128 tiles, then smaller ones
    x = rng.standard_normal((n, d)).astype(np.float32)
    cent = rng.standard_normal((nlist, d)).astype(np.float32)
    odd = np.arange(0, n, 997)
    for i, r in enumerate(odd):
        x[r, i % d] = [np.nan, np.inf, -np.inf, 3e38, 1e25, -np.nan][i % 6]
    if kind == "huge":
        cent[rng.permutation(nlist)[: nlist // 2 + 1]] *= np.float32(1e33)
    if kind == "nan":
        cent[3, 2], cent[nlist - 1, 0] = np.nan, np.inf
    ix = B.Index(dev(cent), dev(x), metric=metric, insert_reserve=20000)
    try:
        where = lists_of(ix, n)
        if kind == "plain":
            fine = np.setdiff1d(np.arange(n), odd)
            s = x[fine].astype(np.float64) @ cent.astype(np.float64).T
            if metric == L2:
                s = 2 * s - (cent.astype(np.float64) ** 2).sum(1)
            # fp32 rounding of sums of 48 products, as in the tests below (of 600: by the root of their number more)
            assert (s.max(1) - s[np.arange(len(fine)), where[fine]] <= 1e-5 * math.sqrt(d / 48) * (1 + np.abs(s).max(1))).all()
        assert by_first_halves(n, d, nlist) == (d == 600)
        lists = ix.insert(dev(x[:8192]), want_lists=True).cpu().numpy()
        assert ((lists >= 0) & (lists < nlist)).all()
        assert ix.stats().device_error == 0 and ix.stats().n_total == n + 8192
        assert ix.list_lengths().sum() == n + 8192
    finally:
        ix.close()
    if metric == L2:
        assign = torch.empty(n, dtype=torch.int32, device="cuda")
        B.pk_kmeans(dev(x), dev(cent), 1, assign)
        assert int(assign.min()) >= 0 and int(assign.max()) < nlist


@pytest.mark.parametrize("metric,storage,d", [(IP, F32, 100), (L2, F16, 64)])
def test_probes_of_near_tied_lists_do_not_depend_on_the_call(gpu_device, metric, storage, d):
    """Centroids in pairs that differ in the last bits, and one probe, so that rounding decides which of a pair is
    searched: one handle's search, the same segment in a call over two handles, and a search of the probes that the
    coarse step gives alone have the same rows, bit for bit."""
    g = torch.Generator(device="cuda").manual_seed(d)
    half, n, nq, nprobe = 1030, 400000, 1024, 1

    def around(m):
        at = torch.randint(half, (m,), device="cuda", generator=g)
        return c[at] + 0.5 * torch.randn((m, d), device="cuda", generator=g)

    c = torch.randn((half, d), device="cuda", generator=g)
    cent = torch.cat([c, c * (1 + torch.randint(-2, 3, c.shape, device="cuda", generator=g) * 2.0 ** -23)])
    x, q = around(n), around(nq + 70)
    a, b = B.Index(cent, x, metric=metric, storage=storage), B.Index(cent, x, metric=metric, storage=storage)
    try:
        ids, dist = a.search(q[:nq], 10, nprobe)
        mi, md = B.search_multi([a, b], [0, nq, nq + 70], q, 10, nprobe)
        assert torch.equal(ids, mi[:nq]) and torch.equal(dist, md[:nq])
        ci, cd = a.scan_probes(q[:nq], 10, a.coarse(q[:nq], nprobe))
        assert torch.equal(ids, ci) and torch.equal(dist, cd)
    finally:
        a.close()
        b.close()


def near_pairs(d, half, apart, seed, every=1):
    """Centroids in pairs `apart` lists from each other, and a source of rows around them.  Those of one pair in `every`
    differ in the last bits."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    c = torch.randn((half, d), device="cuda", generator=g)
    twin = c * (1 + torch.randint(-2, 3, c.shape, device="cuda", generator=g) * 2.0 ** -23)
    cent = torch.empty((2 * half, d), device="cuda")
    at = torch.arange(half, device="cuda")
    at = at // apart * (2 * apart) + at % apart  # blocks of `apart` centroids (a divisor of half), each followed by its twins
    twin = torch.where(at[:, None] % every == 0, twin, torch.randn((half, d), device="cuda", generator=g))
    cent[at], cent[at + apart] = c, twin

    def around(m):
        return c[torch.randint(half, (m,), device="cuda", generator=g)] + 0.5 * torch.randn((m, d), device="cuda", generator=g)

    return cent, around


@pytest.mark.parametrize("n,metric,d,half,apart,every", [
    (16384, IP, 100, 128, 1, 1),  # every row is a near tie: large tiles of listed rows
    (16384, L2, 64, 130, 130, 1),  # ... of lists in different tiles
    (2 * 32768 + 16384 + 70, IP, 33, 96, 32, 1),  # ... found out in the first chunk, a last one that fills no tiles
    (2 * 32768 + 5, L2, 128, 300, 300, 1),
    (32768 + 16384, L2, 100, 192, 1, 3),  # one in three: the second chunk takes the split GEMM, too
    (16384, IP, 64, 512, 512, 200),  # a few hundred rows: small tiles of listed rows
    (16384 + 3, L2, 36, 600, 600, 150),
    (2 * 32768 + 16384 + 70, IP, 520, 96, 32, 1),  # after the first halves: every row a near tie, found out in the first chunk
    (32768 + 16384, L2, 600, 192, 1, 3)])  # ... one in three
def test_near_tied_rows_of_a_build_go_where_the_fp32_scores_say(gpu_device, n, metric, d, half, apart, every):
    """Centroids that differ in the last bits of their scores: the lists are those of the fp32 coarse step, row for row."""
    cent, around = near_pairs(d, half, apart, n + d, every)
    x = around(n)
    ix = B.Index(cent, x, metric=metric)
    try:
        where = torch.from_numpy(lists_of(ix, n))
        want = torch.cat([ix.coarse(x[i:i + 16384].contiguous(), 1)[:, 0].cpu() for i in range(0, n, 16384)])
        assert torch.equal(where, want.long())
    finally:
        ix.close()
    if metric == L2:
        assign = torch.empty(n, dtype=torch.int32, device="cuda")
        B.pk_kmeans(x, cent.clone(), 1, assign)
        assert torch.equal(assign.cpu(), want)


@pytest.mark.parametrize("n,metric,d,half,apart,every", [
    (32768, IP, 600, 40, 1, 1),  # 128 x 128 tiles that the lists do not fill
    (5 * 32768 + 5, IP, 64, 960, 960, 3),  # two steps
    (32768 + 16384 + 3, L2, 600, 130, 130, 1),  # the rule: the second chunk goes to all three products at once; odd rows
    (2 * 32768 + 5, IP, 603, 300, 300, 4),  # one in four: the first halves' kernel goes on; rows that are not aligned
    (65536, L2, 1536, 512, 1, 8),  # 256 x 256 tiles, the longest rows
    (16384, L2, 1300, 16, 4, 2),  # 64 x 64 tiles
    (16384, IP, 64, 40, 1, 1), (32768 + 16384 + 3, L2, 200, 130, 130, 1), (2 * 32768 + 5, IP, 33, 300, 300, 4)])  # small sets: all three products of every row
def test_rows_that_first_halves_cannot_tell_apart_go_where_the_fp32_scores_say(gpu_device, n, metric, d, half, apart, every):
    """Pairs of centroids that differ by 2^-11 of their elements: less than the first halves leave out, far more than
    what fp32 sums are off by.  The lists are those of the fp32 coarse step, row for row."""
    assert by_first_halves(n, d, 2 * half) == ((n, d) not in ((16384, 64), (32768 + 16384 + 3, 200), (2 * 32768 + 5, 33)))
    cent, around = near_pairs(d, half, apart, n + d, every)
    g = torch.Generator(device="cuda").manual_seed(d)
    cent *= 1 + torch.randint(-1, 2, cent.shape, device="cuda", generator=g) * 2.0 ** -11
    x = around(n)
    ix = B.Index(cent, x, metric=metric)
    try:
        where = torch.from_numpy(lists_of(ix, n))
        # (chunks that the GEMM scores; a shorter last one takes the centroid kernel in both)
        want = torch.cat([ix.coarse(x[i:i + 16384].contiguous(), 1)[:, 0].cpu() for i in range(0, n, 16384)])
        assert torch.equal(where, want.long())
    finally:
        ix.close()


@pytest.mark.parametrize("metric,d,half,apart", [(IP, 128, 128, 1), (L2, 100, 130, 130), (L2, 64, 256, 64), (IP, 33, 1100, 1100), (IP, 1536, 130, 130), (L2, 1024, 150, 1)])
def test_near_tied_vectors_go_to_the_same_lists_in_inserts_of_any_size(gpu_device, metric, d, half, apart):
    """Every vector has two lists that differ in the last bits of their scores, in one tile or in two: an insert large
    enough for the split GEMM takes the ones that inserts of 64 (fp32 throughout) and calls over handles take."""
    cent, around = near_pairs(d, half, apart, half)
    x = around(4097)
    a, b, c = (B.Index(cent, None, metric=metric, insert_reserve=9000) for _ in range(3))
    try:
        large = a.insert(x, want_lists=True)
        small = torch.cat([b.insert(x[i:i + 64].contiguous(), want_lists=True) for i in range(0, len(x), 64)])
        n = len(x) if d < 1024 else 4096  # (the last one comes alone: eight waves add up its long products, in another order)
        assert torch.equal(large[:n], small[:n])
        if 8 * ((2 * half + 127) // 128) < 128:  # (with more lists, segments of 1000 take their scores from the fp32 GEMM)
            multi = torch.empty(2000, dtype=torch.int32, device="cuda")
            B.pk_insert_multi([b.handle, c.handle], [0, 1000, 2000], x[:2000].contiguous(), None, multi)
            assert torch.equal(multi, small[:2000])
    finally:
        for ix in (a, b, c):
            ix.close()


@pytest.mark.parametrize("nq,storage,metric,d", [(1024, F16, L2, 100), (1024, F32, IP, 128), (999, F32, L2, 70), (128, F16, IP, 64)])
def test_searches_whose_coarse_step_is_a_gemm(gpu_device, nq, storage, metric, d):
    """Batches with 128 tiles or more of 128 x 128 scores, against the oracle; both copies of a half-precision memory's
    queries are made in one pass."""
    cfg = W.scaled(W.C1, n=20000, d=d, nlist=16384 if nq == 128 else 2050, ncomp=64, train="lloyd", train_iters=0)
    rng = np.random.default_rng(d)
    x = W.vectors(cfg, 0, cfg.n)
    p = Pair(x, x[rng.permutation(len(x))[:cfg.nlist]].copy(), metric, storage)
    try:
        q = W.queries(cfg, 1, nq)
        some = np.sort(rng.permutation(nq)[:40])
        gi, gv = p.gpu.search(dev(q), 10, 16)
        # a row does not depend on the batch around it: a few rows again, through the other coarse kernel
        probes = p.gpu.coarse(dev(q), 16).cpu().numpy()
        fi, fv = p.gpu.scan_probes(dev(q[some]), 10, dev(probes[some]))
        assert torch.equal(gi[some.tolist()], fi) and torch.equal(gv[some.tolist()], fv)
        op, sc = p.orc.coarse(q[some], 17, with_scores=True)
        assert np.mean(op[:, :16] == probes[some]) > 0.99
        p.check_scan(q[some], 10, probes[some], where="gemm")
    finally:
        p.close()


@pytest.mark.parametrize("n,d,storage,metric,nq,page", [
    (300_000, 700, F32, IP, 60, 0),  # the kernel that holds whole query groups
    (150_000, 1500, F32, L2, 40, 96),  # the kernel that stages slices of them
    (600_000, 680, F16, L2, 60, 64), (300_000, 1500, F16, IP, 250, 0)])
def test_rows_of_large_memories_are_read_a_line_at_a_time(gpu_device, n, d, storage, metric, nq, page):
    """More than 768 MB of rows and a call that reads more than 256 MB of them: whole lines, past the caches, moved into
    place between lanes.  A query alone reads less and its rows the other way: the same results, bit for bit."""
    nlist, nprobe = 512, 24
    g = torch.Generator(device="cuda").manual_seed(d)
    x = torch.randn((n, d), device="cuda", generator=g)
    cent = x[torch.randperm(n, device="cuda", generator=g)[:nlist]].contiguous()
    width = (d * (2 if storage == F16 else 4) + 255) // 256 * 256
    assert n * width > 768 << 20 and nq * nprobe * n / nlist * width > 256 << 20 > nprobe * n / nlist * width
    q = x[:nq] + 0.3 * torch.randn((nq, d), device="cuda", generator=g)
    ix = B.Index(cent, x, metric=metric, storage=storage, page_vecs=page)
    del x
    try:
        probes = ix.coarse(q, nprobe)  # (one probe list: a near tie may fall either way in the two kernels' coarse steps)
        ids, dist = ix.scan_probes(q, 10, probes)
        for i in list(range(0, nq, 7)) + [nq - 1]:
            one_ids, one_dist = ix.scan_probes(q[i:i + 1].contiguous(), 10, probes[i:i + 1].contiguous())
            assert torch.equal(one_ids[0], ids[i]) and torch.equal(one_dist[0], dist[i]), i
        assert ids[:, 0].tolist() == list(range(nq)) or metric == IP  # (the row a query was made from is its nearest)
    finally:
        ix.close()


def test_overflowed_queries_of_calls_over_handles_and_beside_the_rows_in_registers_kernel(gpu_device):
    """Queries that are scored again belong to either of two handles; and in a batch whose busiest lists go to the kernel
    that counts no candidates, beside the scan that does: the rows of regions that hold everything, bit for bit."""
    pairs = [make_pair(W.scaled(W.C1, n=n, d=96), agent=a, metric=IP, storage=F16)[0] for a, n in enumerate((9001, 7000))]
    cfg = W.scaled(W.C1, n=30000, ncomp=96, nlist=96)
    hot, _ = make_pair(cfg, metric=L2, storage=F16)
    try:
        q = torch.cat([dev(W.queries(W.scaled(W.C1, d=96), 30, m, agent=a)) for a, m in enumerate((150, 110))])
        qh = dev(W.queries(cfg, 40, 768))
        gpus = [p.gpu for p in pairs]
        calls = [(gpus[0], lambda: B.search_multi(gpus, [0, 150, 260], q, 20, 16)), (hot.gpu, lambda: hot.gpu.search(qh, 10, 6))]
        for own, call in calls:
            want = call()
            for cap in (1, 48):  # (1: the fewest the library takes, k + 1)
                B.pk_index_set_emit_cap(own.handle, cap)
                B.pk_profile_begin(own.handle)
                got = call()
                pr = B.pk_profile_end(own.handle)
                B.pk_index_set_emit_cap(own.handle, 0)
                assert pr.overflowed > 0 or cap > 1
                assert own is gpus[0] or pr.scan_hot_ms > 0
                assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    finally:
        for p in pairs + [hot]:
            p.close()


@pytest.mark.parametrize("n,d,nlist,nprobe,k,nq,page,storage", [
    (60000, 80, 20, 8, 37, 150, 0, F32), (6000, 100, 40, 12, 90, 20, 1024, F16), (9000, 64, 12, 12, 60, 300, 32, F16), (40000, 48, 3, 3, 100, 5, 64, F32)])
def test_thresholds_from_several_sample_pages(gpu_device, n, d, nlist, nprobe, k, nq, page, storage):
    """Long lists and large k take more than one page of sample (short and long pages, few and many queries); the
    sample decides what is emitted, never what is found."""
    cfg = W.scaled(W.C1, n=n, d=d, nlist=nlist, ncomp=nlist, train_iters=2)
    p, _ = make_pair(cfg, metric=L2, storage=storage, page_vecs=page)
    try:
        q = W.queries(cfg, 3, nq)
        probes = p.gpu.coarse(dev(q), nprobe).cpu().numpy()
        gi, gv = p.gpu.search(dev(q), k, nprobe)
        some = np.arange(0, nq, max(1, nq // 15))
        p.check_scan(q[some], k, probes[some], where="sample pages")
        fi, fv = p.gpu.scan_probes(dev(q[some]), k, dev(probes[some]))
        assert torch.equal(gi[some.tolist()], fi) and torch.equal(gv[some.tolist()], fv)
    finally:
        p.close()


@pytest.mark.parametrize("metric,storage,d,nlist,page", [(IP, F32, 128, 40, 0), (L2, F16, 70, 260, 32), (IP, F32, 64, 9000, 64)])
def test_inserts_around_the_sizes_where_their_path_changes(gpu_device, metric, storage, d, nlist, page):
    """One group and several (1024), the centroid kernel and the GEMM (520 000 scores, or fewer over many lists), and rows
    of one batch that meet in one list: every list ends up with its members in the order in which they came."""
    rng = np.random.default_rng(d + nlist)
    x = rng.standard_normal((12000, d)).astype(np.float32)
    if storage == F16:
        x = x.astype(np.float16).astype(np.float32)
    cent = x[rng.permutation(len(x))[:nlist]].copy()
    ix = B.Index(dev(cent), None, metric=metric, storage=storage, page_vecs=page, insert_reserve=20000)
    try:
        members, first, c64 = [[] for _ in range(nlist)], 0, cent.astype(np.float64)
        for m in (1, 64, 65, 1023, 1025, 2500, 700, 6200):
            rows = x[first:first + m]
            lists = ix.insert(dev(rows), want_lists=True).cpu().numpy()
            s = rows.astype(np.float64) @ c64.T
            if metric == L2:
                s = 2 * s - (c64 ** 2).sum(1)
            gap = s.max(1) - s[np.arange(len(rows)), lists]
            assert (gap <= 1e-5 * (1 + np.abs(s).max(1))).all()  # fp32 rounding of sums of up to 128 products
            for i, l in enumerate(lists):
                members[l].append(first + i)
            first += len(rows)
        assert ix.stats().device_error == 0 and ix.stats().n_total == first
        assert ix.list_lengths().tolist() == [len(v) for v in members]
        for l in np.argsort([-len(v) for v in members])[:12]:
            assert ix.list_ids(int(l)).cpu().numpy().tolist() == members[l]
    finally:
        ix.close()


@pytest.mark.parametrize("n,metric,d,half,copies", [
    (32768, IP, 600, 40, 2),  # fewer tiles than workgroups; two candidates a row: settled by their fp32 sums, or alike bit for bit
    (65536 + 3, L2, 603, 200, 3),  # three: the products of the whole values; rows that are not aligned
    (5 * 32768 + 5, IP, 64, 384, 4),  # more tiles than workgroups, two steps each
    (2 * 32768, L2, 1536, 300, 2)])  # 256 x 256 tiles, the longest rows
def test_rows_with_several_lists_alike_go_where_the_fp32_scores_say(gpu_device, n, metric, d, half, copies):
    """Lists that are given several times: the first copy differs by 2^-11 of its elements (less than first halves can tell), the
    second is the same bit for bit, in tiles far apart.  The lists are those of the fp32 coarse step, row for row."""
    assert by_first_halves(n, d, copies * half)
    g = torch.Generator(device="cuda").manual_seed(n + d)
    c = torch.randn((half, d), device="cuda", generator=g)
    other = c * (1 + torch.randint(-1, 2, c.shape, device="cuda", generator=g) * 2.0 ** -11)
    other[::3] = c[::3]
    cent = torch.cat([c, other, c, other][:copies])
    x = c[torch.randint(half, (n,), device="cuda", generator=g)] + 0.5 * torch.randn((n, d), device="cuda", generator=g)
    ix = B.Index(cent, x, metric=metric)
    try:
        where = torch.from_numpy(lists_of(ix, n))
        want = torch.cat([ix.coarse(x[i:i + 16384].contiguous(), 1)[:, 0].cpu() for i in range(0, n, 16384)])
        assert torch.equal(where, want.long())
    finally:
        ix.close()


@pytest.mark.parametrize("metric,d", [(IP, 512), (L2, 451)])
@pytest.mark.parametrize("many", [1, 64, 65, 4096, 4097, 9000])  # (512 lists: quarter tiles up to 4096 rows on 256 CUs)
def test_few_rows_with_several_near_lists_among_many_clear_ones(gpu_device, metric, d, many):
    """Rows that the first halves leave to the products of the whole values, `many` of a chunk, beside rows that are clear: the
    lists are those of the fp32 coarse step, row for row."""
    n, half = 2 * 32768, 500
    assert by_first_halves(n, d, 512)
    g = torch.Generator(device="cuda").manual_seed(d + many)
    c = torch.randn((half, d), device="cuda", generator=g)
    near = [c[:4] * (1 + torch.randint(-1, 2, (4, d), device="cuda", generator=g) * 2.0 ** -11) for _ in range(3)]
    cent = torch.cat([c] + near)
    lists = torch.randint(4, half, (n,), device="cuda", generator=g)
    for first in (0, 32768):  # (the chunks after the first are decided together)
        at = first + torch.randperm(32768, device="cuda", generator=g)[:many]
        lists[at] = torch.randint(4, (many,), device="cuda", generator=g)
    x = c[lists] + 0.2 * torch.randn((n, d), device="cuda", generator=g)
    ix = B.Index(cent, x, metric=metric)
    try:
        want = torch.cat([ix.coarse(x[i:i + 16384].contiguous(), 1)[:, 0].cpu() for i in range(0, n, 16384)])
        assert torch.equal(torch.from_numpy(lists_of(ix, n)), want.long())
    finally:
        ix.close()


@pytest.mark.parametrize("at", [0, 37, 1500])
def test_list_whose_products_are_nothing_is_found(gpu_device, at):
    """Inner product, every list but one on the other side of the rows and that one across them: its product is zero, and the best."""
    n, d, nlist = 5 * 32768, 64, 1536
    g = torch.Generator(device="cuda").manual_seed(at)
    x, cent = torch.rand((n, d), device="cuda", generator=g), -torch.rand((nlist, d), device="cuda", generator=g) - 0.1
    x[:, d // 2:] = 0
    cent[at, :d // 2], cent[at, d // 2:] = 0, 1
    ix = B.Index(cent, x, metric=IP)
    try:
        lengths = ix.list_lengths()
        assert by_first_halves(n, d, nlist) and lengths[at] == n and lengths.sum() == n
    finally:
        ix.close()


@pytest.mark.parametrize("n,nlist", [(16384, 256), (5 * 32768, 1536)])  # (by all three products; by those of the first halves to begin with)
@pytest.mark.parametrize("of_rows,of_lists", [(1e-24, 1.0), (1.0, 1e-24), (1e-12, 1e-12), (1e-24, 1e-10), (1e-19, 1.0)])
def test_assignment_of_rows_whose_squared_length_is_nothing(gpu_device, of_rows, of_lists, n, nlist):
    """Inner product, rows or lists so short that their squared lengths underflow: lists that lie closer together than half
    precision can tell are still told apart as fp32 sums do, by builds and by large inserts."""
    g = torch.Generator(device="cuda").manual_seed(3)
    d = 64
    assert by_first_halves(n, d, nlist) == (nlist > 256)
    half = torch.randn((nlist // 2, d), device="cuda", generator=g)
    cent = torch.stack([half, half * (1 + 2.0 ** -12 * torch.randn(half.shape, device="cuda", generator=g))], 1).reshape(nlist, d) * of_lists
    # (whole numbers: what half precision leaves out of the products is then all the lists')
    x = torch.randint(-8, 9, (n, d), device="cuda", generator=g) * 2.0 ** round(math.log2(of_rows))
    ix = B.Index(cent, x, metric=IP, insert_reserve=n)
    try:
        built = torch.empty(n, dtype=torch.int64, device="cuda")
        for l in np.nonzero(ix.list_lengths())[0].tolist():
            built[ix.list_ids(l)] = l
        inserted = ix.insert(x, want_lists=True).long()
        score = x.double() @ cent.double().T
        # as in fp32 sums of d products, and (the products themselves may be below fp32's smallest) d of those
        tol = (d + 4) * 2.0 ** -24 * (x.double().abs() @ cent.double().abs().T).amax(1) + d * 2.0 ** -149
        for lists in (built, inserted):
            short = score.amax(1) - score.gather(1, lists[:, None])[:, 0]
            assert (short <= 2 * tol).all(), (short / tol).max()
    finally:
        ix.close()


@pytest.mark.parametrize("nlist,page", [(3, 0), (300, 32), (9000, 64)])
def test_deletes_by_hash_set(gpu_device, nlist, page):
    """Ids of any value (the one that marks a free slot of the set among them), given twice, carried twice, carried by
    nobody; more than a pass takes; whole lists; tables of lists that fit LDS and that do not."""
    rng = np.random.default_rng(nlist)
    n, d = 15000, 32
    x = rng.standard_normal((n, d)).astype(np.float32)
    ids = rng.permutation(n).astype(np.int64) * 7 - 30000
    ids[5], ids[6], ids[7] = np.iinfo(np.int64).min, np.iinfo(np.int64).max, np.iinfo(np.int64).min
    ids[100:6100:2] = ids[101:6101:2]  # 3000 ids carried by two rows each
    ix = B.Index(dev(x[:nlist].copy()), dev(x), metric=L2, ids=dev(ids), page_vecs=page)
    try:
        left = ids.copy()
        whole = ix.list_ids(int(ix.list_lengths().argmax())).cpu().numpy()
        for gone in ([left[8]], [left[9], left[9], 12345678901], [np.iinfo(np.int64).min], whole[:4096], left[100:4100],
                     rng.permutation(left)[:5000], left[:0]):
            gone = np.asarray(gone, dtype=np.int64)
            removed = ix.delete(dev(gone))
            keep = ~np.isin(left, gone)
            assert removed == len(left) - keep.sum()
            left = left[keep]
            assert ix.stats().n_total == len(left)
        got = np.concatenate([ix.list_ids(l).cpu().numpy() for l in np.nonzero(ix.list_lengths())[0]])
        assert np.array_equal(np.sort(got), np.sort(left))
        at = {int(i): r for r, i in enumerate(ids) if (ids == i).sum() == 1}
        some = [i for i in left[:400].tolist() if i in at][:50]
        gi, gv = ix.search(dev(x[[at[i] for i in some]]), 1, min(nlist, 16))
        assert gi[:, 0].tolist() == some and float(gv.max()) < 1e-4  # the row that carries the id is still the id's
    finally:
        ix.close()


@pytest.mark.parametrize("n,d,nlist,nprobe,k,nq,page,storage,metric,equal", [
    (700, 40, 60, 5, 10, 3, 32, F32, IP, 0),  # ranges of a hundred values
    (3000, 40, 30, 9, 150, 33, 64, F32, L2, 0),  # a thousand values and a K beyond what parts serve
    (5000, 100, 12, 6, 300, 17, 0, F16, IP, 0),  # up to 4096 values, K beyond the workgroup's threads
    (9000, 64, 900, 600, 20, 5, 0, F32, L2, 0),  # more probes than threads
    (60000, 48, 20, 8, 23, 70, 0, F32, IP, 0),  # long ranges: 64 parts, the most for them
    (60000, 48, 20, 8, 127, 40, 96, F16, L2, 0),  # ... 256 parts, the most for them
    (60000, 48, 20, 8, 255, 9, 1024, F32, L2, 0),  # ... 1024 parts, the most for them
    (60000, 1100, 60, 20, 10, 15, 0, F32, L2, 0),  # sliced queries, 16 slots, long ranges
    (60000, 1100, 60, 8, 10, 75, 0, F32, IP, 0),  # ... 32 slots, several groups of some lists
    (60000, 1100, 60, 8, 40, 75, 96, F16, L2, 0),
    (60000, 64, 4, 2, 100, 300, 0, F16, IP, 0),  # several groups per list
    (30000, 32, 8, 4, 50, 12, 0, F32, IP, 6000),  # equal values: more than are collected
    (90000, 32, 4, 4, 50, 3, 0, F32, L2, 60000)])  # ... more blocks than are
def test_values_written_whole_give_the_rows_of_the_gated_scan(gpu_device, n, d, nlist, nprobe, k, nq, page, storage, metric, equal):
    """Without the buffer for values, or with a forced emission region, the call goes through sample and gate.  The same
    rows, bit for bit, after inserts (delta pages) and deletes too, and for two memories in one call."""
    g = torch.Generator(device="cuda").manual_seed(n + d)
    x = torch.randn((n, d), device="cuda", generator=g)
    if equal:
        x[torch.randperm(n, device="cuda", generator=g)[:equal]] = x[0].clone()
    x = x.half().float()
    cent = x[torch.randperm(n, device="cuda", generator=g)[:nlist]].clone()
    cent += 1e-3 * torch.randn(cent.shape, device="cuda", generator=g)
    q = torch.randn((nq, d), device="cuda", generator=g)
    q[0] = x[0]
    if d == 1100:  # half of the queries ask the same lists
        q[: nq // 2 + 1] = x[0] + 0.1 * q[: nq // 2 + 1]
    ids = torch.randperm(3 * n, device="cuda", generator=g)[:n].contiguous()
    ix, other = (B.Index(cent, rows, metric=metric, storage=storage, page_vecs=page, ids=i, insert_reserve=4096)
                 for rows, i in ((x, ids), (x[: n // 3].contiguous(), None)))
    try:
        for stage in ("built", "changed"):
            if stage == "changed":
                ix.delete(ids[: n // 10].contiguous())
                ix.insert(x[:700].contiguous(), ids[:700].contiguous())
            offs = [0, nq - nq // 3, nq]
            with route(ix, True) as ran:
                whole = ix.search(q, k, nprobe), B.search_multi([ix, other], offs, q, k, nprobe)
            assert ran.whole
            with route(ix, False):
                gated = ix.search(q, k, nprobe), B.search_multi([ix, other], offs, q, k, nprobe)
            B.pk_index_set_emit_cap(ix.handle, 32768)
            gated += ix.search(q, k, nprobe), B.search_multi([ix, other], offs, q, k, nprobe)
            B.pk_index_set_emit_cap(ix.handle, 0)
            if d == 1100:
                asked = torch.bincount(ix.coarse(q, nprobe).flatten().long())
                assert (asked.max() > 32) == (nq > 32) and np.sort(ix.list_lengths())[-nprobe:].sum() > 8192
            for (wi, wv), (gi, gv) in zip(whole * 2, gated):
                assert torch.equal(wi, gi) and torch.equal(wv, gv), stage
        assert ix.stats().device_error == 0 and other.stats().device_error == 0
    finally:
        ix.close()
        other.close()


@pytest.mark.parametrize("n,d,nlist,nprobe,k,nq,page,storage,metric", [
    (9000, 192, 60, 5, 10, 7, 0, F32, L2),  # three slices: the least
    (9000, 193, 60, 5, 10, 7, 64, F32, IP),  # four: no slice left over
    (9000, 300, 60, 5, 10, 7, 32, F32, L2),  # five; tiles of a page of 32 rows
    (9000, 700, 60, 5, 33, 7, 96, F16, IP),  # six; half a wave's rows missing in every other tile
    (20000, 400, 40, 9, 10, 30, 1024, F32, L2),  # tiles from the middle of pages; groups of 32 slots
    (12000, 300, 12, 6, 20, 90, 256, F16, L2),  # of 64, several per list
    (9000, 1536, 50, 6, 5, 3, 0, F32, IP),  # the longest rows, instead of the sliced queries' kernel
    (9000, 1536, 20, 6, 5, 35, 128, F32, L2),  # ... several groups per list
    (40000, 1000, 4, 2, 20, 2, 256, F16, IP)])  # ranges of which the bests of 16 are written
def test_scans_of_few_tiles_give_the_rows_of_the_gated_scan(gpu_device, n, d, nlist, nprobe, k, nq, page, storage, metric):
    """Searches whose tiles are cut smaller because there are few: the rows of the gated scan, bit for bit, after inserts (delta
    pages) and deletes too, and for two memories in one call.  The number of tiles says that they were cut."""
    g = torch.Generator(device="cuda").manual_seed(n + d)
    c = torch.randn((nlist, d), device="cuda", generator=g)

    def around(m):
        return (c[torch.randint(nlist, (m,), device="cuda", generator=g)] + 0.5 * torch.randn((m, d), device="cuda", generator=g)).half().float()

    x, q = around(n), around(nq)
    ix, other = (B.Index(c, rows, metric=metric, storage=storage, page_vecs=page, insert_reserve=4096) for rows in (x, x[: n // 3].contiguous()))
    unit = 64 if page % 64 == 0 else 32  # (0: pages of 128)
    try:
        for stage in ("built", "changed"):
            if stage == "changed":
                ix.delete(torch.arange(0, n, 11, device="cuda"))
                ix.insert(around(900))
            offs = [0, nq - nq // 3, nq]
            with route(ix, True) as ran:
                whole = ix.search(q, k, nprobe), B.search_multi([ix, other], offs, q, k, nprobe)
            tiles = []
            for one in (lambda: ix.search(q, k, nprobe), lambda: ix.search(q[:1], k, nprobe)):
                B.pk_profile_begin(ix.handle)
                one()
                tiles.append(B.pk_profile_end(ix.handle).tiles)
            assert ran.whole
            asked = [torch.bincount(ix.coarse(r, nprobe).flatten().long(), minlength=nlist).cpu().numpy() for r in (q, q[:1])]
            per_list = nq * nprobe / nlist
            slots = min(16 if per_list <= 6 else 32 if per_list <= 20 else 64, 16 if d == 1536 else 64)
            lengths = ix.list_lengths()
            assert tiles == [int((-(-lengths // unit) * -(-a // s)).sum()) for a, s in zip(asked, (slots, 16))], tiles
            with route(ix, False):
                gated = ix.search(q, k, nprobe), B.search_multi([ix, other], offs, q, k, nprobe)
            for (wi, wv), (gi, gv) in zip(whole, gated):
                assert torch.equal(wi, gi) and torch.equal(wv, gv), stage
        assert ix.stats().device_error == 0 and other.stats().device_error == 0
    finally:
        ix.close()
        other.close()


@pytest.mark.parametrize("d", [1, 3, 4, 5, 63, 64, 65, 127, 129, 192, 255, 256, 259, 1021, 1024, 1025, 1536])
@pytest.mark.parametrize("shift", [0, 1])
def test_kmeans_update_of_rows_of_any_width(gpu_device, d, shift):
    """Clusters of no member, of one, of a piece's number of members and one beside it, of several pieces; rows that begin anywhere.
    Every centroid is the float64 mean of its members, the objective their sum of squared distances, and every row is with
    the nearest centroid (up to the rounding of fp32 sums of d products)."""
    sizes = [1, 0, 255, 256, 257, 2, 900, 7, 511, 513]
    g = torch.Generator(device="cuda").manual_seed(d)
    c = torch.randn((len(sizes), d), device="cuda", generator=g) + 40 * torch.arange(len(sizes), device="cuda")[:, None]
    of = torch.repeat_interleave(torch.arange(len(sizes), device="cuda"), torch.tensor(sizes, device="cuda"))
    of = of[torch.randperm(len(of), device="cuda", generator=g)]
    room = torch.zeros(len(of) * d + 4, device="cuda")
    x = room[shift:shift + len(of) * d].view(len(of), d)
    x[:] = c[of] + torch.randn((len(of), d), device="cuda", generator=g)
    cent, assign = c.clone(), torch.empty(len(of), dtype=torch.int32, device="cuda")
    inertia = B.pk_kmeans(x, cent, 1, assign)
    assert torch.equal(assign.long(), of)
    means = torch.stack([x[of == l].double().mean(0) if m else c[l].double() for l, m in enumerate(sizes)])
    assert (cent.double() - means).abs().max() <= 2.0 ** -23 * means.abs().max()
    want = float((x.double() - c.double()[of]).square().sum())
    assert abs(inertia[0] - want) <= 1e-9 * (want + float(x.double().square().sum()))


@pytest.mark.parametrize("d", [1, 2, 3, 4, 5, 6, 7, 61, 67, 130])
@pytest.mark.parametrize("shift", [0, 1, 2])
@pytest.mark.parametrize("metric", [IP, L2])
def test_rows_of_odd_widths_that_begin_anywhere(gpu_device, d, shift, metric):
    """Rows and queries whose 16-byte pieces are not aligned or run past the row's end, and such that have none: lists of a build (in tiles
    and its last rows beyond them), of inserts and of searches of one and many queries are the nearest in 64 bits, up to the
    rounding of fp32 sums of d products, and so are the rows that are found in them."""
    g = torch.Generator(device="cuda").manual_seed(d)

    def odd(rows):
        room = torch.full((rows.numel() + 4,), float("nan"), device="cuda")
        room[shift:shift + rows.numel()] = rows.flatten()
        return room[shift:shift + rows.numel()].view(rows.shape)

    n, nlist = 33000, 200
    cent = torch.randn((nlist, d), device="cuda", generator=g)
    x, q = torch.randn((n, d), device="cuda", generator=g), torch.randn((300, d), device="cuda", generator=g)
    ix = B.Index(cent, odd(x), metric=metric, insert_reserve=8192)

    def scores(rows, to):
        s = rows.double() @ to.double().T
        return 2 * s - to.double().square().sum(1) - rows.double().square().sum(1)[:, None] if metric == L2 else s

    def bound(rows, to):  # both values of a pair, each 4 sqrt(d) roundings of its terms off
        size = (rows.double().norm(dim=1)[:, None] + to.double().norm(dim=1).max()) ** 2
        return 16 * math.sqrt(d) * 2.0 ** -24 * size

    def nearest(rows, lists):
        s = scores(rows, cent)
        assert (s.max(1).values[:, None] - s.gather(1, lists) <= bound(rows, cent)).all()

    try:
        nearest(x, torch.from_numpy(lists_of(ix, n)).cuda()[:, None])
        nearest(q, ix.coarse(odd(q), 1).long())
        nearest(q[:1], ix.coarse(odd(q[:1]), 1).long())
        for m in (3, 5000):
            nearest(x[:m], ix.insert(odd(x[:m]), want_lists=True).long()[:, None])
        for m in (1, 300):
            ids, dist = ix.search(odd(q[:m]), 5, nlist)
            every = torch.cat([x, x[:3], x[:5000]])
            s = scores(q[:m], every)
            off = bound(q[:m], every)
            assert (s.topk(5, 1).values - s.gather(1, ids) <= off).all() and ((s.gather(1, ids) * (-1 if metric == L2 else 1) - dist).abs() <= off).all()
    finally:
        ix.close()


@pytest.mark.parametrize("nprobe,k", [(30, 20), (30, 23), (30, 24), (30, 100), (30, 127), (30, 128), (10, 23), (10, 24), (10, 100), (10, 127)])
@pytest.mark.parametrize("metric", [IP, L2])
def test_bests_of_short_lists_among_many_values(gpu_device, nprobe, k, metric):
    """Lists of 270 rows that lie apart, 8000 values a query and 2700: the nearest list fills fewer parts of the range than k, and what
    is within the first bound is far more than k.  The rows of the gated scan, bit for bit."""
    g = torch.Generator(device="cuda").manual_seed(k)
    nlist, d = 300, 40
    c = torch.randn((nlist, d), device="cuda", generator=g)

    def around(m):
        return c[torch.randint(nlist, (m,), device="cuda", generator=g)] + 0.3 * torch.randn((m, d), device="cuda", generator=g)

    ix, q = B.Index(c, around(270 * nlist), metric=metric), around(37)
    try:
        with route(ix, True) as ran:
            whole = ix.search(q, k, nprobe)
        with route(ix, False):
            gated = ix.search(q, k, nprobe)
        assert ran.whole and (np.sort(ix.list_lengths())[-nprobe:].sum() > 8192) == (nprobe == 30)
        assert torch.equal(whole[0], gated[0]) and torch.equal(whole[1], gated[1])
    finally:
        ix.close()


@pytest.mark.parametrize("n,kinds,k,nprobe,nq,page,metric,storage", [
    (300000, 50, 100, 16, 1, 0, IP, F32), (300000, 50, 10, 16, 3, 96, L2, F16), (100000, 1, 30, 2, 5, 0, L2, F32),
    (200000, 7, 200, 40, 4, 1024, IP, F16), (300000, 2000, 255, 40, 2, 32, L2, F32), (70000, 3, 1, 40, 9, 0, IP, F32)])
def test_equal_values_beyond_what_is_collected_cost_no_more_than_the_gated_scan(gpu_device, n, kinds, k, nprobe, nq, page, metric, storage):
    """A memory of few different rows: groups of equal values that are larger than what the final selection collects.  The rows of
    the gated scan, ids in ascending order within a group, the largest and the smallest id there is among them; and one more
    pass over the values, not one for each member of a group: the gated route's time is not exceeded (twice it would be a pass
    per member, here three times and more)."""
    g = torch.Generator(device="cuda").manual_seed(kinds)
    d, nlist = 64, 40
    some = torch.randn((kinds, d), device="cuda", generator=g)
    x = some[torch.randint(kinds, (n,), device="cuda", generator=g)].contiguous()
    ids = torch.randperm(5 * n, device="cuda", generator=g)[:n] - 2 * n
    ids[n // 2], ids[n // 3] = 2 ** 63 - 1, -(2 ** 63)
    ix = B.Index(torch.randn((nlist, d), device="cuda", generator=g), x, ids=ids.contiguous(), metric=metric, storage=storage, page_vecs=page,
                 insert_reserve=4096)
    try:
        ix.insert(x[:2000].contiguous(), ids[:2000].contiguous())
        q = torch.randn((nq, d), device="cuda", generator=g)
        rows, times = [], []
        for cap in (32768, 0):
            B.pk_index_set_emit_cap(ix.handle, cap)
            with route(ix, True) as ran:
                rows.append(ix.search(q, k, nprobe))
            assert ran.whole == (cap == 0) or ix.list_lengths().max() == n + 2000
            start, stop = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            best = math.inf
            for _ in range(3):
                start.record()
                ix.search(q, k, nprobe)
                stop.record()
                stop.synchronize()
                best = min(best, start.elapsed_time(stop))
            times.append(best)
        assert torch.equal(rows[0][0], rows[1][0]) and torch.equal(rows[0][1], rows[1][1])
        assert times[1] < 2 * times[0] + 0.1, times
    finally:
        ix.close()


@pytest.mark.parametrize("n,d,nlist,storage,calls", [
    (800_000, 256, 800, F32, [(200, 4, True), (256, 10, False), (600, 20, True), (1, 64, True)]),  # short lists beyond the caches
    (800_000, 1024, 800, F16, [(200, 10, True), (256, 20, False)]),  # ... of wider rows, whose values weigh less
    (1_700_000, 256, 1700, F32, [(600, 6, True), (600, 16, False)]),  # ... of many bytes, for batches with large samples
    (1_000_000, 256, 250, F32, [(64, 32, True), (256, 20, True)]),  # long lists
    (300_000, 256, 300, F32, [(256, 20, True), (512, 15, True)]),  # lists that the caches hold
    (120_000, 1024, 120, F32, [(60, 8, True), (60, 14, False), (110, 7, True)]),  # sliced queries, lists probed by few and by more
    (120_000, 1024, 20, F32, [(500, 1, False)])])
def test_which_calls_write_their_values_whole(gpu_device, n, d, nlist, storage, calls):
    """Both sides of the lines between the two ways: which one a call takes, and the same rows."""
    g = torch.Generator(device="cuda").manual_seed(nlist)
    mu = torch.randn((nlist, d), device="cuda", generator=g)
    x = mu[torch.randint(nlist, (n,), device="cuda", generator=g)]
    for a in range(0, n, 1 << 18):
        x[a:a + (1 << 18)] += 0.3 * torch.randn(x[a:a + (1 << 18)].shape, device="cuda", generator=g)
    ix = B.Index(mu, x, metric=IP, storage=storage)
    del x
    try:
        for nq, nprobe, expected in calls:
            q = mu[torch.randint(nlist, (nq,), device="cuda", generator=g)] + 0.3 * torch.randn((nq, d), device="cuda", generator=g)
            with route(ix, True) as ran:
                rows = ix.search(q, 10, nprobe)
            assert ran.whole == expected, (nq, nprobe, ix.list_lengths().max())
            with route(ix, False) as ran:
                gated = ix.search(q, 10, nprobe)
            assert not ran.whole and torch.equal(rows[0], gated[0]) and torch.equal(rows[1], gated[1])
    finally:
        ix.close()


@pytest.mark.parametrize("reserve", [False, True])
@pytest.mark.parametrize("nq,k,nprobe,storage,metric", [(1, 10, 6, F32, IP), (64, 20, 12, F16, L2), (300, 5, 40, F32, L2)])
def test_searches_without_the_buffer_for_whole_values(gpu_device, reserve, nq, k, nprobe, storage, metric):
    """A search that may not have room for its values goes through sample and gate: the same rows, and no more memory
    than that route takes.  Then it may: in the workspace, or (300 queries of every list) in a buffer that comes beside it
    and leaves the graph of a captured search valid."""
    g = torch.Generator(device="cuda").manual_seed(nq)
    n, d, nlist = 60000, 48, 40
    x = torch.randn((n, d), device="cuda", generator=g)
    q = torch.randn((nq, d), device="cuda", generator=g)
    ix = B.Index(x[:nlist].clone(), x, metric=metric, storage=storage, insert_reserve=1000)
    try:
        def gated(cap):
            B.pk_index_set_values_cap(ix.handle, cap)
            if reserve:
                ix.reserve(nq, k, nprobe)
            B.pk_profile_begin(ix.handle)
            rows = ix.search(q, k, nprobe)
            pr = B.pk_profile_end(ix.handle)
            assert pr.emitted < pr.candidates
            return rows, ix.stats()

        rows, first = gated(1)
        width = int(np.sort(ix.list_lengths())[-nprobe:].sum())
        assert first.workspace_grows == 1
        ids, dist = torch.empty_like(rows[0]), torch.empty_like(rows[1])
        graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            with torch.cuda.graph(graph, stream=side):
                B.pk_search(ix.handle, q, k, nprobe, ids, dist)
        for cap in (4 * nq * width, 0):  # (of the values alone: not enough for what goes with them; then as much as it takes)
            if cap:
                again, st = gated(cap)
            else:
                with route(ix, True) as ran:
                    again = ix.search(q, k, nprobe)
                assert ran.whole
                grown = ix.stats()
                if nprobe == nlist:
                    assert grown.workspace_grows == st.workspace_grows + 1 and grown.workspace_bytes > 4 * nq * width > first.workspace_bytes
                else:
                    assert grown.workspace_bytes == st.workspace_bytes
            assert torch.equal(again[0], rows[0]) and torch.equal(again[1], rows[1])
            for _ in range(2):
                ids.fill_(-7)
                torch.cuda.synchronize()
                graph.replay()
                torch.cuda.synchronize()
                assert torch.equal(ids, rows[0]) and torch.equal(dist, rows[1])
    finally:
        ix.close()


@pytest.mark.parametrize("gated", [False, True])
@pytest.mark.parametrize("d,nq,k,metric", [(32, 1, 10, IP), (64, 40, 200, L2), (100, 300, 10, IP), (1100, 6, 5, L2)])
def test_a_work_list_without_room_scans_nothing(gpu_device, gated, d, nq, k, metric):
    """Whichever way the values go: padding for every query and the sticky flag, and the same rows as before once there is room
    again."""
    g = torch.Generator(device="cuda").manual_seed(d)
    n, nlist, nprobe = 6000, 12, 5
    x = torch.randn((n, d), device="cuda", generator=g)
    q = torch.randn((nq, d), device="cuda", generator=g)
    ix = B.Index(x[:nlist].clone(), x, metric=metric)
    try:
        B.pk_index_set_emit_cap(ix.handle, 4096 if gated else 0)
        ids, dist = ix.search(q, k, nprobe)
        assert ix.stats().device_error == 0 and int(ids.min()) >= 0
        for cap in (1, 4):
            B.pk_index_set_tile_cap(ix.handle, cap)
            none, worst = ix.search(q, k, nprobe)
            assert (none == -1).all() and torch.isinf(worst).all()
            assert ix.stats().device_error == 4
        B.pk_index_set_tile_cap(ix.handle, 0)
        again = ix.search(q, k, nprobe)
        assert torch.equal(again[0], ids) and torch.equal(again[1], dist)
    finally:
        ix.close()


@pytest.mark.parametrize("storage", [F32, F16])
@pytest.mark.parametrize("metric", [IP, L2])
@pytest.mark.parametrize("d,nlist,nq", [
    (1, 3, 1), (63, 40, 17), (64, 130, 49), (65, 16, 200), (100, 40, 64), (130, 300, 33), (1030, 70, 12),
    (411, 333, 365), (411, 333, 366), (1030, 832, 90), (100, 1200, 700)])  # (both sides of 5e7 products; those of 100 by their alignment only)
def test_queries_copied_beside_the_coarse_step(gpu_device, storage, metric, d, nlist, nq):
    """Small batches, and larger ones of whole 16-byte pieces, have their padded copies and norms made by the centroid kernel: the probes are the best by 64 bits, and
    the rows those of a scan of the same probes, which prepares the queries by itself.  Of any alignment, over two memories."""
    g = torch.Generator(device="cuda").manual_seed(d * nlist + nq)
    n, nprobe, k = 20 * nlist, min(3, nlist // 2 + 1), 10
    cent = torch.randn((nlist, d), device="cuda", generator=g)
    x = torch.randn((n, d), device="cuda", generator=g)
    flat = torch.randn(nq * d + 1, device="cuda", generator=g)
    q = flat[:-1].view(nq, d)
    off = torch.empty_like(flat)[1:].view(nq, d)  # 4 bytes from any wider boundary
    off.copy_(q)
    ix, other = (B.Index(c, rows, metric=metric, storage=storage) for c, rows in ((cent, x), (cent[: nlist // 2 + 1].contiguous(), x)))
    try:
        probes = ix.coarse(q, nprobe)
        c64, q64 = cent.double(), q.double()
        score = q64 @ c64.T if metric == IP else -((q64 ** 2).sum(1)[:, None] - 2 * q64 @ c64.T + (c64 ** 2).sum(1))
        # fp32 sums of d products, each term rounded once and added in some order: d + 4 halves of an ulp of the sum of magnitudes
        tol = (d + 4) * 2.0 ** -24 * ((q64.abs() @ c64.abs().T).max() * 2 + (q64 ** 2).sum(1).max() + (c64 ** 2).sum(1).max())
        got = score.gather(1, probes.long())
        best = score.topk(nprobe, 1).values
        assert (got.sort(1, descending=True).values >= best - 2 * tol).all()
        ids, vals = ix.search(q, k, nprobe)
        want = ix.scan_probes(q, k, probes)
        assert torch.equal(ids, want[0]) and torch.equal(vals, want[1])
        cut = nq // 3
        both = B.search_multi([ix, other], [0, cut, nq], q, k, nprobe)
        if cut:
            assert torch.equal(both[0][:cut], ids[:cut]) and torch.equal(both[1][:cut], vals[:cut])
        rest = other.search(q[cut:].contiguous(), k, nprobe)
        assert torch.equal(both[0][cut:], rest[0]) and torch.equal(both[1][cut:], rest[1])
        if d % 64:  # (rows that are padded)
            a, b = ix.search(off, k, nprobe), B.search_multi([ix, other], [0, cut, nq], off, k, nprobe)
            assert torch.equal(a[0], ids) and torch.equal(a[1], vals)
            assert torch.equal(b[0], both[0]) and torch.equal(b[1], both[1])
    finally:
        ix.close()
        other.close()


@pytest.mark.parametrize("nlist", [1, 63, 64, 65, 1023, 1024, 1025, 2500])
def test_extents_of_built_lists_are_laid_one_behind_the_other(gpu_device, nlist):
    """Lists of no row, of less than a page, of whole pages and of more, on both sides of what the layout takes at a time: every
    row in its own list, and as many pages as the lists' lengths need; with a page less the build is refused."""
    page = 32
    lens = (torch.arange(nlist) * 37 % 70) * (torch.arange(nlist) % 5 != 3)
    lens[0] = 3 * page
    lists = torch.repeat_interleave(torch.arange(nlist), lens)
    lists = lists[torch.randperm(len(lists), generator=torch.Generator().manual_seed(nlist))]
    cent = torch.stack([torch.arange(nlist) % 50, torch.arange(nlist) // 50, torch.zeros(nlist), torch.ones(nlist)], 1).float()
    pages = int(((lens + page - 1) // page).sum())
    # rows are their list's centroid: under L2 every other list is a unit away at least
    c = B.pk_config(4, nlist, L2, F32, page, 1)
    one = B.pk_arena_bytes(c, 0, (nlist + 1) * page) - B.pk_arena_bytes(c, 0, nlist * page)  # a page's bytes
    room = B.pk_arena_bytes(c, 0, 0)
    ix = B.Index(cent.cuda(), cent[lists].cuda(), metric=L2, page_vecs=page, max_delta_pages=1, arena_bytes=room + (pages + 1) * one)
    try:
        st = ix.stats()
        assert st.pages_used == pages and st.device_error == 0 and st.n_total == len(lists)
        assert ix.list_lengths().tolist() == lens.tolist()
        for l in {0, 1, nlist // 2, nlist - 2, nlist - 1} & set(range(nlist)):
            assert sorted(ix.list_ids(l).tolist()) == (lists == l).nonzero()[:, 0].tolist()
        ids, _ = ix.search(cent[lists[:64]].cuda().contiguous(), 1, 1)
        assert (lists[ids[:, 0].cpu()] == lists[: len(ids)]).all()
        spare = int(st.pages_total) - pages
        assert spare >= 0
    finally:
        ix.close()
    with pytest.raises(B.PancakeError) as e:
        B.Index(cent.cuda(), cent[lists].cuda(), metric=L2, page_vecs=page, max_delta_pages=1,
                arena_bytes=room + (pages + 1) * one - (spare + 1) * one)
    assert e.value.status == B.PK_ERR_NOMEM


@pytest.mark.parametrize("d", [1, 2, 3])
def test_narrowest_rows_take_the_tiled_products_too(gpu_device, d):
    """Rows of less than 16 bytes: a build that begins with the products of first halfs, in whole chunks and a rest, finds the lists
    of the fp32 coarse step, up to the rounding of its sums; and a k-means iteration takes about as long as one of rows of 16 bytes
    (262 144 rows, 4096 lists: 1.2 to 2.4 times as long; by the small inserts' kernel, row group after row group, 17 times as long)."""
    n, nlist = 5 * 32768 + 5, 1536
    assert by_first_halves(n, 64, nlist)
    g = torch.Generator(device="cuda").manual_seed(d)
    x, cent = torch.randn((n, d), device="cuda", generator=g), torch.randn((nlist, d), device="cuda", generator=g)
    for metric in (IP, L2):
        ix = B.Index(cent, x, metric=metric)
        try:
            lists = torch.from_numpy(lists_of(ix, n)).cuda()
        finally:
            ix.close()
        for a in range(0, n, 32768):
            rows = x[a:a + 32768].double()
            s = rows @ cent.double().T
            size = rows.norm(dim=1) * cent.double().norm(dim=1).max()
            if metric == L2:
                s = 2 * s - cent.double().square().sum(1)
                size = (rows.norm(dim=1) + cent.double().norm(dim=1).max()) ** 2
            # both values of a pair, each 4 sqrt(d) roundings of its terms off
            assert (s.max(1).values - s.gather(1, lists[a:a + 32768, None])[:, 0] <= 16 * math.sqrt(d) * 2.0 ** -24 * size).all()

    def seconds(width):
        rows = torch.randn((262144, width), device="cuda", generator=g)
        taken = []
        for _ in range(4):
            c = rows[:4096].clone()
            torch.cuda.synchronize()
            t = time.perf_counter()
            B.pk_kmeans(rows, c, 1, None)
            taken.append(time.perf_counter() - t)
        return min(taken)

    assert seconds(d) < 4 * seconds(4)


@pytest.mark.parametrize("metric", [IP, L2])
@pytest.mark.parametrize("apart", [1, 2, 3, 4, 5, 8, 31, 32, 36, 63, 64, 255, 256])
def test_two_near_lists_at_any_distance_are_told_by_their_fp32_scores(gpu_device, metric, apart):
    """Pairs of lists as far apart as `apart`: in one lane's columns, in the other half wave's, in other waves' and other tiles'; every third
    pair the same bit for bit.  The lists are those of the fp32 coarse step, row for row (of two that are the same the lower)."""
    n, d, nlist = 2 * 32768 + 5, 512, 512
    assert by_first_halves(n, d, nlist)
    g = torch.Generator(device="cuda").manual_seed(apart)
    cent = torch.randn((nlist, d), device="cuda", generator=g)
    first = torch.tensor([l for l in range(nlist - apart) if l // apart % 2 == 0], device="cuda")
    other = cent[first] * (1 + torch.randint(-1, 2, (len(first), d), device="cuda", generator=g) * 2.0 ** -11)
    other[::3] = cent[first[::3]]
    cent[first + apart] = other
    x = cent[first[torch.randint(len(first), (n,), device="cuda", generator=g)]] + 0.4 * torch.randn((n, d), device="cuda", generator=g)
    ix = B.Index(cent, x, metric=metric)
    try:
        where = torch.from_numpy(lists_of(ix, n))
        want = torch.cat([ix.coarse(x[i:i + 16384].contiguous(), 1)[:, 0].cpu() for i in range(0, n, 16384)])
        assert torch.equal(where, want.long())
        assert (where % nlist).unique().numel() > len(first)  # (either of a pair is some row's)
    finally:
        ix.close()


@pytest.mark.parametrize("rows,per_cu,cut", [(600, 2.1, True), (600, 2.6, False), (600, 3.6, False), (86, 0.9, True), (86, 1.5, False)])
def test_tiles_of_large_pages_are_cut_only_while_that_was_measured_to_pay(gpu_device, rows, per_cu, cut):
    """Pages of 256 rows, lists of several pages and of a third of one, on both sides of the lines (tiles of 64 rows per CU) from which smaller
    tiles are no gain: the number of tiles says whether they were cut, and the rows are those of the gated scan either way."""
    d, nprobe, nq, page = 200, 10, 12, 256
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    # share of the lists that are probed: share * nlist * (rows / 64 + 0.75) = per_cu * cus
    if rows > 128:
        nlist = next(m for m in range(11, 4000) if (1 - (1 - nprobe / m) ** nq) * m * (rows / 64 + 0.75) >= per_cu * cus)
    else:
        nlist = 1000
        nprobe = next(m for m in range(1, 999) if (1 - (1 - m / nlist) ** nq) * nlist * (rows / 64 + 0.75) >= per_cu * cus)
    g = torch.Generator(device="cuda").manual_seed(rows)
    c = torch.randn((nlist, d), device="cuda", generator=g)
    x = c.repeat(rows, 1) + 0.3 * torch.randn((nlist * rows, d), device="cuda", generator=g)
    q = c[torch.randperm(nlist, device="cuda", generator=g)[:nq]] + 0.3 * torch.randn((nq, d), device="cuda", generator=g)
    ix = B.Index(c, x, metric=L2, page_vecs=page)
    try:
        assert (ix.list_lengths() == rows).all()
        with route(ix, True) as ran:
            whole = ix.search(q, 10, nprobe)
        with route(ix, False):
            gated = ix.search(q, 10, nprobe)
        assert torch.equal(whole[0], gated[0]) and torch.equal(whole[1], gated[1])
        probed = len(ix.coarse(q, nprobe).unique())
        assert ran.whole and ran.profile.tiles == probed * -(-rows // (64 if cut else page))
    finally:
        ix.close()
