"""Edges of single kernels and of the rules that choose between them: tile remainders, the smallest and
largest sizes of a path, and the sizes on both sides of a dispatch."""
import numpy as np
import pytest
import torch

from gpu_util import Pair, dev, make_pair
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
