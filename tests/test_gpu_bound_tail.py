"""The terms without a column of their own (the tail) in the bounds' table: where a query's list of them ends (32 entries at once, 128 in
all, then straight from the query), where a bucket of a tile's postings holds more entries than are read at once, at the edges of the
tiles, and the counts of required terms beside the values."""
import numpy as np
import pytest
import torch

from paper_2511_00855_amd import binding as B
from paper_2511_00855_amd.synth import VecSet
from test_gpu_bounds import _slack

pytestmark = pytest.mark.gpu


def _lists(rng, rows, lengths, lo, vocab):
    """CSR of lengths[r] distinct terms of lo .. vocab a row, ascending, with values of both signs."""
    idx = [np.sort(rng.choice(np.arange(lo, vocab, dtype=np.int32), k, replace=False)) for k in lengths]
    ip = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    return ip, np.concatenate(idx).astype(np.int32), rng.standard_normal(int(ip[-1])).astype(np.float32)


# few terms (every bucket holds many documents) and many; queries of no tail at all up to more than a list of 128 takes
@pytest.mark.parametrize("n,vocab,doc_terms", [(1, 700, 3), (256, 700, 60), (257, 4000, 90), (511, 700, 200), (600, 20_000, 150)])
def test_tail_of_every_length(n, vocab, doc_terms):
    rng, dim = np.random.default_rng(n + vocab), 64
    lengths = [0, 1, 7, 8, 9, 31, 32, 33, 63, 64, 65, 127, 128, 129, 130, 200, 300, 500] * 15   # 270 queries: two tiles
    nq = len(lengths)
    def vecs(m, sp, tx):
        tx = (tx[0], tx[1], rng.integers(1, 4, len(tx[1])).astype(np.float32))
        return VecSet(m, dim, rng.standard_normal((m, dim)).astype(np.float32) / 8, *sp, *tx, vocab, vocab)
    few = np.maximum(rng.integers(0, doc_terms, (2, n)), np.arange(n) % 2 == 0)
    docs = vecs(n, _lists(rng, n, few[0], 0, vocab), _lists(rng, n, few[1], 0, vocab))
    queries = vecs(nq, _lists(rng, nq, lengths, 0, vocab), _lists(rng, nq, lengths[::-1], 0, vocab))
    d, q = B.DeviceVecs(docs), B.DeviceVecs(queries)
    ix = B.Index.ingest(d, B.build_params(8))
    for pw in (np.ones((nq, 3)), rng.uniform(-1.0, 1.0, (nq, 3))):
        pw = pw.astype(np.float32)
        sc = ix.hybrid_scores(q, np.tile(np.arange(n, dtype=np.int32), (nq, 1)), pw)[:, :, 3].double()
        up = ix.stage_score_bounds(q, pw).double()
        assert (up >= sc).all()
        assert (up - sc <= _slack(ix, queries, docs, pw, False)).all()
    # required terms: those that few documents hold have no column, and the entries count them
    df = np.bincount(docs.tx_idx, minlength=vocab) + np.zeros(vocab)
    both = np.sort(np.concatenate([df, np.bincount(docs.sp_idx, minlength=vocab)]))[::-1]
    rare = np.flatnonzero((df > 0) & (df < (both[512] if len(both) > 512 else 0) / 2))
    if len(rare):
        kw = rng.choice(rare, (nq, 16)).astype(np.int32)
        kw[:, 12:] = -1
        kw[::3, 3] = vocab + 5
        held = np.zeros((n, vocab), np.int32)
        held[np.repeat(np.arange(n), np.diff(docs.tx_indptr)), docs.tx_idx] = 1
        want = sum(np.where((kw[:, j] >= 0) & (kw[:, j] < vocab), held[:, np.clip(kw[:, j], 0, vocab - 1)], 0).T for j in range(16))
        with_kw = ix.stage_score_bounds(q, pw, torch.from_numpy(kw).cuda())
        assert np.array_equal((with_kw.view(torch.int32) & 31).cpu().numpy(), want)
        assert ((with_kw.view(torch.int32) & ~31).view(torch.float32).double() >= sc).all()
    ix.close()


# one pass over the documents' columns for up to 64 queries: 32 and 64 of them, two to seven chunks of 64 columns, read two at a time
@pytest.mark.parametrize("nq", [1, 31, 32, 33, 64, 65])
@pytest.mark.parametrize("n,dim,vocab,bf16", [(255, 64, 30, False), (257, 72, 30, True), (300, 192, 30, True), (1, 128, 40, False), (256, 260, 30, False), (513, 320, 60, True)])
def test_bounds_of_few_queries(n, dim, vocab, bf16, nq):
    rng = np.random.default_rng(dim + nq)
    def vecs(m):
        ip, idx, val = _lists(rng, m, np.full(m, 9), 0, vocab)
        ip2, idx2, _ = _lists(rng, m, np.full(m, 7), 0, vocab)
        return VecSet(m, dim, rng.standard_normal((m, dim)).astype(np.float32), ip, idx, val, ip2, idx2, rng.integers(1, 4, len(idx2)).astype(np.float32), vocab, vocab)
    docs, queries = vecs(n), vecs(nq)
    if bf16:
        bits = torch.from_numpy(docs.dense).bfloat16()
        docs.dense, docs.dense_bf16 = bits.float().numpy(), bits.view(torch.int16).numpy().view(np.uint16)
    ix, q = B.Index.ingest(B.DeviceVecs(docs, bf16=bf16), B.build_params(8)), B.DeviceVecs(queries)
    pw = rng.uniform(-1.0, 1.0, (nq, 3)).astype(np.float32)
    sc = ix.hybrid_scores(q, np.tile(np.arange(n, dtype=np.int32), (nq, 1)), pw)[:, :, 3].double()
    up = ix.stage_score_bounds(q, pw).double()
    assert (up >= sc).all() and (up - sc <= _slack(ix, queries, docs, pw, bf16)).all()
    ix.close()


# documents of lists so long that a tile's postings get more than 2^13 buckets, and any number of buckets on the same lists: buckets that one
# lane reads, that a query's eight lanes read together (a term that most documents hold), lists of queries in the middle of a batch of 32
@pytest.mark.parametrize("buckets", [0, 8, 13, 15])
@pytest.mark.parametrize("n,vocab,doc_terms,nq", [(300, 3_000, 700, 65), (513, 20_000, 500, 300), (256, 1_500, 1_000, 20)])
def test_long_lists(debug_knobs, n, vocab, doc_terms, nq, buckets):
    rng, dim = np.random.default_rng(n + nq), 64
    lengths = np.resize([0, 40, 127, 129, 160, 161, 400, 1000], nq)
    def vecs(m, sp, tx):
        tx = (tx[0], tx[1], rng.integers(1, 4, len(tx[1])).astype(np.float32))
        return VecSet(m, dim, rng.standard_normal((m, dim)).astype(np.float32) / 8, *sp, *tx, vocab, vocab)
    docs = vecs(n, _lists(rng, n, rng.integers(doc_terms // 2, doc_terms, n), 0, vocab), _lists(rng, n, rng.integers(doc_terms // 2, doc_terms, n), 0, vocab))
    queries = vecs(nq, _lists(rng, nq, lengths, 0, vocab), _lists(rng, nq, lengths[::-1], 0, vocab))
    debug_knobs("bound_buckets", buckets)
    ix, q = B.Index.ingest(B.DeviceVecs(docs), B.build_params(8)), B.DeviceVecs(queries)
    pw = rng.uniform(-1.0, 1.0, (nq, 3)).astype(np.float32)
    sc = ix.hybrid_scores(q, np.tile(np.arange(n, dtype=np.int32), (nq, 1)), pw)[:, :, 3].double()
    up = ix.stage_score_bounds(q, pw).double()
    assert (up >= sc).all() and (up - sc <= _slack(ix, queries, docs, pw, False)).all()
    # required terms without a column: rarer than the 512th of both vocabularies' frequencies by more than a bin of them is wide (an eighth)
    df = [np.bincount(i, minlength=vocab) for i in (docs.sp_idx, docs.tx_idx)]
    rare = np.flatnonzero((df[1] > 0) & (df[1] < np.sort(np.concatenate(df))[::-1][512] / 2))
    if not len(rare):
        rare = np.array([vocab + 5])   # all alike: none is sure to have no column
    kw = rng.choice(rare, (nq, 13)).astype(np.int32)
    kw[::3, 3], kw[1::3, 9:] = vocab + 5, -1
    held = np.zeros((n, vocab), np.int32)
    held[np.repeat(np.arange(n), np.diff(docs.tx_indptr)), docs.tx_idx] = 1
    want = sum(np.where((kw[:, j] >= 0) & (kw[:, j] < vocab), held[:, np.clip(kw[:, j], 0, vocab - 1)], 0).T for j in range(13))
    with_kw = ix.stage_score_bounds(q, pw, torch.from_numpy(kw).cuda())
    assert np.array_equal((with_kw.view(torch.int32) & 31).cpu().numpy(), want)
    assert ((with_kw.view(torch.int32) & ~31).view(torch.float32).double() >= sc).all()
    ix.close()


def test_long_lists_get_the_buckets_they_need(debug_knobs):
    """1,250 entries a document: with 2^13 buckets a lookup reads past tens of entries, which costs a quarter of the time and more."""
    rng, n, nq, vocab = np.random.default_rng(2), 10_240, 1024, 250_000
    def vecs(m, terms):
        lists = []
        for _ in range(2):   # strictly ascending ids: a random start and steps below the vocabulary's share
            steps = rng.integers(1, vocab // terms, (m, terms))
            lists.append((np.arange(m + 1, dtype=np.int64) * terms, (np.cumsum(steps, 1) - 1).astype(np.int32).ravel()))
        (ip, idx), (ip2, idx2) = lists
        return VecSet(m, 64, rng.standard_normal((m, 64)).astype(np.float32), ip, idx, rng.random(len(idx)).astype(np.float32), ip2, idx2,
                      np.ones(len(idx2), np.float32), vocab, vocab)
    docs, q = B.DeviceVecs(vecs(n, 625)), B.DeviceVecs(vecs(nq, 400))
    pw = np.ones((nq, 3), np.float32)
    took = {}
    for buckets in (0, 13, 15):
        debug_knobs("bound_buckets", buckets)
        ix = B.Index.ingest(docs, B.build_params(8))
        times = []
        for _ in range(6):
            a, b = torch.cuda.Event(True), torch.cuda.Event(True)
            a.record(); ix.stage_score_bounds(q, pw); b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b))
        took[buckets] = min(times[1:])
        ix.close()
    print(took, flush=True)
    assert took[0] <= 1.1 * min(took.values()), took
