"""The table of upper bounds: never below a score that the scoring kernels give, no further above it than its rounding
allows, and searches that use it return the same ids, scores and counts of scored documents, bit for bit, as searches
that score every neighbour."""
import threading
import time

import numpy as np
import pytest
import torch

from paper_2511_00855_amd import binding as B
from paper_2511_00855_amd.synth import VecSet, make_keywords, make_workload, subset_vecset

pytestmark = pytest.mark.gpu


def _workload(base, **kw):
    w = make_workload(base, seed=11, **kw)
    bf16 = getattr(w.docs, "dense_bf16", None) is not None
    return w, B.DeviceVecs(w.docs, bf16=bf16), B.DeviceVecs(w.queries)


def _slack(ix, q, d, weights, bf16):
    """The most a bound may lie above its score, per query and document.  Rounding x to x^ in bf16 takes |x - x^| off a part; a
    product of two rounded parts is off by |q - q^| |d| + |q^| |d - d^| at most, the bound adds as much again, and 1e-3 of the
    norms is more than all sums in 32 bits take (the parts here are whole lists, of which the head is rounded)."""
    dev = ix.device
    t = lambda a: torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float32, device=dev)
    txw = ix.export_ingest()[0]
    out = 0.0
    for p, (qi, qv, di, dv) in enumerate(((None, q.dense, None, d.dense), (q.sp_indptr, q.sp_val, d.sp_indptr, d.sp_val),
                                          (q.tx_indptr, q.tx_val, d.tx_indptr, txw))):
        def norms(ip, v, w):   # of the values, of the rounded ones, of the difference
            rows = torch.arange(v.shape[0], device=dev) if ip is None else \
                torch.repeat_interleave(torch.arange(len(ip) - 1, device=dev), torch.as_tensor(np.diff(ip), device=dev))
            n = v.shape[0] if ip is None else len(ip) - 1
            x = v if w is None else (v * (w[:, None] if ip is None else w[rows]))
            y = x.bfloat16().float()
            sq = [(z.double() ** 2).sum(1) if ip is None else torch.zeros(n, dtype=torch.float64, device=dev).index_add_(0, rows, z.double() ** 2)
                  for z in (x, y, x - y)]
            return [z.sqrt() for z in sq]
        qn, qr, qd = [z[:, None] for z in norms(qi, t(qv), t(weights[:, p]))]
        dn, _, dd = [z[None, :] for z in norms(di, dv if torch.is_tensor(dv) else t(dv), None)]
        if p == 0 and bf16:
            dd = torch.zeros_like(dd)
        out = out + 2 * (qd * dn + qr * dd) + 1e-3 * qn * dn
    return out + 1e-12


# tiles of 256 x 256, chunks of 64 columns, at most 512 head columns: below, at and above their edges; a vocabulary that is
# all head, one of which nearly nothing is
@pytest.mark.parametrize("base,n,nq,dim,vocab", [("tiny", 1, 1, 4, 50), ("tiny", 255, 257, 64, 300), ("tiny", 257, 255, 260, 10_000),
                                                 ("cfg2", 1300, 40, 768, 30_522), ("cfg3", 513, 20, 520, 5_000),
                                                 ("cfg3", 512, 256, 1024, 250_002), ("cfg3", 700, 3, 8, 1_000)])
def test_bounds_hold_and_are_tight(base, n, nq, dim, vocab):
    w, docs, qs = _workload(base, n=n, nq=nq, dim=dim, vocab=vocab, **({} if vocab > 400 else dict(sp=("fixed", 12), tx=("fixed", 10))))
    ix = B.Index.ingest(docs, B.build_params(8))
    rng = np.random.default_rng(3)
    cand = np.tile(np.arange(n, dtype=np.int32), (nq, 1))
    for weights in (rng.uniform(0.05, 1.0, (nq, 3)), rng.uniform(-1.0, 1.0, (nq, 3)), np.tile([0.0, 0.0, 1.0], (nq, 1)), np.tile([1e-6, 3e4, 0.0], (nq, 1))):
        pw = weights.astype(np.float32)
        sc = ix.hybrid_scores(qs, cand, pw).double()
        up = ix.stage_score_bounds(qs, pw).double()
        torch.cuda.synchronize()
        assert (up >= sc[:, :, 3]).all()
        assert (up - sc[:, :, 3] <= _slack(ix, w.queries, w.docs, pw, docs.dtype == B.AP_BF16)).all()
    ix.close()


def _rounded_most(rng, n):
    """Values that lose nearly 2^-8 when they are rounded to bf16 (just below the middle between two neighbours, and above
    it), and ordinary ones."""
    v = 1.0 + 2.0 ** -8 + rng.choice([-1.0, 1.0], n) * rng.integers(1, 64, n) * 2.0 ** -18
    return np.where(rng.random(n) < 0.5, v, 1.0 + rng.random(n)).astype(np.float32)


@pytest.mark.parametrize("n,dim,bf16", [(4500, 64, False), (4200, 100, False), (4300, 1024, True), (4100, 72, True)])
def test_bounds_hold_where_rounding_takes_most(debug_knobs, n, dim, bf16):
    """One-term lists and rows of one magnitude, signs aligned: every rounding error of a product points the same way, and the
    inequality the slack comes from is all but an equation."""
    rng, nq = np.random.default_rng(17), 96
    sign = rng.choice([-1.0, 1.0], dim).astype(np.float32)
    def vecs(m):
        dense = sign * _rounded_most(rng, m)[:, None] / np.float32(np.sqrt(dim))
        term = np.arange(m, dtype=np.int32) % 2   # two terms, half of the documents each (a term of all has a BM25 weight of nearly nothing)
        ip = np.arange(m + 1, dtype=np.int64)
        return VecSet(m, dim, dense.astype(np.float32), ip, term + 5, _rounded_most(rng, m), ip, term + 3, _rounded_most(rng, m), 50, 50)
    d, q = vecs(n), vecs(nq)
    if bf16:
        bits = torch.from_numpy(d.dense).bfloat16()
        d.dense, d.dense_bf16 = bits.float().numpy(), bits.view(torch.int16).numpy().view(np.uint16)
    docs, qs = B.DeviceVecs(d, bf16=bf16), B.DeviceVecs(q)
    ix = B.Index.build(docs, B.build_params(16, nd_rounds=1, n_entry=16))
    cand = np.tile(np.arange(n, dtype=np.int32), (nq, 1))
    scale = _rounded_most(rng, nq * 3).reshape(nq, 3)
    for which in ([1, 0, 0], [0, 1, 0], [0, 0, 1], [-1, 0, 0], [0, -1, 1], [1, 1, 1]):
        pw = (scale * np.float32(which)).astype(np.float32)
        print(which, flush=True)
        sc = ix.hybrid_scores(qs, cand, pw)[:, :, 3]
        up = ix.stage_score_bounds(qs, pw).double()
        assert (up >= sc.double()).all(), (which, ((sc.double() - up) / sc.double().abs().clamp(min=1e-9)).max())
        assert (up - sc.double() <= _slack(ix, q, d, pw, bf16)).all(), which
        for k in (1, 200):
            ids, got = ix.bruteforce_topk(qs, k, pw)
            want, at = torch.sort(sc, dim=1, descending=True, stable=True)
            assert torch.equal(got, want[:, :k]) and torch.equal(ids, at[:, :k].to(torch.int32)), (which, k)
        for k, beam, width in ((10, 64, 1), (50, 2000, 4)):
            got = []
            for mode in (1, 2):
                debug_knobs("search_bounds", mode)
                got.append([t.clone() for t in ix.search_batch(qs, k, beam, pw, search_width=width)])
            debug_knobs("search_bounds", 0)
            assert all(torch.equal(a, b) for a, b in zip(*got)), (which, beam)
    ix.close()


@pytest.mark.parametrize("base,n,dim,vocab", [("tiny", 1500, 128, 10_000), ("cfg2", 2100, 260, 30_522), ("cfg3", 1100, 520, 5_000), ("cfg3", 900, 128, 250_002)])
def test_searches_with_and_without_bounds_are_the_same(debug_knobs, base, n, dim, vocab):
    w, docs, qs = _workload(base, n=n, nq=70, dim=dim, vocab=vocab)
    ix = B.Index.build(docs, B.build_params(16, nd_rounds=2, n_entry=16))
    pw = np.random.default_rng(5).uniform(-0.3, 1.0, (qs.n, 3)).astype(np.float32)
    kw = make_keywords(w.queries, seed=6, max_terms=3, stride=4, p_none=0.1)
    kw[3] = [-1, 2 ** 30, w.docs.tx_vocab, -5]     # terms that no document can hold
    for k, beam, width, iters in ((10, 16, 1, 0), (5, 64, 3, 0), (10, 200, 16, 7), (1, 1, 1, 0), (10, 150, 2, 0), (10, n + 50, 16, 0)):
        got = {}
        for mode in (1, 2):
            debug_knobs("search_bounds", mode)
            out = []
            for weights in (pw, np.abs(pw)):
                out += list(ix.search_batch(qs, k, beam, weights, search_width=width, max_iters=iters))
                out.append(ix.search_stats(qs.n)[0][:, :2].clone())
                for kw_all in (False, True):
                    out += list(ix.search_batch_keywords(qs, k, beam, kw, weights, kw_all=kw_all, search_width=min(width, 4), max_iters=iters))
                    out.append(ix.search_stats(qs.n)[0][:, :2].clone())
            got[mode] = [t.clone() for t in out]
        debug_knobs("search_bounds", 0)
        assert all(torch.equal(a, b) for a, b in zip(got[1], got[2])), (k, beam, width, iters)
    # slabs of queries, each with a table of its own
    debug_knobs("search_bounds", 2)
    ref = [t.clone() for t in ix.search_batch(qs, 10, 64, pw)]
    debug_knobs("search_workspace_bytes", 9 * 4 * ((n + 31) // 32))
    for _ in range(2):
        assert all(torch.equal(a, b) for a, b in zip(ref, ix.search_batch(qs, 10, 64, pw)))
    ix.close()


@pytest.mark.parametrize("base,n,dim", [("tiny", 6007, 96), ("cfg3", 6100, 256)])
def test_large_pools_with_a_floor_are_the_same(debug_knobs, base, n, dim):
    """Workgroups of 512 and 1,024 threads: without bounds; with them and a floor; no neighbour waits; the floor is so high
    that everything that waits has to be scanned for (in several rounds: more waits than the candidates' array holds)."""
    w, docs, qs = _workload(base, n=n, nq=33, dim=dim, vocab=5_000)
    ix = B.Index.build(docs, B.build_params(64, nd_rounds=1, n_entry=16))
    pw = np.random.default_rng(5).uniform(-0.2, 1.0, (qs.n, 3)).astype(np.float32)
    for k, beam, width, iters in ((10, 800, 16, 0), (10, 900, 16, 9), (1, 4300, 2, 0), (50, 5900, 16, 0), (10, 9000, 16, 0), (10, 12000, 1, 0)):
        got = {}
        for mode, floor in ((1, 0), (2, 0), (2, 1), (2, 2)):
            debug_knobs("search_bounds", mode)
            debug_knobs("search_floor", floor)
            out = list(ix.search_batch(qs, k, beam, pw, search_width=width, max_iters=iters))
            got[mode, floor] = [t.clone() for t in out] + [ix.search_stats(qs.n)[0][:, :2].clone()]
        debug_knobs("search_bounds", 0)
        debug_knobs("search_floor", 0)
        for key in got:
            assert all(torch.equal(a, b) for a, b in zip(got[1, 0], got[key])), (key, k, beam, width, iters)
    ix.close()


@pytest.mark.parametrize("bf16", [False, True])
def test_rows_that_are_not_finite_are_scored(debug_knobs, bf16):
    """Infinities and NaN of either sign in a third of the dense rows: bounds that compare with nothing keep nothing out.  The
    order of such scores is that of their keys (a NaN with the sign bit ranks last), with and without bounds."""
    n, nq, dim = 6007, 25, 64
    w, _, qs = _workload("tiny", n=n, nq=nq, dim=dim, vocab=5_000)
    rng, d = np.random.default_rng(6), w.docs
    bits = d.dense.view(np.uint32)
    bits &= np.uint32(0xffff0000)    # bf16 values in either case
    rows = rng.permutation(n)[:n // 3]
    bits[rows, rng.integers(0, dim, len(rows))] = rng.choice(np.array([0x7f800000, 0xff800000, 0x7fc00000, 0xffc00000, 0xffc00000, 0xffc00000, 0xffc00000], np.uint32), len(rows))
    if bf16:
        d.dense_bf16 = (bits >> 16).astype(np.uint16)
    docs = B.DeviceVecs(d, bf16=bf16)
    ix = B.Index.import_graph(docs, B.build_params(64, n_entry=16), rng.integers(0, n, (n, 64)).astype(np.int32), rng.permutation(n)[:16].astype(np.int32))
    pw = rng.uniform(0.1, 1.0, (nq, 3)).astype(np.float32)
    bytes_of = lambda t: t.view(torch.int32) if t.dtype == torch.float32 else t
    for k, beam, width in ((10, 64, 2), (10, 800, 16), (100, 4300, 2), (1, 9000, 16)):
        got = {}
        for mode, floor in ((1, 0), (2, 0), (2, 1), (2, 2)):
            debug_knobs("search_bounds", mode)
            debug_knobs("search_floor", floor)
            out = ix.search_batch(qs, k, beam, pw, search_width=width)
            got[mode, floor] = [bytes_of(t).clone() for t in out] + [ix.search_stats(nq)[0][:, :2].clone()]
        for key in got:
            assert all(torch.equal(a, b) for a, b in zip(got[1, 0], got[key])), (key, k, beam, width)
    debug_knobs("search_bounds", 0)
    debug_knobs("search_floor", 0)
    full = [bytes_of(t) for t in ix.bruteforce_topk(qs, 257, pw)]   # more than the bounds are used for: every document scored
    for k in (1, 10, 200):
        assert all(torch.equal(a[:, :k], bytes_of(b)) for a, b in zip(full, ix.bruteforce_topk(qs, k, pw))), k
    ix.close()


@pytest.mark.parametrize("where", ["dense", "lists"])
def test_partial_sums_that_overflow(debug_knobs, where):
    """Sums of the scoring kernels that are infinite although the bounds' are not: weights that make up for values beyond the
    range only after the sum, and products of 3e38 of either sign in an order in which they cancel."""
    n, nq, dim, rng = 2000, 20, 64, np.random.default_rng(9)
    d, q = _one_term(rng, n, dim), _one_term(rng, nq, dim)
    far = rng.permutation(n)[:40]
    if where == "dense":
        q.dense[:, 4] = np.float32(1e30)
        d.dense[:, 4] = 0.0
        d.dense[far, 4] = np.float32(1e9)
    else:   # entries 0 and 64 of a list are summed by one lane, 1 and 66 by others; the bounds add the terms in ascending order
        terms = 600   # as frequent as each other, more than there are columns: none has one
        d.sp_indptr = np.arange(0, n * terms + 1, terms, dtype=np.int64)
        d.sp_idx = np.tile(np.arange(terms, dtype=np.int32) * 3, n)
        val = np.ones((n, terms), np.float32)
        val[far[:, None], [0, 1, 64, 66]] = np.float32(1.7e19) * np.array([1, -1, 1, -1], np.float32)
        d.sp_val, d.sp_vocab, q.sp_vocab = val.reshape(-1), 1800, 1800
        q.sp_indptr = np.arange(0, nq * 4 + 1, 4, dtype=np.int64)
        q.sp_idx, q.sp_val = np.tile(np.array([0, 3, 192, 198], np.int32), nq), np.full(nq * 4, np.float32(1.7e19))
    docs, qs = B.DeviceVecs(d), B.DeviceVecs(q)
    ix = B.Index.import_graph(docs, B.build_params(64, n_entry=16), rng.integers(0, n, (n, 64)).astype(np.int32), rng.permutation(n)[:16].astype(np.int32))
    for pw in (np.ones((nq, 3)), np.tile([1e-20, 1e-20, 1.0], (nq, 1))):
        pw = pw.astype(np.float32)
        sc = ix.hybrid_scores(qs, np.tile(np.arange(n, dtype=np.int32), (nq, 1)), pw)[:, :, 3]
        up = ix.stage_score_bounds(qs, pw)
        assert bool(torch.isinf(sc).any()) and not bool((up < sc).any())
        got = []
        for mode in (1, 2):
            debug_knobs("search_bounds", mode)
            got.append([t.view(torch.int32).clone() for t in ix.search_batch(qs, 10, 64, pw)])
        debug_knobs("search_bounds", 0)
        assert all(torch.equal(a, b) for a, b in zip(*got))
    ix.close()


def test_what_waits_comes_before_scores_that_are_no_numbers(debug_knobs):
    """A hundred documents above the floor lead to 300 that wait below it and to 100 whose score is a NaN that ranks last; the
    first lead to 700 more, the second to 500 that score higher.  Those that wait are expanded before the NaN are, and push
    them out of the pool: the 500 are never met."""
    n, R, nq, L = 20_000, 64, 3, 800
    rng = np.random.default_rng(1)
    d, q = _one_term(rng, n, 64), _one_term(rng, nq, 64)
    d.dense[:] = 0.0
    q.dense[:] = 0.0
    q.dense[:, 0] = 1.0
    top, W, X, N, Y = np.arange(100), 2000 + np.arange(300), 3000 + np.arange(700), 4000 + np.arange(100), 5000 + np.arange(500)
    d.dense[:1200, 0] = 1.2     # what the estimate of the floor is made of: a twentieth of the documents
    for group, score in ((top, 2.0), (W, 0.5), (X, 0.4), (Y, 0.6)):
        d.dense[group, 0] = score - 1e-4 * np.arange(len(group))
    d.dense.view(np.uint32)[N, 1] = 0xffc00000
    graph = np.full((n, R), -1, np.int32)
    for j in range(100):   # the first 80, which are expanded first, know only their like: waiting has begun when the others are met
        graph[top[j]] = top[(j + 1 + np.arange(R)) % 100] if j < 80 else np.concatenate([W[(15 * (j - 80) + np.arange(44)) % 300], N[(5 * (j - 80) + np.arange(20)) % 100]])
        graph[N[j]] = Y[(5 * j + np.arange(R)) % 500]
    for j in range(300):
        graph[W[j]] = X[(3 * j + np.arange(R)) % 700]
    docs, qs = B.DeviceVecs(d), B.DeviceVecs(q)
    ix = B.Index.import_graph(docs, B.build_params(R, n_entry=16), graph, top[:16].astype(np.int32))
    pw = np.tile(np.float32([1.0, 0.0, 0.0]), (nq, 1))
    got = {}
    for mode, floor in ((1, 0), (2, 0), (2, 1)):
        debug_knobs("search_bounds", mode)
        debug_knobs("search_floor", floor)
        got[mode, floor] = [t.clone() for t in ix.search_batch(qs, L, L, pw, search_width=16)] + [ix.search_stats(nq)[0][:, :2].clone()]
    ids = got[1, 0][0].cpu().numpy()
    assert set(ids[0]) == set(top) | set(W) | set(ids[0][400:]) and set(ids[0][400:]) <= set(X)
    for key in got:
        assert all(torch.equal(a, b) for a, b in zip(got[1, 0], got[key])), key
    ix.close()


def test_slabs_of_the_table_and_a_captured_search(debug_knobs):
    """A table that holds some twenty of 70 queries: the search runs in slabs, each with a table of its own.  A captured search
    goes without bounds, and after such a search of the same batch it needs no memory that is not there."""
    n = 1500
    w, docs, qs = _workload("tiny", n=n, nq=70)
    ix = B.Index.build(docs, B.build_params(16, nd_rounds=2, n_entry=16))
    rng = np.random.default_rng(4)
    pws = [torch.from_numpy(rng.uniform(-0.2, 1.0, (qs.n, 3)).astype(np.float32)).to(docs.device) for _ in range(3)]
    debug_knobs("search_visited_global", 1)   # a corpus this small would keep its visited sets in LDS
    debug_knobs("search_bounds", 2)
    debug_knobs("search_bounds_bytes", 256 * (2 * (128 + 512) + 36) + 20 * 4 * 1536)
    got = [[t.clone() for t in ix.search_batch(qs, 10, 96, p, search_width=2)] for p in pws]
    torch.cuda.synchronize()
    pw, out = pws[0].clone(), [t.clone() for t in got[0]]
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        ix.search_batch(qs, 10, 96, pw, search_width=2, out=out)
    debug_knobs("search_bounds", 1)
    want = [[t.clone() for t in ix.search_batch(qs, 10, 96, p, search_width=2)] for p in pws]
    for i in (0, 2, 1, 1, 0):
        pw.copy_(pws[i])
        for t in out:
            t.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(out, want[i])), i
        assert all(torch.equal(a, b) for a, b in zip(got[i], want[i])), i
    ix.close()


def test_two_streams_search_one_index_with_tables_of_their_own(debug_knobs):
    w, docs, qs = _workload("tiny", n=3000, nq=60)
    ix = B.Index.build(docs, B.build_params(16, nd_rounds=2, n_entry=16))
    rng = np.random.default_rng(8)
    pws = [torch.from_numpy(rng.uniform(0.1, 1.0, (qs.n, 3)).astype(np.float32)).to(docs.device) for _ in range(2)]
    debug_knobs("search_bounds", 1)
    ref = [[t.clone() for t in ix.search_batch(qs, 10, 96, p)] for p in pws]
    debug_knobs("search_bounds", 2)
    streams = [torch.cuda.Stream() for _ in range(2)]
    torch.cuda.synchronize()
    outs = [[], []]
    for _ in range(5):
        for i, s in enumerate(streams):
            with torch.cuda.stream(s):
                outs[i].append(ix.search_batch(qs, 10, 96, pws[i]))
    torch.cuda.synchronize()
    for i in range(2):
        for o in outs[i]:
            assert all(torch.equal(a, b) for a, b in zip(o, ref[i]))
    ix.close()


def test_a_search_does_not_wait_on_the_host_for_an_exact_topk(debug_knobs):
    """Weights of zero: every document ties, which the bounds leave undecided, and every document is scored.  Meanwhile another
    thread enqueues a search of the same index on another stream."""
    n, nq = 20_000, 20_000
    w, docs, qs = _workload("tiny", n=n, nq=nq, dim=32, sp=("fixed", 2), tx=("fixed", 2))
    few = B.DeviceVecs(subset_vecset(w.queries, np.arange(20)))
    ix = B.Index.build(docs, B.build_params(16, nd_rounds=1, n_entry=16))
    debug_knobs("search_bounds", 2)
    streams = [torch.cuda.Stream() for _ in range(2)]
    zero = torch.zeros((nq, 3), device=docs.device)
    out = None
    for _ in range(2):   # workspaces are there afterwards
        with torch.cuda.stream(streams[1]):
            out = ix.search_batch(few, 10, 64, out=out)
        torch.cuda.synchronize()
    t = {}

    def exact():
        with torch.cuda.stream(streams[0]):
            t["begin"] = time.perf_counter()
            t["ids"] = ix.bruteforce_topk(qs, 100, zero)[0]
            t["end"] = time.perf_counter()
    for _ in range(2):   # the first call also loads its kernels
        exact()
        torch.cuda.synchronize()
    took = t["end"] - t["begin"]
    assert torch.equal(t["ids"], torch.arange(100, dtype=torch.int32, device=docs.device).repeat(nq, 1))
    th = threading.Thread(target=exact)
    th.start()
    time.sleep(0.2 * took)
    with torch.cuda.stream(streams[1]):
        t0 = time.perf_counter()
        ix.search_batch(few, 10, 64, out=out)
        t1 = time.perf_counter()
    th.join()
    torch.cuda.synchronize()
    print(f"exact top-k {took * 1e3:.1f} ms, the search's call {(t1 - t0) * 1e3:.2f} ms, begun {(t['end'] - t0) * 1e3:.1f} ms before its end")
    assert t0 < t["end"] and t1 - t0 < 0.5 * (t["end"] - t0)
    ix.close()


def _one_term(rng, n, dim):
    """n rows of a few columns with lists of one term: what a test needs that is about amounts of memory."""
    ip = np.arange(n + 1, dtype=np.int64)
    dense = rng.standard_normal((n, dim)).astype(np.float32)
    return VecSet(n, dim, dense, ip, rng.integers(0, 50, n).astype(np.int32), np.ones(n, np.float32), ip, rng.integers(0, 50, n).astype(np.int32),
                  np.ones(n, np.float32), 50, 50)


def _many_terms(n, dim, terms=60):
    """As _one_term, with lists of 60 of 400 terms."""
    rng = np.random.default_rng(2)
    d = _one_term(rng, n, dim)
    d.sp_indptr = d.tx_indptr = np.arange(0, n * terms + 1, terms, dtype=np.int64)
    d.sp_idx = d.tx_idx = np.tile(np.arange(terms, dtype=np.int32), n) + np.repeat(rng.integers(0, 340, n).astype(np.int32), terms)
    d.sp_val = d.tx_val = np.ones(n * terms, np.float32)
    d.sp_vocab = d.tx_vocab = 400
    return d


def _leave_free(want):
    """Tensors that leave about `want` bytes of the device's memory free."""
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    hold = []
    while torch.cuda.mem_get_info()[0] > want + (4 << 20):
        hold.append(torch.empty(max(torch.cuda.mem_get_info()[0] - want, 2 << 20), dtype=torch.uint8, device="cuda:0"))
    print("free", torch.cuda.mem_get_info()[0] >> 20, "MB", flush=True)
    return hold


def test_the_table_takes_a_share_of_the_free_memory(debug_knobs):
    rng, nq = np.random.default_rng(2), 10_000
    d = _one_term(rng, 20_000, 16)
    docs, qs = B.DeviceVecs(d), B.DeviceVecs(_one_term(rng, nq, 16))
    ix = B.Index.build(docs, B.build_params(16, nd_rounds=1, n_entry=16))
    debug_knobs("search_bounds", 1)
    want = [t.clone() for t in ix.search_batch(qs, 5, 32)]
    out = [t.clone() for t in want]
    torch.cuda.synchronize()
    hold = _leave_free(2 << 30)
    free0 = torch.cuda.mem_get_info()[0]
    assert 1 << 30 < free0 < 3 << 30
    debug_knobs("search_bounds", 2)
    for _ in range(2):   # a table of all queries would be 0.8 GB
        ix.search_batch(qs, 5, 32, out=out)
        torch.cuda.synchronize()
        taken = free0 - torch.cuda.mem_get_info()[0]
        assert all(torch.equal(a, b) for a, b in zip(out, want))
        assert 0 < taken <= free0 // 4 + (8 << 20), taken
    del hold
    torch.cuda.empty_cache()
    ix.close()


def test_an_exact_topk_gets_the_memory_of_its_table_for_its_scores():
    """All documents tie: the scores of all queries, 2 GiB at a time, fit what is free, but not beside the table of bounds that
    left them undecided."""
    rng, n, nq = np.random.default_rng(2), 20_000, 30_000
    docs, qs = B.DeviceVecs(_one_term(rng, n, 16)), B.DeviceVecs(_one_term(rng, nq, 16))
    ix = B.Index.ingest(docs, B.build_params(8))
    zero = torch.zeros((nq, 3), device=docs.device)
    hold = _leave_free(2300 << 20)
    ids, sc = ix.bruteforce_topk(qs, 2, zero)
    del hold
    torch.cuda.empty_cache()
    assert torch.equal(ids, torch.arange(2, dtype=torch.int32, device=docs.device).repeat(nq, 1)) and (sc == 0).all()
    ix.close()


def test_a_search_gets_the_memory_of_its_table_for_its_visited_sets(debug_knobs):
    rng, n = np.random.default_rng(2), 20_000
    q = _one_term(rng, 30_000, 16)
    docs, qs, few = B.DeviceVecs(_one_term(rng, n, 16)), B.DeviceVecs(q), B.DeviceVecs(subset_vecset(q, np.arange(5000)))
    ix = B.Index.build(docs, B.build_params(16, nd_rounds=1, n_entry=16))
    out = (torch.empty((qs.n, 5), dtype=torch.int32, device=docs.device), torch.empty((qs.n, 5), device=docs.device))
    debug_knobs("search_visited_global", 1)
    debug_knobs("search_bounds", 2)
    small = [t.clone() for t in ix.search_batch(few, 5, 32)]   # visited sets 12.5 MB, a table of 400 MB
    hold = _leave_free(40 << 20)
    ix.search_batch(qs, 5, 32, out=out)                        # visited sets 75 MB
    torch.cuda.synchronize()
    del hold
    torch.cuda.empty_cache()
    assert all(torch.equal(a, b[:few.n]) for a, b in zip(small, out))
    ix.close()


def test_a_construction_has_the_memory_that_its_bounds_take_afterwards(debug_knobs):
    """The seed sweep multiplies half of D D^T where its buffers (80 MB here) fit 62 % of the free memory, and all of it where
    they do not.  With some 190 MB free at that
    point they fit, unless the columns of the bounds (80 MB) are there before."""
    d = _many_terms(20_000, 1024)
    docs, bp = B.DeviceVecs(d), B.build_params(16, knn_k=32, nd_rounds=0, n_entry=16)
    debug_knobs("seed_sample_cols", 2048)
    flops = {}
    for one_sided in (1, 0):
        debug_knobs("seed_one_sided", one_sided)
        ix = B.Index.build(docs, bp)
        flops[one_sided] = ix.build_counters()["seed_flops"]
        graph = [t.clone() for t in ix.export_graph()]
        ix.close()
    assert flops[0] < 0.8 * flops[1]
    hold = _leave_free(235 << 20)
    ix = B.Index.build(docs, bp)
    assert ix.build_counters()["seed_flops"] < 0.8 * flops[1]
    del hold
    torch.cuda.empty_cache()
    assert all(torch.equal(a, b) for a, b in zip(graph, ix.export_graph()))
    ix.close()


def test_an_insertion_has_the_memory_that_its_bounds_take():
    """With 380 MB free the columns of the bounds (80 MB) are less than a quarter of it, and what is left does not hold the pair
    similarities (260 MB) beside the lists."""
    d = _many_terms(20_000, 1024)
    docs = B.DeviceVecs(d)
    old = B.Index.build(B.DeviceVecs(subset_vecset(d, np.arange(19_000))), B.build_params(16, knn_k=256, nd_rounds=0, n_entry=16))
    new = old.insert(docs)
    graph = [t.clone() for t in new.export_graph()]
    new.close()
    hold = _leave_free(380 << 20)
    new = old.insert(docs)
    got = [t.clone() for t in new.export_graph()]
    new.close()
    del hold
    torch.cuda.empty_cache()
    assert all(torch.equal(a, b) for a, b in zip(graph, got))
    old.close()


def test_workspaces_of_single_calls_are_given_back(debug_knobs):
    rng, n, nq = np.random.default_rng(2), 20_000, 30_000
    d = _one_term(rng, n, 16)
    q = _one_term(rng, nq, 16)
    docs, qs, few = B.DeviceVecs(d), B.DeviceVecs(q), B.DeviceVecs(subset_vecset(q, np.arange(1000)))
    ix = B.Index.build(B.DeviceVecs(subset_vecset(d, np.arange(12_000))), B.build_params(16, nd_rounds=1, n_entry=16))
    debug_knobs("search_bounds", 2)
    torch.cuda.synchronize()
    free0 = torch.cuda.mem_get_info()[0]
    new = ix.insert(docs)         # searches for 8,000 documents among 20,000: a table of 640 MB
    torch.cuda.synchronize()
    free1 = torch.cuda.mem_get_info()[0]
    assert free0 - free1 < 200 << 20, free0 - free1
    small = new.bruteforce_topk(few, 3)     # 80 MB, which stay
    out = new.bruteforce_topk(qs, 3)        # 2.4 GB
    torch.cuda.synchronize()
    assert free1 - torch.cuda.mem_get_info()[0] < 200 << 20, free1 - torch.cuda.mem_get_info()[0]
    assert all(torch.equal(a, b[:1000]) for a, b in zip(small, out))
    ix.close(); new.close()


def test_any_number_of_streams_in_turn_search_with_bounds(debug_knobs):
    """A search with bounds decides more documents without their dense rows: every stream's does, and none beyond the first few
    takes more memory."""
    w, docs, qs = _workload("tiny", n=3000, nq=2000)
    ix = B.Index.build(docs, B.build_params(16, nd_rounds=2, n_entry=16))
    pw = torch.from_numpy(np.random.default_rng(8).uniform(0.1, 1.0, (qs.n, 3)).astype(np.float32)).to(docs.device)
    seen = {}
    for mode in (1, 2):
        debug_knobs("search_bounds", mode)
        out = ix.search_batch(qs, 10, 96, pw)
        seen[mode] = [t.clone() for t in out] + [ix.search_stats(qs.n)[0].clone()]
    assert seen[2][2][:, 2].sum() > seen[1][2][:, 2].sum()
    streams = [torch.cuda.Stream() for _ in range(9)]
    free = []
    for i in list(range(9)) + [0, 5]:
        torch.cuda.synchronize()
        with torch.cuda.stream(streams[i]):
            ix.search_batch(qs, 10, 96, pw, out=out)
        torch.cuda.synchronize()
        got = list(out) + [ix.search_stats(qs.n)[0]]
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(got, seen[2])), i
        free.append(torch.cuda.mem_get_info()[0])
    assert free[4] - min(free[4:]) < 16 << 20   # less than a table (25 MB); a stream has resources of its own
    ix.close()


@pytest.mark.parametrize("base,n,dim,k", [("tiny", 4096, 128, 1), ("tiny", 4097, 100, 10), ("cfg2", 4500, 768, 100), ("cfg3", 5000, 1024, 256),
                                          ("cfg3", 4200, 520, 10), ("tiny", 9001, 64, 37)])
def test_exact_topk_out_of_the_bounds(base, n, dim, k):
    """Against a sort of the scores of all documents (hybrid_scores): the same ids and the same bits."""
    w, docs, qs = _workload(base, n=n, nq=19, dim=dim, **({} if n < 9000 else dict(sp=("fixed", 1), tx=("fixed", 1))))
    if n >= 9000:   # every document the same: thousands of candidates tie, more than a workgroup lists
        docs.dense[:] = docs.dense[0]
        docs.sp_idx[:] = 7; docs.sp_val[:] = 1.0
        docs.tx_idx[:] = 3; docs.tx_val[:] = 1.0
    ix = B.Index.ingest(docs, B.build_params(8))
    for pw in (np.random.default_rng(1).uniform(0.1, 1.0, (qs.n, 3)), np.random.default_rng(2).uniform(-1.0, 1.0, (qs.n, 3)), np.zeros((qs.n, 3))):
        pw = pw.astype(np.float32)
        ids, sc = ix.bruteforce_topk(qs, k, pw)
        all_sc = ix.hybrid_scores(qs, np.tile(np.arange(n, dtype=np.int32), (qs.n, 1)), pw)[:, :, 3]
        want, at = torch.sort(all_sc, dim=1, descending=True, stable=True)    # equal scores: smaller id first
        assert torch.equal(sc, want[:, :k]) and torch.equal(ids, at[:, :k].to(torch.int32))
    ix.close()


def test_scattered_undecided_queries_of_an_exact_topk():
    """Weights of zero tie all documents, which the bounds leave undecided.  Every third query decided, the others not: the same
    results, and no slower than none decided."""
    n, nq, k = 20_000, 600, 20
    w, docs, qs = _workload("tiny", n=n, nq=nq, dim=32, sp=("fixed", 2), tx=("fixed", 2))
    ix = B.Index.ingest(docs, B.build_params(8))
    pw = np.random.default_rng(1).uniform(0.1, 1.0, (nq, 3)).astype(np.float32)
    pw[np.arange(nq) % 3 != 0] = 0
    took = {}
    for name, weights in (("none", np.zeros_like(pw)), ("some", pw)) * 2:
        weights = torch.from_numpy(weights).to(docs.device)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        ids, sc = ix.bruteforce_topk(qs, k, weights)
        torch.cuda.synchronize()
        took[name] = time.perf_counter() - t0
    print({a: f"{1e3 * b:.1f} ms" for a, b in took.items()})
    all_sc = ix.hybrid_scores(qs, np.tile(np.arange(n, dtype=np.int32), (nq, 1)), pw)[:, :, 3]
    want, at = torch.sort(all_sc, dim=1, descending=True, stable=True)
    assert torch.equal(sc, want[:, :k]) and torch.equal(ids, at[:, :k].to(torch.int32))
    assert took["some"] < 1.25 * took["none"]
    ix.close()


@pytest.mark.parametrize("w_k", [0.5, -0.4, 0.0])
def test_entity_searches_with_and_without_bounds_are_the_same(debug_knobs, w_k):
    from paper_2511_00855_amd.synth import make_entity_graph
    w, docs, qs = _workload("tiny", n=2500, nq=60)
    ix = B.Index.build(docs, B.build_params(16, nd_rounds=2, n_entry=16))
    kgs = make_entity_graph(2500, 60, seed=9, n_ent=300)
    ix.set_knowledge_graph(kgs, le_cap=16)
    pw = np.random.default_rng(5).uniform(-0.2, 1.0, (qs.n, 3)).astype(np.float32)
    for k, beam, hops in ((10, 16, 2), (5, 200, 0), (1, 64, 255)):
        got = []
        for mode in (1, 2):
            debug_knobs("search_bounds", mode)
            got.append([t.clone() for t in ix.search_batch_entities(qs, k, beam, kgs.q_ent, w_k, hops, pw)] + [ix.search_stats(qs.n)[0][:, :2].clone()])
        assert all(torch.equal(a, b) for a, b in zip(*got)), (k, beam, hops)
    ix.close()


def _plain_corpus(rng, n, nq, dim, vocab, terms, q_terms, degree):
    """Vector sets whose lists all have `terms` (`q_terms`) strictly ascending terms, and a random graph's index of the first."""
    def vecs(m, k):
        lists = [(np.cumsum(rng.integers(1, vocab // k, (m, k)), 1) - 1).astype(np.int32).ravel() for _ in range(2)]
        ip = np.arange(m + 1, dtype=np.int64) * k
        return VecSet(m, dim, rng.standard_normal((m, dim)).astype(np.float32), ip, lists[0], rng.random(m * k).astype(np.float32), ip, lists[1],
                      np.ones(m * k, np.float32), vocab, vocab)
    docs, qs = B.DeviceVecs(vecs(n, terms)), B.DeviceVecs(vecs(nq, q_terms))
    ix = B.Index.import_graph(docs, B.build_params(degree, n_entry=16), rng.integers(0, n, (n, degree)).astype(np.int32), rng.permutation(n)[:16].astype(np.int32))
    return ix, qs


def _way(debug_knobs, ix, qs, beam):
    """What a search's counters say without bounds, with them, and by the library's own choice; the answers are the same."""
    debug_knobs("search_walk", 1)
    pw, got, counts = np.ones((qs.n, 3), np.float32), {}, {}
    for mode in (1, 2, 0):
        debug_knobs("search_bounds", mode)
        got[mode] = [t.clone().view(torch.int32) for t in ix.search_batch(qs, min(10, beam), beam, pw)]
        counts[mode] = ix.search_stats(qs.n)[0][:, 2].clone()
    assert all(torch.equal(a, b) for mode in (2, 0) for a, b in zip(got[1], got[mode]))
    assert not torch.equal(counts[1], counts[2])
    return counts


# an iteration of few edges spares little by the bounds, and one of a few dozen queries as much as one of many
@pytest.mark.parametrize("n,nq,degree,beam,mode", [(40_960, 1024, 16, 16, 1), (40_960, 1024, 64, 16, 2), (250_000, 24, 64, 10, 2), (250_000, 24, 16, 10, 1)])
def test_small_pools_by_what_their_iterations_spare(debug_knobs, n, nq, degree, beam, mode):
    ix, qs = _plain_corpus(np.random.default_rng(n), n, nq, 64, 10_000, 20, 12, degree)
    counts = _way(debug_knobs, ix, qs, beam)
    assert torch.equal(counts[0], counts[mode])
    ix.close()


# a search without bounds reads the lists: the longer they are, the smaller the pool from which on bounds pay
@pytest.mark.parametrize("terms,mode", [(20, 1), (625, 2)])
def test_small_pools_by_the_length_of_the_lists(debug_knobs, terms, mode):
    ix, qs = _plain_corpus(np.random.default_rng(terms), 40_960, 1024, 64, 100_000, terms, 12, 32)
    counts = _way(debug_knobs, ix, qs, 6)
    assert torch.equal(counts[0], counts[mode])
    ix.close()


def test_small_pools_with_keywords(debug_knobs):
    """With keywords an iteration has half as many edges again: bounds pay from smaller pools on."""
    n, nq, degree, beam, rng = 40_960, 1024, 32, 6, np.random.default_rng(3)
    plain, qs = _plain_corpus(rng, n, nq, 64, 10_000, 20, 12, degree)
    sem, _, _, entry = plain.export_graph()
    edges = torch.randint(0, n, (n, degree // 2), generator=torch.Generator().manual_seed(3)).to(torch.int32)
    ix = B.Index.import_graph(plain.docs, B.build_params(degree, n_entry=16), sem, entry, edges, torch.full((n,), degree // 2, dtype=torch.int32))
    assert torch.equal(_way(debug_knobs, ix, qs, beam)[0], _way(debug_knobs, ix, qs, beam)[1])   # without keywords they do not
    kw = torch.randint(0, 10_000, (nq, 2), generator=torch.Generator().manual_seed(4)).to(torch.int32)
    got, counts = {}, {}
    for mode in (1, 2, 0):
        debug_knobs("search_bounds", mode)
        got[mode] = [t.clone().view(torch.int32) for t in ix.search_batch_keywords(qs, 5, beam, kw)]
        counts[mode] = ix.search_stats(nq)[0][:, 2].clone()
    assert all(torch.equal(a, b) for mode in (2, 0) for a, b in zip(got[1], got[mode]))
    assert torch.equal(counts[0], counts[2]) and not torch.equal(counts[0], counts[1])
    ix.close(); plain.close()
