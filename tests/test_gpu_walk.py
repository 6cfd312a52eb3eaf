"""Searches of small batches by the walk (scores first, then one wave a query) return the ids, scores, counts of scored
documents and of iterations of the searches that score as they go, bit for bit."""
import numpy as np
import pytest
import torch

from paper_2511_00855_amd import binding as B
from paper_2511_00855_amd.synth import make_workload

pytestmark = pytest.mark.gpu


def _searches(ix, qs, pw, calls):
    bits = lambda t: t.view(torch.int32) if t.dtype == torch.float32 else t   # a NaN compares by its bits
    out = []
    for k, beam, width in calls:
        out += [bits(t).clone() for t in ix.search_batch(qs, k, beam, pw, search_width=width)]
        out.append(ix.search_stats(qs.n)[0][:, :2].clone())
    return out


# degrees below, at and above a wave; a corpus smaller than the pool; more parents than the pool; visited sets in LDS and not
@pytest.mark.parametrize("base,n,dim,vocab,degree,n_entry", [("tiny", 1500, 128, 10_000, 16, 16), ("cfg2", 2100, 260, 30_522, 64, 64),
                                                             ("cfg3", 1100, 520, 5_000, 32, 100), ("cfg3", 900, 128, 250_002, 96, 7)])
@pytest.mark.parametrize("visited_global", [0, 1])
def test_walks_and_searches_are_the_same(debug_knobs, base, n, dim, vocab, degree, n_entry, visited_global):
    w = make_workload(base, seed=11, n=n, nq=41, dim=dim, vocab=vocab)
    docs, qs = B.DeviceVecs(w.docs, bf16=getattr(w.docs, "dense_bf16", None) is not None), B.DeviceVecs(w.queries)
    ix = B.Index.build(docs, B.build_params(degree, nd_rounds=1, n_entry=n_entry))
    pw = np.random.default_rng(5).uniform(-0.3, 1.0, (qs.n, 3)).astype(np.float32)
    calls = [(1, 1, 1), (10, 16, 1), (5, 64, 3), (10, 130, 16), (10, 257, 1), (50, 700, 4), (10, n + 50, 1), (10, n + 50, 16)]
    debug_knobs("search_visited_global", visited_global)
    for weights in (pw, np.abs(pw)):
        for deleted in (False, True):
            ix.mark_deleted(np.random.default_rng(7).permutation(n)[:n // 3].astype(np.int32), restore=not deleted)
            got = {}
            for mode in (1, 2, 3):
                debug_knobs("search_walk", mode)
                got[mode] = _searches(ix, qs, weights, calls)
            for mode in (2, 3):
                for i, (a, b) in enumerate(zip(got[1], got[mode])):
                    assert torch.equal(a, b), (mode, deleted, calls[i // 3], i % 3)
    ix.close()


def test_walks_that_start_again(debug_knobs):
    """Graphs of random edges with repeated neighbours and holes, scores that are infinities and NaN: searches that the first
    pass leaves undecided, and queries whose lists are longer than the tables in LDS."""
    n, nq, dim = 6007, 25, 64
    w = make_workload("tiny", seed=11, n=n, nq=nq, dim=dim, vocab=5_000)
    rng, d = np.random.default_rng(6), w.docs
    graph = rng.integers(-1, n, (n, 64)).astype(np.int32)
    graph[:, 1] = graph[:, 0]
    entry = rng.permutation(n)[:16].astype(np.int32)
    pw = rng.uniform(0.1, 1.0, (nq, 3)).astype(np.float32)
    calls = [(10, 64, 2), (10, 700, 16), (100, 1300, 1), (1, 33, 1)]
    for special in (False, True):
        if special:
            rows = rng.permutation(n)[:n // 3]
            d.dense.view(np.uint32)[rows, rng.integers(0, dim, len(rows))] = rng.choice(np.array([0x7f800000, 0xff800000, 0x7fc00000, 0xffc00000], np.uint32), len(rows))
        docs, qs = B.DeviceVecs(d), B.DeviceVecs(w.queries)
        ix = B.Index.import_graph(docs, B.build_params(64, n_entry=16), graph, entry)
        for lists in (0, 1):
            debug_knobs("search_query_lists", lists)
            got = {}
            for mode in (1, 2, 3):
                debug_knobs("search_walk", mode)
                got[mode] = _searches(ix, qs, pw, calls)
            assert all(torch.equal(a, b) for mode in (2, 3) for a, b in zip(got[1], got[mode])), (special, lists)
        ix.close()


def test_noalloc_walk(debug_knobs):
    """The entry point that allocates nothing: its scores ahead lie in the static array; captured into a graph, every replay gives
    the eager result."""
    w = make_workload("tiny", seed=33, n=3000, nq=40)
    docs, qs = B.DeviceVecs(w.docs), B.DeviceVecs(w.queries)
    ix = B.Index.build(docs, B.build_params(w.degree))
    pw = torch.from_numpy(np.random.default_rng(4).uniform(0.1, 1.0, (qs.n, 3)).astype(np.float32)).to(docs.device)
    for k, beam, width in ((10, 96, 1), (10, 300, 4)):
        debug_knobs("search_walk", 1)
        ref = [t.clone() for t in ix.search_batch(qs, k, beam, pw, search_width=width)]
        debug_knobs("search_walk", 3)
        out = (torch.full((qs.n, k), -7, dtype=torch.int32, device=docs.device), torch.full((qs.n, k), float("nan"), device=docs.device))
        ix.search_batch_noalloc(qs, k, beam, pw, out, search_width=width)
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(ref, out))
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            ix.search_batch_noalloc(qs, k, beam, pw, out, search_width=width)
        for _ in range(3):
            out[0].fill_(-7)
            ix.search_batch(qs, k, beam, pw, search_width=width)
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            assert all(torch.equal(a, b) for a, b in zip(ref, out))
    ix.close()


@pytest.mark.parametrize("queries_that_fit", [1, 20, 40])
def test_a_workspace_smaller_than_the_batch(debug_knobs, queries_that_fit):
    """The walk takes a batch as a whole: where its rows of bounds and scores may not be had for all queries, the batch is searched
    as any other, in slabs of as many queries as the workspace holds."""
    w = make_workload("tiny", seed=3, n=1500, nq=41)
    docs, qs = B.DeviceVecs(w.docs), B.DeviceVecs(w.queries)
    ix = B.Index.build(docs, B.build_params(16, nd_rounds=1, n_entry=16))
    calls = [(10, 96, 1), (10, 300, 4)]
    debug_knobs("search_walk", 1)
    want = _searches(ix, qs, None, calls)
    # 256 queries' rows of at most 128 + 512 columns and what goes with them, one row of bounds a query
    debug_knobs("search_bounds_bytes", 256 * (2 * (128 + 512) + 52) + queries_that_fit * 4 * 1536)
    for mode in (2, 3, 0):
        debug_knobs("search_walk", mode)
        assert all(torch.equal(a, b) for a, b in zip(want, _searches(ix, qs, None, calls))), mode
    ix.close()


def test_counts_of_rows_not_read(debug_knobs):
    """The third counter of a search: scored documents whose dense row was not read.  None where all rows are read ahead; what is
    in the pool has been scored out of its row, whichever documents were scored ahead."""
    n, nq = 6007, 25
    w = make_workload("tiny", seed=11, n=n, nq=nq, dim=64, vocab=5_000)
    rng = np.random.default_rng(6)
    docs, qs = B.DeviceVecs(w.docs), B.DeviceVecs(w.queries)
    ix = B.Index.import_graph(docs, B.build_params(64, n_entry=16), rng.integers(-1, n, (n, 64)).astype(np.int32),
                              rng.permutation(n)[:16].astype(np.int32))
    pw = rng.uniform(0.1, 1.0, (nq, 3)).astype(np.float32)
    for k, beam, width in ((10, 64, 1), (10, 64, 2), (10, 700, 16), (100, 1300, 1)):
        for mode in (1, 2, 3):
            debug_knobs("search_walk", mode)
            ix.search_batch(qs, k, beam, pw, search_width=width)
            c = ix.search_stats(nq)[0]
            assert ((c[:, 2] >= 0) & (c[:, 0] - c[:, 2] >= c[:, 0].clamp(max=beam))).all(), (mode, beam)
            assert (c[:, 2] == 0).all() if mode == 3 else (c[:, 2] > 0).any(), (mode, beam)
    ix.close()


def test_one_query_many_queries_and_the_plans_own_choice(debug_knobs):
    """One query alone; a batch whose rows of scores do not fit the L2, which no wave brings near; and a batch that the cost model
    itself gives to the walk out of the bounds: its third counter is that of the walk set by hand, not that of the other searches."""
    n = 20_000
    w = make_workload("tiny", seed=21, n=n, nq=320, dim=768, vocab=30_522, sp=("fixed", 120), tx=("fixed", 60))
    docs = B.DeviceVecs(w.docs)
    rng = np.random.default_rng(8)
    ix = B.Index.import_graph(docs, B.build_params(64, n_entry=64), rng.integers(0, n, (n, 64)).astype(np.int32), rng.permutation(n)[:64].astype(np.int32))
    qs = B.DeviceVecs(w.queries)
    assert qs.n * n * 4 > 24e6
    for first, calls in ((1, [(1, 16, 1), (10, 128, 1), (10, 512, 4)]), (40, [(10, 512, 1)]), (320, [(10, 128, 1)])):
        part = make_workload("tiny", seed=21 + first, n=64, nq=first, dim=768, vocab=30_522, sp=("fixed", 120), tx=("fixed", 60))
        part = B.DeviceVecs(part.queries) if first < 320 else qs
        got, third = {}, {}
        for mode in (1, 2, 3, 0):
            debug_knobs("search_walk", mode)
            got[mode] = _searches(ix, part, None, calls)
            third[mode] = ix.search_stats(first)[0][:, 2].clone()
        for mode in (2, 3, 0):
            assert all(torch.equal(a, b) for a, b in zip(got[1], got[mode])), (first, mode)
        if first == 40:
            assert torch.equal(third[0], third[2]) and not torch.equal(third[0], third[1])
    ix.close()


def test_queries_that_only_the_second_pass_answers(debug_knobs):
    """Every score of a query that holds a NaN is one: the walk with lists gives up at its first document, so the ids, scores and
    counts of such a query are those of the second pass, beside queries that the first one decides."""
    n, nq = 3000, 12
    w = make_workload("tiny", seed=12, n=n, nq=nq, dim=128)
    w.queries.dense = np.array(w.queries.dense, dtype=np.float32)
    w.queries.dense[::3, 5] = np.nan
    docs, qs = B.DeviceVecs(w.docs), B.DeviceVecs(w.queries)
    ix = B.Index.build(docs, B.build_params(16, nd_rounds=1, n_entry=16))
    calls = [(10, 96, 1), (10, 300, 4)]
    got = {}
    for mode in (1, 2, 3):
        debug_knobs("search_walk", mode)
        got[mode] = _searches(ix, qs, None, calls)
        assert (got[mode][0][::3] >= 0).all() and got[mode][1].view(torch.float32)[::3].isnan().all()
    for mode in (2, 3):
        assert all(torch.equal(a, b) for a, b in zip(got[1], got[mode])), mode
    ix.close()


# the way a batch takes: nothing to read is left out where all documents are scored ahead; the walk out of the bounds and the searches
# that score as they go leave out different numbers.  64 edges fill all of a wave's lists, 16 a quarter of them
@pytest.mark.parametrize("degree,beam,way", [(64, 512, 3), (16, 512, 2), (16, 2500, 1)])
def test_walks_whose_lists_would_not_hold_what_enters_them(debug_knobs, degree, beam, way):
    """A query whose lists overflow is searched twice: the cost model takes a way whose lists hold what is to be expected, or none."""
    n = 12_000
    w = make_workload("tiny", seed=degree + beam, n=n, nq=3, dim=128)
    rng = np.random.default_rng(9)
    docs, qs = B.DeviceVecs(w.docs), B.DeviceVecs(w.queries)
    ix = B.Index.import_graph(docs, B.build_params(degree, n_entry=64), rng.integers(0, n, (n, degree)).astype(np.int32), rng.permutation(n)[:64].astype(np.int32))
    got, third = {}, {}
    for mode in (1, 2, 3, 0):
        debug_knobs("search_walk", mode)
        got[mode] = _searches(ix, qs, None, [(10, beam, 1)])
        third[mode] = ix.search_stats(3)[0][:, 2].tolist()
    assert all(torch.equal(a, b) for mode in (2, 3, 0) for a, b in zip(got[1], got[mode]))
    assert third[1] != third[2] and max(third[3]) == 0 < min(third[1] + third[2])
    assert third[0] == third[way], third
    ix.close()


def test_the_plans_choice_with_several_parents(debug_knobs):
    """16 queries with four parents, where the cost model has the walk out of the bounds just a fifth faster than the search."""
    n, nq, rng = 20_000, 16, np.random.default_rng(4)
    w = make_workload("tiny", seed=4, n=n, nq=nq, dim=768, vocab=30_522, sp=("fixed", 100), tx=("fixed", 60))
    docs, qs = B.DeviceVecs(w.docs), B.DeviceVecs(w.queries)
    ix = B.Index.import_graph(docs, B.build_params(64, n_entry=16), rng.integers(0, n, (n, 64)).astype(np.int32), rng.permutation(n)[:16].astype(np.int32))
    got, third = {}, {}
    for mode in (1, 2, 3, 0):
        debug_knobs("search_walk", mode)
        got[mode] = _searches(ix, qs, None, [(10, 128, 4)])
        third[mode] = ix.search_stats(nq)[0][:, 2].clone()
    assert all(torch.equal(a, b) for mode in (2, 3, 0) for a, b in zip(got[1], got[mode]))
    assert torch.equal(third[0], third[2]) and not torch.equal(third[0], third[1]) and (third[2] > 0).any()
    ix.close()
