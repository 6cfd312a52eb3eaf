"""The table of upper bounds: never below a score that the scoring kernels give, no further above it than its rounding
allows, and searches that use it return the same ids, scores and counts of scored documents, bit for bit, as searches
that score every neighbour."""
import numpy as np
import pytest
import torch

from paper_2511_00855_amd import binding as B
from paper_2511_00855_amd.synth import make_keywords, make_workload

pytestmark = pytest.mark.gpu


def _workload(base, **kw):
    w = make_workload(base, seed=11, **kw)
    bf16 = getattr(w.docs, "dense_bf16", None) is not None
    return w, B.DeviceVecs(w.docs, bf16=bf16), B.DeviceVecs(w.queries)


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
        wd, ws, wf = [torch.from_numpy(np.abs(weights[:, i])).to(sc.device)[:, None] for i in range(3)]
        assert (up >= sc[:, :, 3]).all()
        # two roundings to bf16 (2^-9 each) of norm-bounded parts, once in the product and once in the slack, and 1e-3 for all sums
        q, d = w.queries, w.docs
        qn = torch.from_numpy(np.linalg.norm(q.dense, axis=1)).to(sc.device)[:, None]
        dn = torch.from_numpy(np.linalg.norm(d.dense, axis=1)).to(sc.device)[None, :]
        rows = lambda ip, v: torch.from_numpy(np.array([np.linalg.norm(v[a:b]) for a, b in zip(ip[:-1], ip[1:])])).to(sc.device)
        txw = ix.export_ingest()[0].cpu().numpy()
        parts = wd * qn * dn + ws * rows(q.sp_indptr, q.sp_val)[:, None] * rows(d.sp_indptr, d.sp_val)[None, :] \
            + wf * rows(q.tx_indptr, q.tx_val)[:, None] * rows(d.tx_indptr, txw)[None, :]
        assert (up - sc[:, :, 3] <= (4 * 2.0 ** -9 + 1e-3) * parts + 1e-12).all()
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
