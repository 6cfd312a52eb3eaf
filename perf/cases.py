"""What this library is asked to do, as cases that can be timed: one call of a public entry point each.

A corpus holds what the generators of ``paper_2511_00855_amd.synth`` draw -- unit Gaussian dense rows (f32, or stored
bf16), Zipf(1.1) term lists of a learned-sparse encoder, texts of log-normal length -- drawn here on the GPU, because the
inputs of a case are made many times.  The sizes are those of the named workloads (``tiny``; 768 columns of f32 on
100,000 documents; 1,024 columns of bf16) and of the sweeps that ``bench.py`` runs over them, with odd ones beside them.
"""
from __future__ import annotations

import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_2511_00855_amd import binding as B

DEVICE = "cuda:0"

# The shapes of the named workloads: width and storage of the dense rows, vocabulary, entries of a document's
# learned-sparse list, tokens of its text; and of a query's.
TINY = dict(dim=128, bf16=False, vocab=10_000, sp=32, tokens=40, q_sp=8, q_tokens=6, weights="0.5,0.3,0.2")
F32 = dict(dim=768, bf16=False, vocab=30_522, sp=120, tokens=60, q_sp=20, q_tokens=8, weights="0.5,0.3,0.2")
BF16 = dict(dim=1024, bf16=True, vocab=250_002, sp=100, tokens=60, q_sp=20, q_tokens=8, weights="0.4,0.4,0.2")
# degree, refinement rounds and entry points of the index that a case builds or searches
INDEX = dict(degree=64, rounds=3, n_entry=64)
# a plain search's options: deleted = share of mark-deleted documents; mixed = every query has weights of its own
SEARCH = dict(kind="search", k=10, deleted=0.0, mixed=False, noalloc=False)


def listed():
    return [
        # one user's query against a corpus of 100,000 documents: nothing but latency
        dict(SEARCH, name="search one query", **F32, **INDEX, n=100_000, nq=1, beam=128, width=1),
        # a serving process's micro-batch: a few dozen requests, every one with fusion weights of its own
        dict(SEARCH | {"mixed": True}, name="search micro-batch", **BF16, **INDEX, n=120_011, nq=37, beam=512, width=1),
        # the nominal batch of the benchmark: 10,000 queries, a pool of 128
        dict(SEARCH, name="search batch", **F32, **INDEX, n=100_000, nq=10_000, beam=128, width=1),
        # the batch at the benchmark's setting for recall 0.95 on 100,000 documents
        dict(SEARCH, name="search at recall 0.95", **F32, **INDEX, n=100_000, nq=4_000, beam=2112, width=16),
        # the deep pool that recall 0.95 takes on large bf16 corpora (about n / 64 entries): one query fills a compute unit
        dict(SEARCH, name="search deep pool", **BF16, **INDEX, n=500_000, nq=2_000, beam=8_192, width=16),
        # keyword-constrained search on an index that has seen deletions
        dict(kind="keywords", name="search with keywords", **F32, **INDEX, n=100_000, nq=2_500, beam=512, width=1, k=10,
             deleted=0.02, kw_all=False),
        # entity-aware search of a small, high-value shard
        dict(kind="entities", name="search with entities", **F32, **INDEX, n=20_000, nq=4_000, beam=128, k=10),
        # construction: a small collection, where launches and allocations count
        dict(kind="build", name="build small", **TINY, degree=32, rounds=3, n_entry=64, n=2_000),
        # construction of the two benchmark shapes (the second over an odd number of documents)
        dict(kind="build", name="build f32", **F32, **INDEX, n=100_000),
        dict(kind="build", name="build bf16", **BF16, **INDEX, n=200_003),
        # new documents go into an index (5 % of it)
        dict(kind="insert", name="insert 5 %", **BF16, **INDEX, n=80_000, new=4_000),
        # exact top-k by enumeration, the ground truth of a recall measurement
        dict(kind="exact", name="exact top-k", **F32, n=100_000, nq=1_000, k=10),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _reached(n, beam, degree):
    """Documents a search scores, about: as many as beam expansions of `degree` random neighbours reach."""
    return n * (1.0 - math.exp(-beam * degree / n))


def draw(rng):
    kind = rng.choice(["search", "search", "search", "keywords", "entities", "build", "build", "insert", "exact"])
    shape = dict(rng.choice([TINY, F32, BF16]))
    if rng.random() < 0.5:   # other widths; a row is a multiple of 4 (f32) or 8 (bf16) columns
        shape["dim"] = rng.choice([256, 384, 520, 1000, 1536] if shape["bf16"] else [96, 260, 384, 500, 1024])
    shape["sp"] = rng.randint(20, 130)
    shape["tokens"] = rng.randint(15, 80)
    shape["vocab"] = _log(rng, 5_000, 250_002)
    index = dict(degree=rng.choice([16, 32, 64]), rounds=rng.choice([2, 3]), n_entry=rng.choice([16, 64]))
    if kind == "build":
        return dict(kind=kind, **shape, **index, n=_log(rng, 500, 150_000))
    if kind == "insert":
        n = _log(rng, 2_000, 80_000)
        return dict(kind=kind, **shape, **index, n=n, new=max(1, int(n * rng.uniform(0.005, 0.1))))
    if kind == "exact":
        n = _log(rng, 1_000, 150_000)
        return dict(kind=kind, **shape, n=n, nq=_log(rng, 1, max(2, min(4_000, 80_000_000 // n))), k=rng.choice([1, 10, 100]))
    beam = _log(rng, 16, 512 if kind == "entities" else 4_096 if kind == "keywords" else 15_000)
    width = 1 if kind == "entities" else rng.choice([1, 1, 2, 4]) if beam < 1024 else rng.choice([1, 4, 16])
    if kind == "keywords":
        width = min(width, 4)
    n = _log(rng, 1_000, 20_000 if kind == "entities" else 150_000)
    most = 60_000_000 if kind in ("keywords", "entities") else 150_000_000   # similarities of the pass
    nq = max(1, min(_log(rng, 1, 10_000), int(most / _reached(n, beam, index["degree"]))))
    case = dict(kind=kind, **shape, **index, n=n, nq=nq, beam=beam, width=width, k=min(beam, rng.choice([1, 10, 10, 50])))
    if kind == "entities":
        del case["width"]
    if kind == "keywords":
        case.update(deleted=rng.choice([0.0, 0.05]), kw_all=rng.random() < 0.3)
    if kind == "search":
        case.update(deleted=rng.choice([0.0, 0.0, 0.05]), mixed=rng.random() < 0.5, noalloc=rng.random() < 0.25)
    return case


# ---------------------------------------------------------------- inputs

def _csr_rows(keep):
    """Row offsets of a CSR whose row r holds the marked places of keep[r]."""
    ip = torch.zeros(len(keep) + 1, dtype=torch.int64, device=DEVICE)
    ip[1:] = torch.cumsum(keep.sum(dim=1), 0)
    return ip


def _zipf(g, rows, width, vocab, perm):
    """rows x width term ids: ranks by Zipf(1.1), ids by a fixed permutation of the ranks."""
    cdf = torch.cumsum(torch.arange(1, vocab + 1, dtype=torch.float64, device=DEVICE) ** -1.1, 0)
    r = torch.searchsorted(cdf / cdf[-1], torch.rand(rows, width, dtype=torch.float64, generator=g, device=DEVICE))
    return perm[r.clamp_(max=vocab - 1)]


def _distinct_lists(g, counts, vocab, perm):
    """CSR of counts[r] distinct terms a row, ascending: the first ones of a long enough run of draws."""
    need = counts.clamp(max=vocab // 4)
    width = 4 * int(need.max()) + 16
    ips, idx = [torch.zeros(1, dtype=torch.int64, device=DEVICE)], []
    for r0 in range(0, len(need), 1 << 15):
        n = need[r0:r0 + (1 << 15)]
        v, at = torch.sort(_zipf(g, len(n), width, vocab, perm), dim=1, stable=True)
        first = torch.ones_like(v, dtype=torch.bool)
        first[:, 1:] = v[:, 1:] != v[:, :-1]
        drawn = torch.zeros_like(first).scatter_(1, at, first)          # a term's first draw, in the order of the draws
        keep = first & (torch.cumsum(drawn, 1) <= n[:, None]).gather(1, at)
        ips.append(ips[-1][-1] + _csr_rows(keep)[1:])
        idx.append(v[keep].to(torch.int32))
    return torch.cat(ips), torch.cat(idx)


def _texts(g, lengths, vocab, perm):
    """CSR of the bags of lengths[r] tokens a row: terms ascending, and how often each occurs."""
    width = int(lengths.max())
    ips, idx, tf = [torch.zeros(1, dtype=torch.int64, device=DEVICE)], [], []
    for r0 in range(0, len(lengths), 1 << 15):
        n = lengths[r0:r0 + (1 << 15)]
        toks = _zipf(g, len(n), width, vocab, perm)
        v = torch.sort(torch.where(torch.arange(width, device=DEVICE)[None] < n[:, None], toks, vocab), dim=1)[0]
        first = v < vocab
        first[:, 1:] &= v[:, 1:] != v[:, :-1]
        row, col = torch.nonzero(first, as_tuple=True)
        until = n[row]                                                  # where a term's run ends: at the next term or the row's end
        until[:-1] = torch.where(row[1:] == row[:-1], col[1:], until[:-1])
        ips.append(ips[-1][-1] + _csr_rows(first)[1:])
        idx.append(v[first].to(torch.int32))
        tf.append((until - col).to(torch.float32))
    return torch.cat(ips), torch.cat(idx), torch.cat(tf)


def _vectors(g, n, case, sp, tokens, spread, perms, bf16):
    """A vector set: n dense rows, lists of Poisson(sp) terms, texts of about `tokens` tokens (log-normal, or Poisson if
    not `spread`)."""
    dense = torch.randn(n, case["dim"], generator=g, device=DEVICE)
    dense /= dense.norm(dim=1, keepdim=True)
    counts = torch.poisson(torch.full((n,), float(sp), device=DEVICE), generator=g).to(torch.int64).clamp_(min=1)
    if spread:
        z = torch.randn(n, generator=g, device=DEVICE)
        lengths = torch.exp(math.log(tokens) - 0.125 + 0.5 * z).round().to(torch.int64).clamp_(5, 512)
    else:
        lengths = torch.poisson(torch.full((n,), float(tokens), device=DEVICE), generator=g).to(torch.int64).clamp_(min=1)
    v = SimpleNamespace(n=n, dim=case["dim"], dense=dense, sp_vocab=case["vocab"], tx_vocab=case["vocab"])
    v.sp_indptr, v.sp_idx = _distinct_lists(g, counts, case["vocab"], perms[0])
    v.sp_val = torch.randn(len(v.sp_idx), generator=g, device=DEVICE).abs_().clamp_(min=1e-3)
    v.tx_indptr, v.tx_idx, v.tx_val = _texts(g, lengths, case["vocab"], perms[1])
    if bf16:   # bit patterns of the rounded rows, as the binding takes them
        v.dense_bf16 = dense.to(torch.bfloat16).view(torch.int16).cpu().numpy().view(np.uint16)
    return v


def _first_rows(v, n):
    """The first n rows of a vector set."""
    w = SimpleNamespace(**vars(v))
    w.n, w.dense, w.sp_indptr, w.tx_indptr = n, v.dense[:n], v.sp_indptr[:n + 1], v.tx_indptr[:n + 1]
    w.sp_idx, w.sp_val = v.sp_idx[:int(w.sp_indptr[-1])], v.sp_val[:int(w.sp_indptr[-1])]
    w.tx_idx, w.tx_val = v.tx_idx[:int(w.tx_indptr[-1])], v.tx_val[:int(w.tx_indptr[-1])]
    if hasattr(v, "dense_bf16"):
        w.dense_bf16 = v.dense_bf16[:n]
    return w


def _own_tokens(g, queries, stride=2):
    """One or two of each query's own tokens as required terms, -1 in unused slots."""
    beg, size = queries.tx_indptr[:-1], queries.tx_indptr[1:] - queries.tx_indptr[:-1]
    place = (torch.rand(queries.n, stride, generator=g, device=DEVICE) * size[:, None]).to(torch.int64)
    kw = queries.tx_idx[beg[:, None] + place]
    drop = (torch.rand(queries.n, generator=g, device=DEVICE) < 0.5) | (place[:, 0] == place[:, 1])
    kw[:, 1] = torch.where(drop, torch.full_like(kw[:, 1], -1), kw[:, 1])
    return kw.contiguous()


def _entity_graph(g, n, nq):
    """One to three of n / 8 entities a document, about four relations an entity, one or two entities of one document a query."""
    n_ent = max(8, n // 8)
    ents = torch.sort(torch.randint(n_ent, (n, 3), generator=g, device=DEVICE), dim=1)[0]
    keep = torch.arange(3, device=DEVICE)[None] < torch.randint(1, 4, (n, 1), generator=g, device=DEVICE)
    keep[:, 1:] &= ents[:, 1:] != ents[:, :-1]
    pairs = torch.randint(n_ent, (2 * n_ent, 2), generator=g, device=DEVICE)
    pairs = pairs[pairs[:, 0] != pairs[:, 1]]
    pairs = torch.unique(torch.cat([pairs, pairs.flip(1)]), dim=0)
    kg_ip = torch.zeros(n_ent + 1, dtype=torch.int64, device=DEVICE)
    kg_ip[1:] = torch.cumsum(torch.bincount(pairs[:, 0], minlength=n_ent), 0)
    of = ents[torch.randint(n, (nq,), generator=g, device=DEVICE)]
    q_ent = torch.full((nq, 4), -1, dtype=torch.int32, device=DEVICE)
    q_ent[:, 0] = of[:, 0]
    q_ent[:, 1] = torch.where((torch.rand(nq, generator=g, device=DEVICE) < 0.5) & (of[:, 1] != of[:, 0]), of[:, 1], -1)
    kg = SimpleNamespace(n_ent=n_ent, doc_ent_indptr=_csr_rows(keep), doc_ent=ents[keep].to(torch.int32), kg_indptr=kg_ip,
                         kg_idx=pairs[:, 1].to(torch.int32).contiguous())
    return kg, q_ent


def prepare(case, seed):
    g = torch.Generator(DEVICE)
    g.manual_seed(seed)
    perms = [torch.randperm(case["vocab"], generator=g, device=DEVICE) for _ in range(2)]
    corpus = _vectors(g, case["n"], case, case["sp"], case["tokens"], True, perms, case["bf16"])
    docs = B.DeviceVecs(corpus, DEVICE, bf16=case["bf16"])
    s = dict(case=case, docs=docs)
    if case["kind"] != "exact":
        # lists of twice the degree while the graph is made, as build_params chooses by itself
        s["params"] = B.build_params(case["degree"], nd_rounds=case["rounds"], n_entry=case["n_entry"])
    if case["kind"] == "build":
        return s
    if case["kind"] == "insert":
        old = B.DeviceVecs(_first_rows(corpus, case["n"] - case["new"]), DEVICE, bf16=case["bf16"])
        s["old"] = B.Index.build(old, s["params"])
        return s
    nq = case["nq"]
    s["queries"] = B.DeviceVecs(_vectors(g, nq, case, case["q_sp"], case["q_tokens"], False, perms, False), DEVICE)
    s["weights"] = torch.tensor([[float(x) for x in case["weights"].split(",")]], device=DEVICE).repeat(nq, 1)
    if case.get("mixed"):
        u = torch.rand(nq, 3, generator=g, device=DEVICE) + 0.05
        s["weights"] = u / u.sum(dim=1, keepdim=True)
    if case["kind"] == "exact":
        s["index"] = B.Index.ingest(docs, B.build_params(32))
        return s
    s["index"] = ix = B.Index.build(docs, s["params"])
    if case.get("deleted"):
        ix.mark_deleted(torch.randperm(case["n"], generator=g, device=DEVICE)[:int(case["n"] * case["deleted"])].to(torch.int32))
    if case["kind"] == "keywords":
        s["terms"] = _own_tokens(g, s["queries"])
    if case["kind"] == "entities":
        kg, s["entities"] = _entity_graph(g, case["n"], nq)
        ix.set_knowledge_graph(kg, le_cap=16)
    if case.get("noalloc"):   # such a caller brings its own result arrays
        s["out"] = (torch.empty((nq, case["k"]), dtype=torch.int32, device=DEVICE), torch.empty((nq, case["k"]), device=DEVICE))
    return s


# ---------------------------------------------------------------- the calls

def run(state):
    case, kind = state["case"], state["case"]["kind"]
    if kind == "build":
        ix = B.Index.build(state["docs"], state["params"])
        out = ix.export_graph()        # semantic edges, keyword edges and their counts, entry points
        ix.close()
        return out
    if kind == "insert":
        ix = state["old"].insert(state["docs"])
        out = ix.export_graph()
        ix.close()
        return out
    ix, q, w, k = state["index"], state["queries"], state["weights"], case["k"]
    if kind == "exact":
        return ix.bruteforce_topk(q, k, w)
    if kind == "keywords":
        return ix.search_batch_keywords(q, k, case["beam"], state["terms"], w, kw_all=case["kw_all"], search_width=case["width"])
    if kind == "entities":
        return ix.search_batch_entities(q, k, case["beam"], state["entities"], 0.5, 2, w)
    if case["noalloc"]:
        return ix.search_batch_noalloc(q, k, case["beam"], w, state["out"], search_width=case["width"])
    return ix.search_batch(q, k, case["beam"], w, search_width=case["width"])


# ---------------------------------------------------------------- what a pass cannot do without

def _list_bytes(case):
    """Bytes of a document's two lists (a text's distinct terms are some three quarters of its tokens)."""
    return 8 * (case["sp"] + 0.75 * case["tokens"])


def _corpus_bytes(case):
    return case["n"] * (case["dim"] * (2 if case["bf16"] else 4) + _list_bytes(case))


def work(case):
    """Bytes: every input read once, every output written once.  FLOPs: two per multiply-add of the inner products."""
    n, dim, lists = case["n"], case["dim"], _list_bytes(case) / 8
    if case["kind"] in ("build", "insert"):
        degree, new = case["degree"], case.get("new", case["n"])
        knn = 2 * degree                               # entries of a list while the graph is made
        pairs = new * (new - 1) / 2                    # exact dense lists of the new documents
        explored = new * case["rounds"] * (knn + min(32, knn) ** 2)   # similarities of the refinement rounds, at most
        around = new * knn * (knn - 1) / 2             # similarities inside the neighbourhoods
        # the lists of every explored pair, and the dense rows of at least those that enter a list
        dense = pairs + new * case["rounds"] * knn + around
        return {"bytes": _corpus_bytes(case) + n * 4 * (degree + degree // 2 + 1), "flops": 2 * dim * dense + 2 * lists * (min(explored, pairs) + around)}
    nq = case["nq"]
    query = 4 * dim + 8 * (case["q_sp"] + case["q_tokens"]) + 12 + 8 * case["k"]
    if case["kind"] == "exact":
        return {"bytes": _corpus_bytes(case) + nq * query, "flops": nq * n * (2 * dim + 2 * (case["q_sp"] + case["q_tokens"]))}
    # A search reads the lists of the documents that it reaches and its pool's edges; a dense row only where the lists
    # leave the answer open, of which the pool's own entries are the least.
    reached = _reached(n, case["beam"], case["degree"])
    rows = min(n, nq * reached)
    kept = min(n, nq * min(case["beam"], reached))
    return {"bytes": rows * (_list_bytes(case) + 16) + kept * (dim * (2 if case["bf16"] else 4) + 4 * case["degree"]) + nq * query,
            "flops": nq * (reached * 2 * (case["q_sp"] + case["q_tokens"]) + min(case["beam"], reached) * 2 * dim)}


def tolerance(case):
    """Measured by running every case with its sums in 64 bits and its matrix products in the reverse order of k.
    Scores then move by 5e-8 (largest 2.4e-7); near-ties among them change 0.0037 of a f32 graph's ids and 0.0006 of a
    bf16 graph's, and a search of the graphs so changed ends elsewhere for 0.003 of its ids (scores by 0.0016, largest
    0.21).  About four times that, as far as a share of ids may go."""
    graph = 0.0025 if case["bf16"] else 0.01
    if case["kind"] in ("build", "insert"):
        return {"rel": 1e-6, "differ": graph}
    if case["kind"] == "exact":
        return {"rel": 1e-6, "max": 4e-6, "differ": 0.001}
    return {"rel": 0.006, "max": 0.85, "differ": 0.01}
