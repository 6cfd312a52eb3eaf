"""The refinement rounds of a construction leave out candidates scored in earlier rounds and dense rows whose bound
cannot reach a list; a round called on its own scores everything.  Both must give the same lists, bit for bit."""
import numpy as np
import pytest
import torch

from paper_2511_00855_amd import binding as B
from paper_2511_00855_amd.synth import make_workload

pytestmark = pytest.mark.gpu

CASES = {
    # name: (workload, R, K, S, P, build weights, what is done to the dense rows)
    "ordinary": (dict(n=1500, dim=96), 32, 64, 32, 6, (1.0, 1.0, 1.0), None),
    "only the dense part": (dict(n=900, dim=100), 16, 40, 32, 8, (1.0, 0.0, 0.0), "clusters"),
    "duplicate rows": (dict(n=700, dim=64, sp=("fixed", 3), tx=("fixed", 6)), 16, 48, 24, 32, (1.0, 0.2, 0.1), "duplicates"),
    "negative dense weight": (dict(n=800, dim=128), 16, 48, 32, 8, (-1.0, 0.3, 0.2), "norms"),
    "no dense weight": (dict(n=600, dim=64), 16, 32, 20, 4, (0.0, 1.0, 1.0), None),
    "every document in every list": (dict(n=40, dim=32), 16, 64, 32, 11, (1.0, 1.0, 1.0), "norms"),
    "lists too long for the tables": (dict(n=260, dim=512, bf16=True, sp=("fixed", 300), tx=("fixed", 200)), 12, 24, 5, 3, (1.0, 1.0, 1.0), None),
    "bf16": (dict(n=1200, dim=1032, bf16=True, sp=("poisson", 100), tx=("lognormal", 60)), 64, 128, 32, 11, (1.0, 1.0, 1.0), None),
    "path lists longer than the lists": (dict(n=300, dim=260), 4, 4, 4, 32, (1.0, 1.0, 1.0), None),
}


@pytest.mark.parametrize("name", list(CASES))
def test_rounds_of_a_construction_equal_rounds_called_one_by_one(name):
    kw, R, K, S, P, wv, dense = CASES[name]
    w = make_workload("tiny", seed=77, nq=2, **kw)
    d, rng = w.docs, np.random.default_rng(3)
    if dense == "clusters":
        d.dense[:] = d.dense[rng.integers(0, 30, d.n)] + 0.02 * d.dense
    elif dense == "duplicates":
        d.dense[:] = d.dense[rng.integers(0, 12, d.n)]
    elif dense == "norms":
        d.dense[:] = d.dense * rng.uniform(0.05, 4.0, (d.n, 1)).astype(np.float32)
    docs = B.DeviceVecs(d, bf16=bool(kw.get("bf16")))
    for rounds in (1, 2, 4):
        print(name, rounds, flush=True)
        full = B.Index.build(docs, B.build_params(R, knn_k=K, nd_rounds=rounds, nd_sample=S, sp_len=P, n_entry=4, build_w=wv))
        se, srt, spi, sps = full.export_build_state()
        ix = B.Index.ingest(docs, B.build_params(R, knn_k=K, nd_rounds=rounds, nd_sample=S, sp_len=P, n_entry=4, build_w=wv))
        ids, sc = ix.stage_seed_knn(K)
        i2 = torch.full((3, d.n, P), -1, dtype=torch.int32, device=docs.device)
        s2 = torch.full((3, d.n, P), -np.inf, dtype=torch.float32, device=docs.device)
        for _ in range(rounds):
            ids, sc, i2, s2 = ix.stage_refine(K, S, P, ids, i2, s2)
        g = ix.stage_prune(K, R, ids, sc, want_pm=False)
        assert torch.equal(spi, i2) and torch.equal(sps, s2)
        assert torch.equal(srt, g["sorted_ids"]) and torch.equal(se, g["se"])
        # a round of a construction evaluates no more similarities than the same round on its own
        assert full.build_counters()["refine_similarities"] <= ix.build_counters()["refine_similarities"]
        full.close(); ix.close()



def _twice(d):   # every document, and once more with a slightly other dense row
    half = d.n // 2
    d.dense[half:] = d.dense[:half] + np.float32(0.01) * d.dense[half:]
    for p in ("sp", "tx"):
        ip, idx, val = getattr(d, p + "_indptr"), getattr(d, p + "_idx"), getattr(d, p + "_val")
        end = ip[half]
        setattr(d, p + "_indptr", np.concatenate([ip[:half + 1], ip[1:half + 1] + end]))
        setattr(d, p + "_idx", np.concatenate([idx[:end]] * 2))
        setattr(d, p + "_val", np.concatenate([val[:end]] * 2))


# Scored in full of what the first round meets: 0.08 to 0.15.  Bins over the first four octaves alone: 0.99, 0.23, 0.33, 0.15 (these scores lie within
# four octaves) and 1.0.
@pytest.mark.parametrize("name,wv,twice,packed", [("near duplicates", (1.0, 1.0, 1.0), True, True), ("near duplicates, sparse parts", (0.2, 1.0, 0.2), True, True),
                                                  ("negative sparse weight", (0.5, -0.3, 0.2), False, False), ("all weights negative", (-0.5, -0.3, -0.2), False, False),
                                                  ("near duplicates, negative sparse weight", (0.5, -0.3, 0.2), True, False)])
def test_first_scored_far_below_the_best_bound(name, wv, twice, packed):
    """Where the K best lie more than four octaves below the best bound, or below zero, only about K candidates are scored first all the
    same; the lists are those of rounds that score everything."""
    w = make_workload("tiny", seed=5, n=3000, nq=2, dim=96, vocab=60_000, sp=("poisson", 100), tx=("lognormal", 60))
    if twice:
        _twice(w.docs)
    docs = B.DeviceVecs(w.docs)
    K, S, P = 48, 32, 11
    bp = B.build_params(16, knn_k=K, nd_rounds=1, nd_sample=S, sp_len=P, n_entry=4, build_w=wv)
    full = B.Index.build(docs, bp)
    assert full.packed_lists() == packed
    _, srt, spi, sps = full.export_build_state()
    ix = B.Index.ingest(docs, bp)
    ids, sc = ix.stage_seed_knn(K)
    i2 = torch.full((3, docs.n, P), -1, dtype=torch.int32, device=docs.device)
    s2 = torch.full((3, docs.n, P), -np.inf, dtype=torch.float32, device=docs.device)
    ids, sc, i2, s2 = ix.stage_refine(K, S, P, ids, i2, s2)
    g = ix.stage_prune(K, 16, ids, sc, want_pm=False)
    assert torch.equal(spi, i2) and torch.equal(sps.view(torch.int32), s2.view(torch.int32))
    assert torch.equal(srt, g["sorted_ids"])
    met, scored = full.build_counters()["refine_similarities"], full.refine_scored()
    print(name, met, scored, scored / met, flush=True)
    assert ix.refine_scored() == ix.build_counters()["refine_similarities"]   # a round on its own scores all
    assert scored < 0.2 * met
    full.close(); ix.close()


def test_dense_scores_beyond_the_range_keep_their_place():
    """Rows of +-3e19 in one column: products of two are +-inf in f32.  A list with room takes a -inf like any other score, in a
    round of a construction and in one on its own, as the oracle does."""
    import oracle as O
    from paper_2511_00855_amd.synth import VecSet
    n, K, S, P, rng = 8, 8, 8, 6, np.random.default_rng(5)
    dense = np.zeros((n, 4), np.float32)
    dense[:, 0] = np.float32(3e19) * np.array([1, -1, 1, 1, -1, -1, 1, -1], np.float32)
    ip = np.arange(0, 3 * n + 1, 3, dtype=np.int64)
    terms = lambda: np.concatenate([np.sort(rng.permutation(10)[:3]) for _ in range(n)]).astype(np.int32)
    d = VecSet(n, 4, dense, ip, terms(), rng.uniform(0.5, 2.0, 3 * n).astype(np.float32), ip, terms(), np.ones(3 * n, np.float32), 10, 10)
    docs, bp = B.DeviceVecs(d), B.build_params(8, knn_k=K, nd_rounds=1, nd_sample=S, sp_len=P, n_entry=4)
    full = B.Index.build(docs, bp)
    _, _, spi, sps = [t.cpu().numpy() for t in full.export_build_state()]
    ix = B.Index.ingest(docs, bp)
    ids, _ = ix.stage_seed_knn(K)
    i2, s2 = O.empty_sp(n, P)
    _, _, gi, gs = [t.cpu().numpy() for t in ix.stage_refine(K, S, P, ids, i2, s2)]
    D = O.encode_docs(d)
    _, _, oi, os_ = O.refine_round(D, [1.0, 1.0, 1.0], K, S, P, ids.cpu().numpy(), i2, s2)
    assert np.isneginf(os_[0]).any() and (oi[0] >= 0).all()
    assert np.array_equal(oi[0], gi[0]) and np.array_equal(os_[0], gs[0])
    assert np.array_equal(spi, gi) and np.array_equal(sps, gs)
    full.close(); ix.close()
