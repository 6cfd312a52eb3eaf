"""The stages of a construction share their scratch while it is small (64 MiB: the exact seed lists' scores and the neighbourhood similarities
of 4,096 documents with lists of 64), an insertion's take the memory of its search: same graph as from stages that each make their own."""
import numpy as np
import pytest
import torch

from paper_2511_00855_amd import binding as B
from paper_2511_00855_amd.synth import make_workload, subset_vecset

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,rounds", [(300, 0), (4000, 1), (4200, 2)])
def test_graph_of_shared_scratch(n, rounds):
    w = make_workload("tiny", seed=5, n=n, nq=2, dim=32)
    docs, R, K, S, P = B.DeviceVecs(w.docs), 32, 64, 8, 6
    bp = B.build_params(R, knn_k=K, nd_rounds=rounds, nd_sample=S, sp_len=P, n_entry=64)
    full = B.Index.build(docs, bp)
    ix = B.Index.ingest(docs, bp)
    ids, sc = ix.stage_seed_knn(K)
    spi = torch.full((3, n, P), -1, dtype=torch.int32, device=docs.device)
    sps = torch.full((3, n, P), -np.inf, dtype=torch.float32, device=docs.device)
    for _ in range(rounds):
        ids, sc, spi, sps = ix.stage_refine(K, S, P, ids, spi, sps)
    if rounds == 0:   # a construction without rounds scores the seed lists by all three parts
        sc = ix.hybrid_scores_docs(np.arange(n, dtype=np.int32), ids, bp_weights(bp))[:, :, 3].contiguous()
    g = ix.stage_prune(K, R, ids, sc, want_pm=False)
    sem, kw, kc, ent = full.export_graph()
    assert torch.equal(full.export_build_state()[2], spi) and torch.equal(full.export_build_state()[1], g["sorted_ids"])
    assert torch.equal(sem, ix.stage_assemble(R, K, P, g["se"], g["sorted_ids"], spi))
    assert torch.equal(kw, g["ke"]) and torch.equal(kc, g["ke_count"]) and torch.equal(ent, ix.stage_entry_points(64))
    full.close(); ix.close()


def bp_weights(bp):
    return [bp.build_w[0], bp.build_w[1], bp.build_w[2]]


# with bounds the steps behind the search take its table's memory, without them their own
@pytest.mark.parametrize("n,new", [(3000, 600), (3000, 1), (900, 450)])
def test_insertion_in_borrowed_scratch(debug_knobs, n, new):
    w = make_workload("tiny", seed=6, n=n, nq=2, dim=32, bf16=True)
    bp = B.build_params(16, knn_k=32, nd_rounds=2, nd_sample=8, n_entry=16)
    old = B.Index.build(B.DeviceVecs(subset_vecset(w.docs, np.arange(n - new)), bf16=True), bp)
    docs = B.DeviceVecs(w.docs, bf16=True)
    got = []
    for mode in (2, 1):
        debug_knobs("search_bounds", mode)
        ix = old.insert(docs)
        got.append([t.clone() for t in (*ix.export_graph(), *ix.export_build_state())])
        ix.close()
    assert all(torch.equal(a, b) for a, b in zip(*got))
    old.close()
