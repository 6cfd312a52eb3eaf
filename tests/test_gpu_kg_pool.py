"""The pool of the search with entities takes an iteration's candidates all at once: pools at the edges of a wave, more than a wave of
candidates at a time (entry points, rows of 128 edges, logical edges), ties.  Replayed by the oracle on the kernel's own scores, bit for bit."""
import numpy as np
import pytest

import oracle as O
from paper_2511_00855_amd import binding as B
from paper_2511_00855_amd.synth import make_entity_graph, make_workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("degree,n_entry,bf16,dim", [(128, 256, False, 128), (16, 4, True, 1544)])
def test_pool_against_the_oracle(degree, n_entry, bf16, dim):
    n, nq = 1400, 12
    w = make_workload("tiny", seed=8, n=n, nq=nq, bf16=bf16, dim=dim)
    d = w.docs
    d.sp_val[:] = np.round(d.sp_val * 2) / 2 + 0.5   # ties among the scores
    docs, qs = B.DeviceVecs(d, bf16=bf16), B.DeviceVecs(w.queries)
    ix = B.Index.build(docs, B.build_params(degree, knn_k=degree, nd_rounds=1, n_entry=n_entry))
    kgs = make_entity_graph(n, nq, seed=3, n_ent=120)
    kgs.q_ent[::3] = -1
    ix.set_knowledge_graph(kgs, le_cap=32)
    le, cnt, en_ip, en = [t.cpu().numpy() for t in ix.export_logical_edges()]
    D, Q = O.encode_docs(d), O.VS(w.queries)
    sem, _, _, ent = [t.cpu().numpy() for t in ix.export_graph()]
    wq = np.random.default_rng(2).uniform(0.1, 1.0, (nq, 3)).astype(np.float32)
    wq[1::4] = [0.0, 1.0, 0.0]
    table = ix.hybrid_scores(qs, np.tile(np.arange(n, dtype=np.int32), (nq, 1)), wq).cpu().numpy()[:, :, 3]
    for k, L in ((1, 1), (2, 2), (10, 63), (10, 64), (10, 65), (50, 127), (64, 129), (10, 400), (20, n + 9)):
        print(degree, k, L, flush=True)
        ids, sc = [t.cpu().numpy() for t in ix.search_batch_entities(qs, k, L, kgs.q_ent, 0.7, 2, wq)]
        counts = ix.search_stats(nq)[0].cpu().numpy()
        for qi in range(nq):
            oi, os_, log, _ = O.search_kg(D, sem, ent, Q, qi, wq[qi], k, L, kgs, le, cnt, en_ip, en, kgs.q_ent[qi], 0.7, max_hops=2,
                                          score_table=table[qi], log=True)
            assert np.array_equal(ids[qi], oi) and np.array_equal(sc[qi], os_) and counts[qi, 0] == len(log), (qi, k, L)
    ix.close()
