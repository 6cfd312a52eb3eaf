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
