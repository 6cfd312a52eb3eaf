"""A construction's rounded seed sweep scores again only the candidates near the lines that its rounds depend on (the last place of a list
and the last of the first nd_sample): its graph and its per-path lists are those of the stages called one by one, whose seed lists are exact."""
import numpy as np
import pytest
import torch

from paper_2511_00855_amd import binding as B
from paper_2511_00855_amd.synth import make_workload

pytestmark = pytest.mark.gpu


# lists longer than the first 32, as long, and shorter; one that counts; many and few open candidates a row (ties by the hundred; f16 rows
# that are exact); the widest rows and a chunk that ends early
@pytest.mark.parametrize("n,dim,R,K,S,P,kind", [
    (16_401, 100, 16, 64, 32, 8, "plain"), (16_384, 64, 16, 32, 32, 4, "norms"), (17_000, 36, 8, 16, 32, 32, "ties"), (16_500, 1024, 16, 200, 1, 6, "plain"),
    (16_500, 64, 32, 100, 20, 11, "ties"), (16_640, 260, 8, 40, 7, 3, "powers")])
def test_construction_equals_its_stages(n, dim, R, K, S, P, kind):
    w = make_workload("tiny", seed=n + K, n=n, nq=1, dim=dim, sp=("fixed", 6), tx=("fixed", 5))
    rng = np.random.default_rng(K)
    d = np.array(w.docs.dense, dtype=np.float32)
    if kind == "norms":
        d *= rng.uniform(0.3, 2.0, (n, 1)).astype(np.float32)
    elif kind == "ties":
        d = d[rng.integers(0, n // 60, n)]
    elif kind == "powers":
        d = (rng.integers(-8, 9, (n, dim)) / np.float32(8)).astype(np.float32)
    w.docs.dense = np.ascontiguousarray(d)
    docs = B.DeviceVecs(w.docs)
    bp = B.build_params(R, knn_k=K, nd_rounds=1, nd_sample=S, sp_len=P, n_entry=4)
    full = B.Index.build(docs, bp)
    assert full.seed_products_bf16()
    ix = B.Index.ingest(docs, bp)
    ids, _ = ix.stage_seed_knn(K)
    spi = torch.full((3, n, P), -1, dtype=torch.int32, device=docs.device)
    sps = torch.full((3, n, P), -np.inf, dtype=torch.float32, device=docs.device)
    ids, sc, spi, sps = ix.stage_refine(K, S, P, ids, spi, sps)
    g = ix.stage_prune(K, R, ids, sc, want_pm=False)
    got = full.export_build_state()
    for name, a, b in zip(("members", "order", "path lists", "path scores"), got, (g["se"], g["sorted_ids"], spi, sps)):
        assert torch.equal(a, b), name
    full.close(); ix.close()
