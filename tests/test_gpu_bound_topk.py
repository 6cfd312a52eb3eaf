"""Exact top-k out of the table of bounds: a thread keeps the four best of its share of the row (four documents in every 2,048 or 4,096:
up to 512 queries, 1,024 for k > 64, get 1,024 threads each, more of them 512).  The
results are those of scoring everything, also where the best documents all lie in one share, where all scores tie, and at the
smallest corpus that takes this way."""
import numpy as np
import pytest
import torch

from paper_2511_00855_amd import binding as B
from paper_2511_00855_amd.synth import make_workload, subset_vecset

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nq", [37, 513, 1025])
@pytest.mark.parametrize("n,dim,bf16,where", [(4096, 64, False, "spread"), (4099, 100, False, "one share"), (20_001, 64, True, "one share"), (9000, 1544, True, "spread"),
                                              (12_345, 768, False, "one share"), (5000, 32, False, "alike")])
def test_against_all_scores(n, dim, bf16, where, nq):
    w = make_workload("tiny", seed=6, n=n, nq=nq, dim=dim, bf16=bf16)
    d = w.docs
    rng = np.random.default_rng(2)
    if where == "one share":   # up to 40 documents that score far above the others, for every query
        best = np.array([2048 * i + e for i in range(10) for e in range(4) if 2048 * i + e < n])
        w.queries.dense[:] = np.abs(w.queries.dense)
        d.dense[best] = np.abs(rng.standard_normal((len(best), dim))).astype(np.float32) * 9
    elif where == "alike":
        d.dense[:] = d.dense[0]
        d.sp_idx[:], d.sp_val[:] = np.tile(d.sp_idx[:32], n), 1.0
    if bf16:
        bits = torch.from_numpy(d.dense).bfloat16()
        d.dense, d.dense_bf16 = bits.float().numpy(), bits.view(torch.int16).numpy().view(np.uint16)
    docs, qs = B.DeviceVecs(d, bf16=bf16), B.DeviceVecs(w.queries)
    ix = B.Index.ingest(docs, B.build_params(8))
    pw = rng.uniform(0.1, 1.0, (nq, 3)).astype(np.float32)
    pw[3], pw[4], pw[5] = [1.0, 0.0, 0.0], [0.0, 0.0, 1.0], [0.5, -0.3, -0.2]   # the last two: thousands of candidates
    if where == "alike":
        pw[::2, 2] = 0.0
    want, at = [], []
    for a in range(0, nq, 205):   # some queries at a time: four scores of every pair
        some = B.DeviceVecs(subset_vecset(w.queries, np.arange(a, min(a + 205, nq))))
        sc = ix.hybrid_scores(some, np.tile(np.arange(n, dtype=np.int32), (some.n, 1)), pw[a:a + 205])[:, :, 3]
        top, first = torch.sort(sc, dim=1, descending=True, stable=True)
        want.append(top[:, :256]); at.append(first[:, :256])
    want, at = torch.cat(want), torch.cat(at)
    for k in (1, 4, 5, 10, 100, 256):
        print(n, dim, where, k, flush=True)
        ids, got = ix.bruteforce_topk(qs, k, pw)
        assert torch.equal(got, want[:, :k]) and torch.equal(ids, at[:, :k].to(torch.int32)), k
    ix.close()
