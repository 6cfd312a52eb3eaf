"""The symmetric seed sweeps note a score once and tell its two sides apart when it is written out: ties at the threshold on either side, a
document's own score, and scores of +inf, which reach any threshold, against the path that materialises every score row."""
import numpy as np
import pytest
import torch

from paper_2511_00855_amd import binding as B
from paper_2511_00855_amd.synth import make_workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("n,huge", [(512, 0), (769, 0), (1100, 300)])
def test_scores_that_reach_both_thresholds(debug_knobs, bf16, n, huge):
    w = make_workload("tiny", seed=n, n=n, nq=2, dim=64, bf16=bf16, sp=("fixed", 4), tx=("fixed", 4))
    w.docs.dense[:] = w.docs.dense[np.arange(n) % 5]   # a fifth of the corpus ties for every row's best
    if huge:
        w.docs.dense[-huge:] = 1e20 * np.abs(w.docs.dense[-huge:])   # their products overflow
    if bf16:
        w.docs.dense_bf16[:] = torch.from_numpy(w.docs.dense).to(torch.bfloat16).view(torch.int16).numpy().view(np.uint16)
    docs = B.DeviceVecs(w.docs, bf16=bf16)
    ix = B.Index.ingest(docs, B.build_params(8, knn_k=24, nd_rounds=1, nd_sample=4, n_entry=4))
    exact = [t.clone().view(torch.int32) for t in ix.stage_seed_knn(24)]
    assert bool((exact[0] != torch.arange(n, device=exact[0].device)[:, None]).all())
    debug_knobs("seed_sample_cols", 128)
    for cap in (0, 512):
        debug_knobs("seed_buffer_cap", cap)
        got = [t.view(torch.int32) for t in ix.stage_seed_knn(24)]
        assert all(torch.equal(a, b) for a, b in zip(got, exact)), cap
    ix.close()


# topics of which the first few hundred or thousand documents are only some, or one
@pytest.mark.parametrize("n,bf16", [(33_000, True), (17_000, False), (33_000, False)])
@pytest.mark.parametrize("topic", [300, 5_000])
def test_corpora_in_the_order_of_their_topics(n, bf16, topic):
    """The thresholds come from documents of every topic: no more rows are left to the exact path than of the same documents in no order."""
    dim, K = 64, 128
    w = make_workload("tiny", seed=topic, n=n, nq=1, dim=dim, sp=("fixed", 2), tx=("fixed", 2), bf16=bf16)
    rng = np.random.default_rng(topic)
    centre = rng.standard_normal((n // topic + 1, dim))
    d = rng.standard_normal((n, dim)) * 0.7 + centre[np.arange(n) // topic]
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    order, flops, ids = rng.permutation(n), [], []
    for rows in (d, d[order]):
        t = torch.from_numpy(rows.astype(np.float32))
        if bf16:
            t = t.bfloat16()
            w.docs.dense_bf16 = t.view(torch.int16).numpy().view(np.uint16)
        w.docs.dense = t.float().numpy()
        ix = B.Index.ingest(B.DeviceVecs(w.docs, bf16=bf16), B.build_params(8, knn_k=K, nd_rounds=1, nd_sample=4, n_entry=4))
        got, sc = ix.stage_seed_knn(K)
        flops.append(ix.build_counters()["seed_flops"])
        assert ix.seed_products_bf16()
        ids.append((got.cpu().numpy(), sc.cpu().numpy()))
        ix.close()
    print(n, bf16, topic, flops, flush=True)
    assert flops[0] <= 1.02 * flops[1]
    assert np.array_equal(ids[0][1][order], ids[1][1])   # the same scores, whatever the order
