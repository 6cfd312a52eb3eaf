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
