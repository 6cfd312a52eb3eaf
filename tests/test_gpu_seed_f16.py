"""The rounded seed sweep scales its rows by a power of two so that f16 holds them: tiny and huge rows, and rows of which many values are too
small for f16 beside the largest, give the lists and scores of the f32 products, bit for bit."""
import numpy as np
import pytest
import torch

from paper_2511_00855_amd import binding as B
from paper_2511_00855_amd.synth import make_workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,K,kind", [(64, 32, "tiny"), (100, 64, "huge"), (260, 16, "wide"), (64, 128, "wide"), (36, 32, "powers")])
def test_scaled_rows(debug_knobs, dim, K, kind):
    n = 16_500
    w = make_workload("tiny", seed=dim, n=n, nq=1, dim=dim, sp=("fixed", 2), tx=("fixed", 2))
    d = np.array(w.docs.dense, dtype=np.float32)
    rng = np.random.default_rng(K)
    if kind == "tiny":
        d *= 1e-9
    elif kind == "huge":
        d *= 3e14
    elif kind == "wide":     # from 2^15 down to far below the smallest f16 number
        d *= np.exp(4 * rng.standard_normal((n, dim))).astype(np.float32)
        d /= np.linalg.norm(d, axis=1, keepdims=True)
    else:                    # rows of a few powers of two: scores tie
        d = np.ldexp(np.float32(1), rng.integers(-3, 1, (n, dim))).astype(np.float32) * rng.choice([-1, 1], (n, dim)).astype(np.float32)
    w.docs.dense = np.ascontiguousarray(d, dtype=np.float32)
    docs = B.DeviceVecs(w.docs)
    got = {}
    for one_sided in (1, 0):
        debug_knobs("seed_one_sided", one_sided)
        ix = B.Index.ingest(docs, B.build_params(8, knn_k=K, nd_rounds=1, nd_sample=4, n_entry=4))
        got[one_sided] = [t.clone().view(torch.int32) for t in ix.stage_seed_knn(K)]
        print(dim, K, kind, one_sided, ix.seed_products_bf16(), flush=True)
        assert ix.seed_products_bf16() == (one_sided == 0)
        ix.close()
    assert all(torch.equal(a, b) for a, b in zip(got[0], got[1]))
