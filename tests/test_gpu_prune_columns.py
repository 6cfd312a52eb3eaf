"""Neighbourhood similarities as a matrix product over the shared terms against the list walks: the same f32 products,
summed in another order."""
import numpy as np
import pytest
import torch

from paper_2511_00855_amd import binding as B
from paper_2511_00855_amd.synth import make_workload

pytestmark = pytest.mark.gpu


# blocks of 16 and chunks of 64 columns at and around their edges; lists longer than the 192 entries a wave keeps in
# registers; nothing shared at all (a vocabulary far larger than the lists), everything shared, the largest vocabulary
@pytest.mark.parametrize("K,vocab,sp,tx,dim,bf16", [(4, 10_000, 32, 40, 64, False), (16, 300, 60, 40, 64, False), (17, 10_000, 32, 40, 64, False),
                                                    (64, 5_000, 250, 300, 64, False), (100, 400, 193, 320, 128, True), (128, 262_144, 120, 60, 64, False),
                                                    (127, 250_002, 1, 1, 64, True), (128, 130, 120, 100, 64, False), (65, 64, 64, 20, 64, False)])
def test_columns_against_walks(debug_knobs, K, vocab, sp, tx, dim, bf16):
    n, nodes = 400, 37
    w = make_workload("cfg3" if bf16 else "tiny", seed=3, n=n, nq=4, dim=dim, vocab=vocab, sp=("fixed", sp), tx=("fixed", tx))
    docs = B.DeviceVecs(w.docs, bf16=bf16)
    ix = B.Index.ingest(docs, B.build_params(4, knn_k=K, n_entry=4))
    rng = np.random.default_rng(1)
    ids = np.stack([rng.permutation(np.setdiff1d(np.arange(n), [u]))[:K] for u in range(n)]).astype(np.int32)
    ids[::3, -2:] = -1
    sc = -np.sort(-rng.random((n, K)).astype(np.float32), axis=1)
    sub = np.arange(0, n, n // nodes)[:nodes].astype(np.int32)
    got = {}
    for walks in (0, 1):
        debug_knobs("prune_walks", walks)
        got[walks] = ix.stage_prune(K, 4, ids, sc, sub)["pm"].clone()
    again = ix.stage_prune(K, 4, ids, sc, sub)["pm"]
    assert torch.equal(again, got[1])
    debug_knobs("prune_walks", 0)
    assert torch.equal(ix.stage_prune(K, 4, ids, sc, sub)["pm"], got[0])   # no sum depends on the order in which anything arrives
    a, b = got[0].double(), got[1].double()
    assert torch.equal(torch.isinf(a), torch.isinf(b)) and torch.equal(a, a.transpose(1, 2))
    fin = ~torch.isinf(b)
    # the dense part is the same number on both sides; the lists' parts are sums of at most max(sp, tx) products that are
    # not negative, each within (terms) 2^-24 of the exact sum, and a few roundings of the fusion
    tol = (2 * max(sp, tx) + 8) * 2.0 ** -24 * (b.abs() + 2.0)
    assert ((a - b).abs()[fin] <= tol[fin]).all()
    ix.close()
