"""Neighbourhood similarities of lists: columns with few holders are added pair by pair, the others multiplied as a matrix;
neighbourhoods with too many columns, or too many entries of columns with few holders, are multiplied whole."""
import numpy as np
import pytest
import torch

from paper_2511_00855_amd import binding as B
from paper_2511_00855_amd.synth import make_workload

pytestmark = pytest.mark.gpu


def _uniform_lists(rng, n, width, terms):
    idx = np.concatenate([np.sort(rng.choice(terms, width, replace=False)) for _ in range(n)]).astype(np.int32)
    return np.arange(0, n * width + 1, width, dtype=np.int64), idx


# few columns of either kind; every column at the limit of 8 holders and one beyond it; 128 x 190 entries over 8,000 terms: more than
# 4,096 columns; over 4,000 terms: more than 6,144 entries; lists at the end of the registers and beyond it; a matrix whose
# rows cannot be stored in fours
@pytest.mark.parametrize("K,width,terms", [(9, 20, 90), (128, 8, 128), (128, 9, 128), (128, 190, 8000), (128, 190, 4000), (64, 192, 3000),
                                           (64, 193, 3000), (126, 40, 900), (128, 120, 12000), (5, 3, 3)])
def test_pairs_and_matrix_against_64_bits(K, width, terms):
    n = 300
    w = make_workload("tiny", seed=K + width, n=n, nq=2, dim=64, vocab=16384, sp=("fixed", 4), tx=("fixed", 4))
    rng = np.random.default_rng(width)
    d = w.docs
    d.sp_indptr, d.sp_idx = _uniform_lists(rng, n, width, terms)
    d.sp_val = np.abs(rng.standard_normal(len(d.sp_idx))).astype(np.float32)
    docs = B.DeviceVecs(d)
    ix = B.Index.ingest(docs, B.build_params(4, knn_k=K, n_entry=4, build_w=(0.0, 1.0, 0.0)))
    ids = np.stack([rng.permutation(np.setdiff1d(np.arange(n), [u]))[:K] for u in range(n)]).astype(np.int32)
    sc = -np.sort(-rng.random((n, K)).astype(np.float32), axis=1)
    sub = np.arange(0, n, 23).astype(np.int32)
    pm = ix.stage_prune(K, 4, ids, sc, sub)["pm"]
    assert torch.equal(pm, ix.stage_prune(K, 4, ids, sc, sub)["pm"])
    ix.close()
    X = torch.zeros(n, terms, dtype=torch.float64)
    X[np.repeat(np.arange(n), width), d.sp_idx] = torch.from_numpy(d.sp_val.astype(np.float64))
    for r, u in enumerate(sub):
        Y = X[ids[u]]
        want, got = Y @ Y.T, pm[r].double().cpu()
        # sums of at most `width` products that are not negative: each addition and product rounds by 2^-24 of the sum at most
        assert ((got - want).abs() <= (width + 4) * 2.0 ** -24 * want).all()


# both sides of the number of columns from which those with few holders are set apart, which depends on K; the second vocabulary alone,
# and both in one workgroup
@pytest.mark.parametrize("K,sp,tx,terms,weights", [
    (32, 100, 4, 1900, (0, 1, 0)), (32, 190, 4, 3000, (0, 1, 0)), (48, 50, 4, 900, (0, 1, 0)), (48, 100, 4, 1900, (0, 1, 0)),
    (128, 4, 50, 1500, (0, 0, 1)), (128, 4, 190, 4000, (0, 0, 1)), (128, 50, 50, 1500, (0, 0.5, 0.5)), (128, 60, 50, 1500, (0, 0.5, 0.5)),
    (128, 50, 2, 1500, (0, 0.5, 0.5)), (64, 100, 100, 2500, (0, 0.25, 1))])
def test_both_vocabularies_against_64_bits(K, sp, tx, terms, weights):
    n = 300
    w = make_workload("tiny", seed=K + sp, n=n, nq=2, dim=64, vocab=16384, sp=("fixed", 4), tx=("fixed", 4))
    rng = np.random.default_rng(sp + tx)
    d = w.docs
    d.sp_indptr, d.sp_idx = _uniform_lists(rng, n, sp, terms)
    d.sp_val = np.abs(rng.standard_normal(len(d.sp_idx))).astype(np.float32)
    d.tx_indptr, d.tx_idx = _uniform_lists(rng, n, tx, terms)
    d.tx_val = rng.integers(1, 5, len(d.tx_idx)).astype(np.float32)
    ix = B.Index.ingest(B.DeviceVecs(d), B.build_params(4, knn_k=K, n_entry=4, build_w=weights))
    ids = np.stack([rng.permutation(np.setdiff1d(np.arange(n), [u]))[:K] for u in range(n)]).astype(np.int32)
    sc = -np.sort(-rng.random((n, K)).astype(np.float32), axis=1)
    sub = np.arange(0, n, 23).astype(np.int32)
    pm = ix.stage_prune(K, 4, ids, sc, sub)["pm"]
    assert torch.equal(pm, ix.stage_prune(K, 4, ids, sc, sub)["pm"])
    bm25 = ix.export_ingest()[0].double().cpu()
    ix.close()
    X = torch.zeros(n, 2 * terms, dtype=torch.float64)
    X[np.repeat(np.arange(n), sp), d.sp_idx] = torch.from_numpy(d.sp_val.astype(np.float64)) * np.sqrt(weights[1])
    X[np.repeat(np.arange(n), tx), terms + d.tx_idx] = bm25 * np.sqrt(weights[2])
    for r, u in enumerate(sub):
        Y = X[ids[u]]
        want, got = Y @ Y.T, pm[r].double().cpu()
        # as above, and two roundings of the fusion
        assert ((got - want).abs() <= (max(sp, tx) + 6) * 2.0 ** -24 * want).all()
