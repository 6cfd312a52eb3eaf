"""A batch a little too large to run at once is searched by workgroups of two waves, its halves by workgroups of four: the same ids,
scores and counts, bit for bit."""
import numpy as np
import pytest
import torch

from paper_2511_00855_amd import binding as B
from paper_2511_00855_amd.synth import make_keywords, make_workload, subset_vecset

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bf16,dim,degree,nq", [(False, 128, 64, 2300), (False, 768, 16, 1972), (True, 1024, 32, 3584), (True, 1536, 64, 2000)])
def test_two_waves_and_four(debug_knobs, bf16, dim, degree, nq):
    w = make_workload("tiny", seed=3, n=1700, nq=nq, dim=dim, bf16=bf16, sp=("poisson", 60))
    docs = B.DeviceVecs(w.docs, bf16=bf16)
    ix = B.Index.build(docs, B.build_params(degree, nd_rounds=1, n_entry=16))
    kw = make_keywords(w.queries, seed=2, max_terms=2, stride=2, p_none=0.1)
    pw = np.random.default_rng(1).uniform(0.0, 1.0, (nq, 3)).astype(np.float32)
    half = nq // 2
    parts = [(0, nq), (0, half), (half, nq)]
    qs = [B.DeviceVecs(w.queries if b - a == nq else subset_vecset(w.queries, np.arange(a, b))) for a, b in parts]
    debug_knobs("search_bounds", 2)
    for deleted in (False, True):
        if deleted:
            ix.mark_deleted(np.arange(0, 1700, 9, dtype=np.int32))
        for beam, glob in ((1, 0), (40, 0), (300, 0), (300, 1)):
            debug_knobs("search_visited_global", glob)
            for words in (False, True):
                print(bf16, dim, nq, beam, glob, words, deleted, flush=True)
                got = []
                for q, (a, b) in zip(qs, parts):
                    k = min(beam, 10)
                    r = ix.search_batch_keywords(q, k, beam, kw[a:b], pw[a:b]) if words else ix.search_batch(q, k, beam, pw[a:b])
                    got.append([t.clone() for t in r] + [ix.search_stats(b - a)[0][:, :2].clone()])
                    # with keywords or deletions a compute unit holds twelve workgroups of two waves: 3,072 queries at once
                    two = b - a == nq and (nq <= 3072 or not (words or deleted))
                    if bf16 and dim > 1024:   # five waves a SIMD: 1,280 queries at once by four waves, and two pay only with keywords or deletions
                        two = two and (words or deleted)
                    assert ix.search_form()["threads"] == (128 if two else 256), (b - a, beam, words, deleted)
                for whole, first, second in zip(*got):
                    assert torch.equal(whole, torch.cat([first, second])), (beam, glob, words, deleted)
    ix.close()


@pytest.mark.parametrize("bf16,dim,cases", [
    (False, 32, ((2400, 1100, 128, False), (2300, 1100, 128, True), (3300, 700, 128, False), (3500, 700, 256, True), (3072, 700, 128, True))),
    (False, 516, ((2400, 1100, 128, False), (2900, 1000, 256, True), (3000, 700, 128, True))),
    (True, 520, ((2400, 1100, 256, True), (2300, 1100, 128, True))),
    (True, 1032, ((1400, 300, 256, True), (2300, 300, 256, True)))])
def test_where_two_waves_keep_their_visited_sets(debug_knobs, bf16, dim, cases):
    """LDS is handed out in blocks of 1,280 bytes.  2,400 queries do not run at once with 15,432 bytes each and the kernel's static arrays
    (nine workgroups a compute unit, not ten): their visited sets stay in memory.  Batches of nearly two rounds of four waves take four
    where only those have the sets in LDS, from 1.6 rounds on where rows are long, and bf16 rows of more than 512 columns always then; wide
    bf16 rows take four whatever fits.  Ids, scores and counts are those of the batch's halves either way."""
    w = make_workload("tiny", seed=5, n=12_000, nq=max(c[0] for c in cases), dim=dim, bf16=bf16, sp=("poisson", 20))
    docs = B.DeviceVecs(w.docs, bf16=bf16)
    ix = B.Index.build(docs, B.build_params(32, nd_rounds=1, n_entry=64))
    debug_knobs("search_bounds", 2)
    for nq, beam, threads, lds in cases:
        print(bf16, dim, nq, beam, flush=True)
        got = []
        for a, b in ((0, nq), (0, nq // 2), (nq // 2, nq)):
            r = ix.search_batch(B.DeviceVecs(subset_vecset(w.queries, np.arange(a, b))), 10, beam)
            if b - a == nq:
                assert ix.search_form() == dict(threads=threads, listed=False, visited_lds=lds), (nq, beam)
            got.append([t.clone() for t in r] + [ix.search_stats(b - a)[0][:, :2].clone()])
        for whole, first, second in zip(*got):
            assert torch.equal(whole, torch.cat([first, second])), (nq, beam)
    ix.close()
