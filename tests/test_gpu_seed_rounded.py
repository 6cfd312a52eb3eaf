"""Seed lists of f32 rows out of a sweep over the rows rounded to bf16, whose candidates are scored again in f32: the same
ids and scores, bit for bit, as the one-sided f32 products give."""
import numpy as np
import pytest
import torch

from paper_2511_00855_amd import binding as B
from paper_2511_00855_amd.synth import make_workload

pytestmark = pytest.mark.gpu


def _lists(docs, K, one_sided):
    B.debug_set("seed_one_sided", one_sided)
    try:
        ix = B.Index.ingest(docs, B.build_params(8, knn_k=max(K, 8), nd_rounds=1, nd_sample=4, n_entry=4))
        out = [t.clone() for t in ix.stage_seed_knn(K)]
        flops = ix.build_counters()["seed_flops"]
        ix.close()
    finally:
        B.debug_reset()
    return out, flops


# the smallest corpus it takes; widths that are no multiple of a chunk, the narrowest and the widest; ragged last tiles; few and
# most neighbours; beyond the smallest corpus of the f32 sweep
@pytest.mark.parametrize("n,dim,K,kind", [
    (16384, 4, 1, "plain"), (16641, 100, 200, "plain"), (20001, 260, 64, "norms"), (18000, 1024, 128, "plain"), (16500, 68, 256, "plain"),
    (33001, 36, 32, "norms"), (17000, 64, 100, "ties"),
    # one row dwarfs the others, a value is no number, all rows nearly the same: the f32 products decide
    (17000, 64, 32, "giant"), (17000, 64, 32, "nan"), (17000, 64, 32, "alike")])
def test_rounded_sweep_gives_the_lists_of_the_f32_products(n, dim, K, kind):
    print(f"rounded seed sweep n={n} dim={dim} K={K} {kind}", flush=True)
    w = make_workload("tiny", seed=n + dim, n=n, nq=1, dim=dim, sp=("fixed", 2), tx=("fixed", 2))
    rng = np.random.default_rng(dim)
    d = np.ascontiguousarray(w.docs.dense, dtype=np.float32)
    if kind == "norms":
        d = d * rng.uniform(0.3, 2.0, (n, 1)).astype(np.float32)
    elif kind == "ties":         # every row eight times: equal scores, ranked by id
        d = d[rng.integers(0, n // 8, n)]
    elif kind == "giant":
        d = d.copy()
        d[n // 3] *= 1e6
    elif kind == "nan":
        d = d.copy()
        d[5, 3] = np.nan
    elif kind == "alike":
        d = (d[:1] + 1e-4 * d).astype(np.float32)
    w.docs.dense = np.ascontiguousarray(d)
    docs = B.DeviceVecs(w.docs)
    want, f_want = _lists(docs, K, 1)
    got, f_got = _lists(docs, K, 0)
    assert torch.equal(got[0], want[0])
    assert torch.equal(got[1].view(torch.int32), want[1].view(torch.int32))
    assert (f_got == f_want) == (kind in ("giant", "nan")), (f_got, f_want)   # which sweep it was


@pytest.mark.parametrize("n,dim,K", [(20001, 100, 64), (33001, 64, 32)])
def test_rows_much_alike_are_not_swept_twice(n, dim, K):
    """Rows around one direction, and rows of which one in seven has near duplicates: the same lists, and what the products of the
    rounded rows may cost beside those of the f32 rows."""
    rng = np.random.default_rng(n)
    w = make_workload("tiny", seed=n, n=n, nq=1, dim=dim, sp=("fixed", 2), tx=("fixed", 2))
    plain = np.ascontiguousarray(w.docs.dense, dtype=np.float32)
    kd = (dim + 63) // 64 * 64
    for kind in ("direction", "duplicates"):
        d = plain.copy()
        if kind == "direction":
            d = plain[:1] + 1e-2 * d
        else:
            m = n // 7
            d[rng.permutation(n)[:m]] = plain[rng.integers(0, max(1, m // 300), m)] + 1e-4 * plain[:m]
        w.docs.dense = np.ascontiguousarray(d)
        docs = B.DeviceVecs(w.docs)
        want, f_want = _lists(docs, K, 1)
        got, f_got = _lists(docs, K, 0)
        assert torch.equal(got[0], want[0]) and torch.equal(got[1].view(torch.int32), want[1].view(torch.int32)), kind
        if kind == "direction":   # 1,024 rows and at most 8,192 columns
            assert f_got - f_want <= 2.0 * 1024 * 8192 * kd, (f_got, f_want)
        else:   # the rounded sweep over the tiles of the upper triangle and what it takes its thresholds from; score rows of half the documents at most
            assert f_got <= 1.1 * n * n * kd + 2.0 * n * 8192 * kd + 1.1 * n * n * dim, (f_got, f_want)


@pytest.mark.parametrize("n", [512, 600, 1023, 1024, 1300])
def test_the_sample_is_no_larger_than_the_corpus(debug_knobs, n):
    """A small sample of columns takes a corpus of a few hundred rows to the rounded sweep: the rows that are looked at before it
    are whole tiles of the corpus, at most 1,024."""
    dim, K = 64, 16
    print(f"rounded seed sweep of a small corpus n={n}", flush=True)
    w = make_workload("tiny", seed=n, n=n, nq=1, dim=dim, sp=("fixed", 2), tx=("fixed", 2))
    docs = B.DeviceVecs(w.docs)
    debug_knobs("seed_one_sided", 1)
    ix = B.Index.ingest(docs, B.build_params(8, knn_k=K, nd_rounds=1, nd_sample=4, n_entry=4))
    want = [t.clone() for t in ix.stage_seed_knn(K)]
    debug_knobs("seed_one_sided", 0)
    debug_knobs("seed_sample_cols", 128)
    flops = []
    for cap in (4096, 0):   # with the buffers' size set nothing is looked at first
        debug_knobs("seed_buffer_cap", cap)
        f0 = ix.build_counters()["seed_flops"]
        got = ix.stage_seed_knn(K)
        assert torch.equal(got[0], want[0]) and torch.equal(got[1].view(torch.int32), want[1].view(torch.int32))
        flops.append(ix.build_counters()["seed_flops"] - f0)
    assert flops[1] - flops[0] == 2.0 * min(1024, n // 256 * 256) * 128 * dim
    ix.close()


def test_which_rows_were_multiplied():
    """What the index says about its seed stage: rounded rows, f32 rows where one dwarfs the others, f32 rows of a small corpus,
    stored bf16 rows."""
    for n, base, giant, want in ((16384, "tiny", False, True), (16384, "tiny", True, False), (2000, "tiny", False, False), (2000, "cfg3", False, True)):
        w = make_workload(base, seed=n, n=n, nq=1, dim=64, vocab=5_000, sp=("fixed", 2), tx=("fixed", 2))
        if giant:
            w.docs.dense = np.array(w.docs.dense, dtype=np.float32)
            w.docs.dense[n // 3] *= 1e6
        ix = B.Index.ingest(B.DeviceVecs(w.docs, bf16=base == "cfg3"), B.build_params(8, knn_k=16, nd_rounds=1, nd_sample=4, n_entry=4))
        ix.stage_seed_knn(16)
        assert ix.seed_products_bf16() == want, (n, base, giant)
        ix.close()


def test_little_memory():
    """The rounded sweep fits what is free, the score rows of the near duplicates that it leaves open do not: the f32 sweep gives
    the lists, as it would have from the start."""
    n, dim, K = 40_000, 1024, 32
    w = make_workload("tiny", seed=5, n=n, nq=1, dim=dim, sp=("fixed", 2), tx=("fixed", 2))
    rng = np.random.default_rng(5)
    d = np.array(w.docs.dense, dtype=np.float32)
    m = n // 20
    d[rng.permutation(n)[:m]] = d[rng.integers(0, m // 400, m)] + 1e-4 * d[:m]
    w.docs.dense = d
    docs = B.DeviceVecs(w.docs)
    want, _ = _lists(docs, K, 1)
    ix = B.Index.ingest(docs, B.build_params(8, knn_k=K, nd_rounds=1, nd_sample=4, n_entry=4))
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    hold, left = [], 430_000_000   # 164 MB of candidates, 82 of rounded rows, 138 of sampled scores; 320 of score rows
    while torch.cuda.mem_get_info()[0] > left + (4 << 20):
        hold.append(torch.empty(max(torch.cuda.mem_get_info()[0] - left, 2 << 20), dtype=torch.uint8, device="cuda:0"))
    print("free", torch.cuda.mem_get_info()[0] >> 20, "MB", flush=True)
    got = ix.stage_seed_knn(K)
    assert torch.equal(got[0], want[0]) and torch.equal(got[1].view(torch.int32), want[1].view(torch.int32))
    del hold
    torch.cuda.empty_cache()
    ix.close()
