"""The rounds of a construction tell by packed lists (three bytes an entry, weights rounded up to 8 bits, rare terms sharing slots)
which candidates can enter a list.  The lists must stay those of rounds that score every candidate, bit for bit: nothing is rounded
but the bounds."""
import numpy as np
import pytest
import torch

from paper_2511_00855_amd import binding as B
from paper_2511_00855_amd.synth import VecSet, make_workload, subset_vecset

pytestmark = pytest.mark.gpu


def _negative(d, rng):   # such a list has no bound; nodes that hold one read every record
    rows = rng.random(d.n) < 0.3
    d.sp_val[np.repeat(rows, np.diff(d.sp_indptr)) & (rng.random(len(d.sp_val)) < 0.5)] *= -1


def _far_apart(d, rng):   # one weight decides a list's scale
    d.sp_val[:] = 10.0 ** rng.uniform(-30, 3, len(d.sp_val))
    d.sp_val[rng.random(len(d.sp_val)) < 0.2] = 0.0


def _beyond(d, rng):   # products of two such weights overflow
    d.sp_val[rng.random(len(d.sp_val)) < 0.01] = 3e38


def _alike(d, rng):   # nothing to tell candidates apart by
    d.sp_val[:], d.tx_val[:] = 1.0, 1.0
    d.dense[:] = d.dense[0]


SP, TX = ("poisson", 100), ("lognormal", 60)
CASES = {   # name: (workload, K, S, P, build weights, what is done to the documents)
    "ordinary": (dict(n=1300, sp=SP, tx=TX), 128, 32, 11, (1.0, 1.0, 1.0), None),
    "rare terms share slots": (dict(n=1500, vocab=200_000, sp=SP, tx=TX), 64, 32, 11, (1.0, 1.0, 1.0), None),
    "units beyond three a lane": (dict(n=600, sp=("fixed", 131), tx=("fixed", 120)), 32, 24, 6, (1.0, 1.0, 1.0), None),
    "lists too long for the tables": (dict(n=520, sp=("fixed", 300), tx=("fixed", 200)), 24, 16, 6, (1.0, 1.0, 1.0), None),
    "fewest that are packed": (dict(n=512, sp=SP, tx=TX), 32, 32, 11, (1.0, 1.0, 1.0), None),
    "one fewer": (dict(n=511, sp=SP, tx=TX), 32, 32, 11, (1.0, 1.0, 1.0), None),
    "too short for it": (dict(n=700, sp=("poisson", 10), tx=("fixed", 10)), 32, 32, 11, (1.0, 1.0, 1.0), None),
    "empty and short lists": (dict(n=14000, sp=("poisson", 1), tx=("fixed", 5)), 32, 32, 32, (1.0, 1.0, 1.0), None),
    "negative weights": (dict(n=900, sp=SP, tx=TX), 64, 32, 11, (1.0, 1.0, 1.0), _negative),
    "weights far apart": (dict(n=900), 64, 32, 11, (1.0, 1.0, 1.0), _far_apart),
    "sums beyond the range": (dict(n=1300), 32, 32, 8, (1.0, 1.0, 1.0), _beyond),
    "documents alike": (dict(n=1400, sp=("fixed", 20), tx=("fixed", 20)), 48, 32, 11, (1.0, 1.0, 1.0), _alike),
    "negative weight of a path": (dict(n=700), 32, 32, 8, (0.5, -1.0, 1.0), None),
    "lexical part alone": (dict(n=1100, sp=SP, tx=TX), 96, 32, 16, (0.0, 0.0, 1.0), None),
}


@pytest.mark.parametrize("name", list(CASES))
def test_packed_lists_change_no_list(name):
    kw, K, S, P, wv, change = CASES[name]
    w = make_workload("tiny", seed=11, nq=2, **kw)
    d = w.docs
    if change:
        change(d, np.random.default_rng(4))
    docs = B.DeviceVecs(d)
    print(name, flush=True)
    bp = B.build_params(16, knn_k=K, nd_rounds=3, nd_sample=S, sp_len=P, n_entry=4, build_w=wv)
    full = B.Index.build(docs, bp)
    assert full.packed_lists() == (name not in ("one fewer", "too short for it", "negative weight of a path"))
    _, srt, spi, sps = full.export_build_state()
    ix = B.Index.ingest(docs, bp)
    ids, sc = ix.stage_seed_knn(K)
    i2 = torch.full((3, d.n, P), -1, dtype=torch.int32, device=docs.device)
    s2 = torch.full((3, d.n, P), -np.inf, dtype=torch.float32, device=docs.device)
    for _ in range(3):
        ids, sc, i2, s2 = ix.stage_refine(K, S, P, ids, i2, s2)
    g = ix.stage_prune(K, 16, ids, sc, want_pm=False)
    assert torch.equal(spi, i2) and torch.equal(sps.view(torch.int32), s2.view(torch.int32))
    assert torch.equal(srt, g["sorted_ids"])
    full.close(); ix.close()


def _longest_lists():
    """Two documents, U and U + 10, with learned-sparse lists of 65,473 terms, of whose sum of products every addition rounds up:
    64 large weights, one at the head of each lane's share, then 1,022 terms a lane whose product is a little more than half a unit
    in the last place above a whole number of them.  All weights lie just below a step of the 8-bit weights, so the packed lists add next
    to nothing.  One other document, U + 1, has a learned-sparse part with U that lies 7e-6 below that sum as it comes out and 5e-5 above
    the exact one."""
    f, n, U, nb, per = np.float32, 600, 300, 64, 1022
    most = f(np.sqrt(1.0034) * 254 / 253)
    scale = f(most * f(f(1.00001) / f(254))); inv = f(f(1.000002) / scale)

    def below(level):   # the largest weight that is rounded up to this step
        x = f(level * scale)
        while int(f(x * inv)) + 1 > level:
            x = np.nextafter(x, f(0))
        return x
    a, s = below(253), below(1)
    lane = f(float(a) ** 2)
    for _ in range(per):   # fused multiply-adds of one lane; the 64 lanes are alike, so their sum is exact
        lane = f(float(lane) + float(s) ** 2)
    exact = nb * (float(a) ** 2 + per * float(s) ** 2)
    total = 64 * float(lane)
    assert total > exact * (1 + 5.5e-5)
    m = nb + 64 * per
    long_idx, long_val = np.arange(m), np.concatenate([np.full(nb, a), np.full(m - nb, s)])
    rng = np.random.default_rng(8)
    sp, tx = [], []
    for u in range(n):
        if u in (U, U + 10):   # the largest weight of each is on a term that the other does not hold
            sp.append((np.append(long_idx, m + (u != U)), np.append(long_val, most)))
        elif u == U + 1:
            sp.append((np.array([m]), np.array([(0.125 * exact + 0.875 * total) / float(most)])))
        else:   # the large terms are frequent, the others share slots
            sp.append((np.append(np.arange(nb), [m, m + 1]), rng.uniform(1e-4, 1e-3, nb + 2)))
        # U and the documents around it, U + 10 not among them, share a keyword: what U + 10 lacks for U's list
        tx.append([1 if U - 12 <= u <= U + 9 else 0])
    ip = lambda rows: np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int64)
    turn = 2 * np.pi * np.arange(n) / n
    dense = np.stack([np.cos(turn), np.sin(turn), 0 * turn, 0 * turn], axis=1).astype(np.float32)
    return VecSet(n, 4, dense, ip([r[0] for r in sp]), np.concatenate([r[0] for r in sp]).astype(np.int32),
                  np.concatenate([r[1] for r in sp]).astype(np.float32), ip(tx), np.concatenate(tx).astype(np.int32), np.ones(n, np.float32), m + 2, 2), U


def test_sums_of_the_longest_lists():
    """A lane's sum may round up at each of its additions, 6e-8 of it at a time: the bound allows for as many as there are."""
    d, U = _longest_lists()
    K, S = 16, 16
    docs = B.DeviceVecs(d)
    bp = B.build_params(16, knn_k=K, nd_rounds=1, nd_sample=S, sp_len=1, n_entry=4, build_w=(1.0, 0.0, 1.0))
    full = B.Index.build(docs, bp)
    assert full.packed_lists()
    _, _, spi, sps = full.export_build_state()
    ix = B.Index.ingest(docs, bp)
    ids, _ = ix.stage_seed_knn(K)
    i2 = torch.full((3, d.n, 1), -1, dtype=torch.int32, device=docs.device)
    s2 = torch.full((3, d.n, 1), -np.inf, dtype=torch.float32, device=docs.device)
    ids, _, i2, s2 = ix.stage_refine(K, S, 1, ids, i2, s2)
    assert int(i2[1, U, 0]) == U + 10 and not bool((ids[U] == U + 10).any())   # it enters the per-path list alone
    assert torch.equal(spi, i2) and torch.equal(sps.view(torch.int32), s2.view(torch.int32))
    full.close(); ix.close()


@pytest.mark.parametrize("bf16,dim,n0", [(False, 96, 1000), (True, 1032, 1003), (False, 128, 3)])
def test_lists_of_the_documents_of_an_insertion(bf16, dim, n0):
    """An insertion packs the lists of its new documents alone: records from the first new one on, slots by the term frequencies of all.
    Its rounds are those that score every candidate, called one by one on the enlarged index."""
    n, K, S, P = n0 + 700, 48, 24, 11
    w = make_workload("tiny", seed=31, n=n, nq=2, dim=dim, bf16=bf16, sp=("poisson", 90), tx=("lognormal", 70))
    d = w.docs
    before = int(d.sp_indptr[n0] + d.tx_indptr[n0])
    if before % 2 == 0:   # an entry less: the new documents' entries begin at an odd place
        d.sp_idx, d.sp_val = d.sp_idx[1:], d.sp_val[1:]
        d.sp_indptr[1:] -= 1
    assert int(d.sp_indptr[n0] + d.tx_indptr[n0]) % 2 == 1
    d.sp_val[d.sp_indptr[n0 + 5]] *= -1   # a list without a scale
    bp = B.build_params(16, knn_k=K, nd_rounds=3, nd_sample=S, sp_len=P, n_entry=4)
    old = B.Index.build(B.DeviceVecs(subset_vecset(d, np.arange(n0)), bf16=bf16), bp)
    docs = B.DeviceVecs(d, bf16=bf16)
    print(bf16, dim, n0, flush=True)
    new, tr = old.insert(docs, trace=True)
    assert new.packed_lists()
    alone = B.Index.ingest(B.DeviceVecs(subset_vecset(d, np.arange(n0, n)), bf16=bf16), bp)
    seeds, _ = alone.stage_seed_knn(K)
    nodes = np.arange(n0, n, dtype=np.int32)
    ids = torch.full((n, K), -1, dtype=torch.int32, device=docs.device)
    i2 = torch.full((3, n, P), -1, dtype=torch.int32, device=docs.device)
    s2 = torch.full((3, n, P), -np.inf, dtype=torch.float32, device=docs.device)
    ids[n0:] = torch.where(seeds >= 0, seeds + n0, seeds)
    for _ in range(3):
        ids[n0:], sc, i2[:, n0:], s2[:, n0:] = new.stage_refine(K, S, P, ids, i2, s2, nodes)
    for mine, theirs in ((tr["cand2_ids"], ids[n0:]), (tr["cand2_sc"], sc), (tr["cand2_sp_ids"], i2[:, n0:]), (tr["cand2_sp_sc"], s2[:, n0:])):
        assert torch.equal(mine.view(torch.int32), theirs.contiguous().view(torch.int32))
    old.close(); new.close(); alone.close()
