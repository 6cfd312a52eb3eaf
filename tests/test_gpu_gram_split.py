"""Dense parts of a neighbourhood's similarities from f32 rows as sums of products of bf16 parts, against 64 bits; neighbourhoods with rows
whose values three bf16 ones may not hold take the f32 instructions."""
import numpy as np
import pytest
import torch

from paper_2511_00855_amd import binding as B
from paper_2511_00855_amd.synth import make_workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,K", [(4, 16), (36, 33), (96, 128), (260, 100), (1024, 48)])
@pytest.mark.parametrize("odd", [None, 1e16, 1e-13, 0.0])
def test_dense_parts(dim, K, odd):
    n = 300
    w = make_workload("tiny", seed=dim, n=n, nq=2, dim=dim, sp=("fixed", 4), tx=("fixed", 4))
    g = torch.Generator().manual_seed(K)
    x = torch.randn(n, dim, generator=g) * torch.exp(2 * torch.randn(n, dim, generator=g))
    if odd is not None:
        x[::50] *= odd / x[::50].norm(dim=1, keepdim=True)
    w.docs.dense[:] = x.numpy()
    docs = B.DeviceVecs(w.docs)
    ix = B.Index.ingest(docs, B.build_params(16, knn_k=K, build_w=(1.0, 0.0, 0.0)))
    knn = torch.stack([torch.randperm(n, generator=g)[:K] for _ in range(n)]).to(torch.int32)
    knn[:, K - 1] = -1   # a list that is not full
    pm = ix.stage_prune(K, 16, knn, torch.zeros(n, K))["pm"].cpu().double()[:, :K - 1, :K - 1]
    X = x.double()[knn.long()[:, :K - 1]]
    ref = X @ X.transpose(1, 2)
    size = X.norm(dim=2)[:, :, None] * X.norm(dim=2)[:, None, :]
    below = torch.tril(torch.ones(K - 1, K - 1, dtype=torch.bool), -1)
    # dim additions of f32 products, each rounded by at most 2^-24 of a partial sum that is no larger than |a||b|; numbers below 1e-37 underflow
    assert bool(((pm - ref).abs() <= dim * 2.0 ** -24 * size + 1e-37)[:, below].all())
    ix.close()


# rows whose columns are all of a size, all positive, of sizes far apart, and rows of which only one, three or twelve columns are not zero
@pytest.mark.parametrize("dim,kind", [(4, 0), (16, 0), (96, 0), (96, "positive"), (96, 1), (96, 3), (260, 0), (260, "apart"), (768, 0), (768, "positive"),
                                      (768, 1), (768, 3), (768, 12), (1024, 0), (1024, 1), (1024, 12), (1024, "apart")])
def test_no_less_precise_than_f32_instructions(dim, kind):
    """The same pairs in neighbourhoods that end in a row whose norm sends them to the f32 instructions."""
    n, K = 400, 100
    w = make_workload("tiny", seed=dim, n=n, nq=2, dim=dim, sp=("fixed", 4), tx=("fixed", 4))
    g = torch.Generator().manual_seed(dim)
    x = torch.randn(n, dim, generator=g)
    if kind == "positive":
        x = x.abs() + 0.5
    elif kind == "apart":
        x *= torch.exp(2 * torch.randn(n, dim, generator=g))
    elif kind:
        x[:, torch.randperm(dim, generator=g)[kind:]] = 0
    x[n - 1] *= 1e16 / x[n - 1].norm()
    w.docs.dense[:] = x.numpy()
    docs = B.DeviceVecs(w.docs)
    ix = B.Index.ingest(docs, B.build_params(16, knn_k=K, build_w=(1.0, 0.0, 0.0)))
    knn = torch.stack([torch.randperm(n - 1, generator=g)[:K] for _ in range(n)]).to(torch.int32)
    X = x.double()[knn.long()[:, :K - 1]]
    ref, size = X @ X.transpose(1, 2), X.norm(dim=2)[:, :, None] * X.norm(dim=2)[:, None, :]
    below = torch.tril(torch.ones(K - 1, K - 1, dtype=torch.bool), -1)
    off = []
    for last in (n - 1, -1):
        knn[:, K - 1] = last
        pm = ix.stage_prune(K, 16, knn, torch.zeros(n, K))["pm"].cpu().double()[:, :K - 1, :K - 1]
        e = ((pm - ref).abs() / size)[:, below]
        off.append((float(e.max()), float((e ** 2).mean().sqrt())))
    print(dim, kind, "f32 instructions %.3e %.3e" % off[0], "split %.3e %.3e" % off[1], flush=True)
    # of two million pairs the largest and the mean square; of a single column both round once, the split after a sum of the smaller products, a 128th
    # of the value, that has lost less than two of its own last places: 2^-6 of a rounding at most, some hundredth
    assert off[1][0] <= (1 + 2.0 ** -6) * off[0][0] and off[1][1] <= (1 + 2.0 ** -6) * off[0][1]
    ix.close()
