"""The walk of the prune stage asks what it needs ahead: bits per pair of neighbours and per keyword of the node.  Its decisions are
the oracle's, replayed on the kernel's own similarities, where the words of those bits begin and end and where a node has so many
keywords that they are searched in another way (tables up to 128, a list in LDS up to 512, lists in memory beyond)."""
import numpy as np
import pytest

import oracle as O
from paper_2511_00855_amd import binding as B
from paper_2511_00855_amd.synth import VecSet

pytestmark = pytest.mark.gpu

COUNTS = [1, 2, 31, 32, 33, 64, 65, 127, 128, 129, 255, 256, 511, 512, 513, 700]   # keywords of a document, one after the other


def _corpus(n, rng):
    centers = rng.standard_normal((20, 32)).astype(np.float32)
    dense = centers[rng.integers(0, 20, n)] + 0.1 * rng.standard_normal((n, 32)).astype(np.float32)
    dense *= rng.uniform(0.2, 3.0, (n, 1)).astype(np.float32) / np.linalg.norm(dense, axis=1, keepdims=True)   # the IP rule rejects many
    sizes = np.array([COUNTS[i % len(COUNTS)] for i in range(n)])
    rows = [np.sort(rng.permutation(900)[:s]) if s > 64 else np.sort(rng.permutation(80)[:s]) for s in sizes]   # short lists share keywords
    ip = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    sp = np.arange(0, 2 * n + 1, 2, dtype=np.int64)
    spi = np.concatenate([np.sort(rng.permutation(50)[:2]) for _ in range(n)]).astype(np.int32)
    return VecSet(n, 32, dense.astype(np.float32), sp, spi, rng.uniform(0.1, 1.0, 2 * n).astype(np.float32), ip,
                  np.concatenate(rows).astype(np.int32), rng.integers(1, 4, int(sizes.sum())).astype(np.float32), 50, 900)


@pytest.mark.parametrize("K,R", [(1, 2), (31, 8), (32, 32), (33, 16), (64, 24), (65, 64), (127, 64), (128, 128), (129, 64), (256, 128)])
def test_walk_against_the_oracle(K, R):
    rng, n = np.random.default_rng(K), 320
    d = _corpus(n, rng)
    wv = np.array([1.0, 0.01, 0.002], np.float32)
    docs = B.DeviceVecs(d)
    ix = B.Index.ingest(docs, B.build_params(4, knn_k=4, build_w=tuple(wv)))
    D = O.encode_docs(d)
    nodes = np.arange(64, dtype=np.int32)
    ids = np.full((n, K), -1, np.int32)
    sc = np.full((n, K), -np.inf, np.float32)
    for u in nodes:
        ids[u] = rng.permutation(np.delete(np.arange(n), u))[:K]
        sc[u] = np.sort(rng.normal(0.3, 0.6, K).astype(np.float32))[::-1]
        if u % 5 == 0 and K > 2:   # holes
            ids[u, K - 1 - u % 3:] = -1
            sc[u, K - 1 - u % 3:] = -np.inf
    print(K, R, flush=True)
    g = {k: v.cpu().numpy() for k, v in ix.stage_prune(K, R, ids, sc, nodes).items()}
    self_gpu = ix.export_ingest()[3].cpu().numpy()
    turned_away = 0
    for x, u in enumerate(nodes):
        cnt, order = O.detour_sort(ids[u], sc[u], g["pm"][x])
        assert np.array_equal(g["count"][x], cnt) and np.array_equal(g["sorted_ids"][x], ids[u][order]), u
        self_s = np.where(ids[u] >= 0, self_gpu[np.maximum(ids[u], 0)], -np.inf).astype(np.float32)
        se_pos, ke_pos, fl = O.ip_prune(D, int(u), R, R // 2, ids[u], order, g["pm"][x], self_s)
        assert np.array_equal(g["se"][x][:len(se_pos)], ids[u][se_pos]) and (g["se"][x][len(se_pos):] == -1).all(), u
        assert g["ke_count"][x] == len(ke_pos) and np.array_equal(g["ke"][x][:len(ke_pos)], ids[u][ke_pos]), u
        assert (g["ke"][x][len(ke_pos):] == -1).all() and np.array_equal(g["flag"][x], fl), u
        turned_away += int((ids[u] >= 0).sum()) - len(se_pos)
    assert K < 31 or turned_away > 0
    ix.close()
