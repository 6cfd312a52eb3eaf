"""Assembly where reverse lists are far longer than their places, at every shape of a row: a lane holds two of its entries, and the padding
runs through one to four waves' width of the sorted list."""
import numpy as np
import pytest

import oracle as O
from paper_2511_00855_amd import binding as B
from paper_2511_00855_amd.synth import make_workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("R,K,P", [(4, 4, 1), (12, 64, 2), (64, 65, 11), (68, 128, 32), (128, 256, 22), (128, 130, 32)])
def test_long_reverse_lists(R, K, P):
    n, rng = 1100, np.random.default_rng(R + K)
    w = make_workload("tiny", seed=1, n=n, nq=1, dim=8)
    ix = B.Index.ingest(B.DeviceVecs(w.docs), B.build_params(8))
    se, srt, spi = np.full((n, R), -1, np.int32), np.full((n, K), -1, np.int32), np.full((3, n, P), -1, np.int32)
    for u in range(n):
        ids = rng.permutation(np.concatenate([np.arange(6), 6 + rng.choice(n - 6, K, replace=False)]))   # everyone's neighbours: six hubs, anywhere in the list
        srt[u] = ids[ids != u][:K]
        m = int(rng.integers(1, R + 1))
        se[u, :m] = srt[u, :m]
        for p in range(3):
            few = rng.choice(12, min(P, 8), replace=False) if u % 2 else rng.choice(n, P, replace=False)
            spi[p, u, :len(few)] = np.where(few == u, -1, few)
    assert np.array_equal(ix.stage_assemble(R, K, P, se, srt, spi).cpu().numpy(), O.assemble(n, R, K, P, se, srt, spi))
    ix.close()
