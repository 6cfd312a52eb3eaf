"""Large pools of which two share a compute unit once an iteration's neighbours are listed by their ids and scored 256 at a time: the
same ids, scores and counts as searches without bounds, which score all of them at once, bit for bit."""
import numpy as np
import pytest
import torch

from paper_2511_00855_amd import binding as B
from paper_2511_00855_amd.synth import make_workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bf16,dim,degree,n_entry", [(False, 128, 64, 256), (True, 1032, 32, 16)])
def test_listed_neighbours(debug_knobs, bf16, dim, degree, n_entry):
    w = make_workload("tiny", seed=13, n=12_000, nq=270, dim=dim, bf16=bf16)
    docs, qs = B.DeviceVecs(w.docs, bf16=bf16), B.DeviceVecs(w.queries)
    ix = B.Index.build(docs, B.build_params(degree, knn_k=degree, nd_rounds=1, n_entry=n_entry))
    pw = np.random.default_rng(1).uniform(-0.1, 1.0, (qs.n, 3)).astype(np.float32)
    # the last three at either degree: lists of 576 ids (or 352) do not end with a block of 256
    for beam, width, iters in ((5000, 16, 0), (8192, 16, 0), (6000, 9, 0), (5000, 16, 40), (7500, 9, 0) if degree == 64 else (8300, 11, 0),
                               (8300, 11, 30), (7500, 16, 25)):
        listed = (degree, beam, width) not in ((64, 6000, 9), (32, 5000, 16), (32, 6000, 9))   # two pools with all candidates beside them fit a compute unit there
        got = {}
        for mode, floor in ((1, 0), (2, 0), (2, 1), (2, 2)):
            print(bf16, beam, width, iters, mode, floor, flush=True)
            debug_knobs("search_bounds", mode)
            debug_knobs("search_floor", floor)
            got[mode, floor] = [t.clone() for t in ix.search_batch(qs, 50, beam, pw, search_width=width, max_iters=iters)]
            got[mode, floor].append(ix.search_stats(qs.n)[0][:, :2].clone())
            assert ix.search_form() == dict(threads=1024 if listed and mode == 1 else 512, listed=listed and mode == 2, visited_lds=False)
        for key in got:
            assert all(torch.equal(a, b) for a, b in zip(got[1, 0], got[key])), (beam, width, iters, key)
    ix.close()
