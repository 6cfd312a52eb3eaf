"""Large pools with a floor: the bit beside a document's visited bit says whether its bound reaches the floor, and the first iterations
take lower floors.  The same ids, scores and counts as without bounds, bit for bit, where the words of the bitmaps and the sample that the floors
are made of end raggedly."""
import numpy as np
import pytest
import torch

from paper_2511_00855_amd import binding as B
from paper_2511_00855_amd.synth import make_workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,width,beam", [(1999, 16, 1100), (4096, 16, 1100), (9_001, 16, 1100), (4129, 9, 3000), (12_287, 5, 4200), (20_033, 1, 4200)])
def test_marked_floors(debug_knobs, n, width, beam):
    w = make_workload("tiny", seed=n, n=n, nq=40)
    if n == 9_001:   # a corpus of a few documents many times over: bounds that tie with the floors
        w.docs.dense[:] = w.docs.dense[np.arange(n) % 7]
    docs, qs = B.DeviceVecs(w.docs), B.DeviceVecs(w.queries)
    ix = B.Index.build(docs, B.build_params(64, nd_rounds=1, n_entry=16))
    pw = np.random.default_rng(n).uniform(-0.1, 1.0, (qs.n, 3)).astype(np.float32)
    pw[:4] = [[0, 0, 0], [1, 0, 0], [0, 0, 1], [np.nan, 1, 0]]
    got = {}
    for mode, floor in ((1, 0), (2, 0), (2, 2)):   # without bounds; with a floor; with one so high that what waits is asked for
        print(n, width, beam, mode, floor, flush=True)
        debug_knobs("search_bounds", mode)
        debug_knobs("search_floor", floor)
        got[mode, floor] = [t.clone().view(torch.int32) for t in ix.search_batch(qs, 20, beam, pw, search_width=width)]
        got[mode, floor].append(ix.search_stats(qs.n)[0][:, :2].clone())
        assert ix.search_form()["threads"] == 512
    for key in got:
        assert all(torch.equal(a, b) for a, b in zip(got[1, 0], got[key])), key
    ix.close()


# pools that two, four and eight waves search, and one that holds all documents
@pytest.mark.parametrize("n,nq,beam,threads", [(30_000, 2400, 64, 128), (30_000, 1500, 256, 256), (30_000, 1500, 1200, 512), (1_400, 20_000, 1200, 512)])
def test_marks_are_laid_out_where_a_floor_is_taken(debug_knobs, n, nq, beam, threads):
    """A search with a limit of iterations takes no floor: what a small pool's search takes of memory is no more than that."""
    w = make_workload("tiny", seed=1, n=n, nq=nq, dim=64, sp=("fixed", 8), tx=("fixed", 8))
    rng = np.random.default_rng(1)
    docs, qs = B.DeviceVecs(w.docs), B.DeviceVecs(w.queries)
    graph, entry = rng.integers(0, n, (n, 64)).astype(np.int32), rng.permutation(n)[:16].astype(np.int32)
    debug_knobs("search_bounds", 2)
    debug_knobs("search_walk", 1)
    took = []
    for iters in (1, 0):
        ix = B.Index.import_graph(docs, B.build_params(64, n_entry=16), graph, entry)
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        before = torch.cuda.mem_get_info()[0]
        ix.search_batch(qs, 10, beam, max_iters=iters, search_width=1 if threads < 512 else 16)
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        took.append(before - torch.cuda.mem_get_info()[0])
        print(beam, iters, ix.search_form(), took, flush=True)
        assert ix.search_form()["threads"] == threads
        ix.close()
    words = nq * (n // 32) * 8   # bytes of the marks
    assert took[1] - took[0] < words // 2 if threads < 512 or beam * 1.25 >= n else took[1] - took[0] > words // 2
