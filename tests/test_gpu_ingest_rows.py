"""What ingest does with 16 lanes a row: list lengths around their number, in every place of a row."""
import numpy as np
import pytest

from paper_2511_00855_amd import binding as B
from paper_2511_00855_amd.synth import VecSet

pytestmark = pytest.mark.gpu

LENGTHS = np.array([1, 0, 15, 16, 17, 31, 32, 33, 100, 0, 64, 47] * 3)


def _corpus():
    rng, n, vocab = np.random.default_rng(2), len(LENGTHS), 120
    idx = np.concatenate([np.sort(rng.choice(vocab, k, replace=False)) for k in LENGTHS]).astype(np.int32)
    ip = np.concatenate([[0], np.cumsum(LENGTHS)]).astype(np.int64)
    tf = rng.integers(1, 9, len(idx)).astype(np.float32)
    return VecSet(n, 8, rng.standard_normal((n, 8)).astype(np.float32), ip, idx.copy(), tf.copy(), ip.copy(), idx.copy(), tf.copy(), vocab, vocab)


def test_weights_of_lists_around_sixteen_entries():
    v = _corpus()
    p = B.build_params(8)
    ix = B.Index.ingest(B.DeviceVecs(v), p)
    w = ix.export_ingest()[0].cpu().numpy()
    n, df = v.n, np.bincount(v.tx_idx, minlength=v.tx_vocab).astype(np.float64)
    length = np.add.reduceat(np.append(v.tx_val, 0.0).astype(np.float64), v.tx_indptr[:-1]) * (LENGTHS > 0)
    k1, b, tf, d = np.float64(p.bm25_k1), np.float64(p.bm25_b), v.tx_val.astype(np.float64), df[v.tx_idx]
    norm = np.repeat(k1 * (1.0 - b + b * length / (length.sum() / n)), LENGTHS)
    want = (np.log(1.0 + (n - d + 0.5) / (d + 0.5)) * tf * (k1 + 1.0) / (tf + norm)).astype(np.float32)
    assert np.allclose(w, want, rtol=1.2e-7, atol=0.0)   # the doubles may differ in their last place, so the floats by one
    ix.close()


@pytest.mark.parametrize("part", ["sp", "tx"])
@pytest.mark.parametrize("what", ["order", "vocab", "nan", "offset"])
def test_what_is_wrong_is_counted_wherever_it_stands(part, what):
    rows = [2, 3, 4, 7, 8, 11]
    v = _corpus()
    ip, idx, val = getattr(v, part + "_indptr"), getattr(v, part + "_idx"), getattr(v, part + "_val")
    if what == "offset":
        ip[3] = ip[4] + 1    # row 2 is longer than it was (its last entries may be out of order), row 3 ends before it begins
    for r in rows if what != "offset" else []:
        last = ip[r + 1] - 1
        if what == "order":
            idx[last] = idx[last - 1]
        elif what == "vocab":
            idx[last] = 120
        else:
            val[last] = np.nan
    with pytest.raises(B.ApError) as e:
        B.Index.ingest(B.DeviceVecs(v), B.build_params(8))
    said = str(e.value)
    assert "malformed" in said and (what == "offset" or f" {len(rows)} places" in said)
