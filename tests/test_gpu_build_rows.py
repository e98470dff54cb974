"""Index building at the edges of its row kernels: a wave, one wave's sort, one workgroup's sort, longer rows."""
import numpy as np
import pytest

import oracle
from synth.corpus import Csr
from tests.parity import assert_parity

pytestmark = pytest.mark.gpu

M = 20_000


def rows_of_lengths(lens, seed):
    rng = np.random.default_rng(seed)
    p = np.arange(1, M + 1, dtype=np.float64) ** -0.7
    p /= p.sum()
    cols, vals = [], []
    for k in lens:
        c = np.sort(rng.choice(M, size=k, replace=False, p=p)) if k else np.zeros(0, np.int64)
        w = rng.lognormal(0.0, 1.0, size=k)
        cols.append(c)
        vals.append(w / np.sqrt((w * w).sum()) if k else w)
    rp = np.zeros(len(lens) + 1, np.int64)
    np.cumsum(lens, out=rp[1:])
    return Csr(len(lens), M, rp, np.concatenate(cols).astype(np.int32), np.concatenate(vals).astype(np.float32))


@pytest.mark.parametrize("longest", [64, 512, 513, 8192, 8193])
@pytest.mark.parametrize("on_device", [False, True])
def test_index_of_rows_at_kernel_edges(longest, on_device):
    import paper_1402_3010_amd as apss
    lens = [0, 1, 2, 3, 31, 63, 64, longest, 5, 0] + [k for k in (65, 127, 128, 129, 511, 512, 513, 1023, 1025) if k < longest]
    V = rows_of_lengths(lens * 3, longest)
    t = np.float32(0.3)
    ix = apss.Index.build(V, t, on_device=on_device)
    try:
        rank, mw, cut = ix.export()
        i, j, s = ix.join(t)
        postings = ix.sizes()["postings"]
    finally:
        ix.close()
    # ranks and cuts are integers of double sums in one order, maxweights are inputs: all equal
    orank, omw, ocut = oracle.prefix_index(V, t)
    assert np.array_equal(rank, orank) and np.array_equal(mw, omw) and np.array_equal(cut, ocut)
    assert postings == V.nnz - int(ocut.sum())
    assert_parity(i, j, s, oracle.join_plain(V, t), float(t), V)


@pytest.mark.parametrize("length", [2, 64, 513, 8193])
def test_repeated_dimension_is_refused_at_every_row_length(length):
    import paper_1402_3010_amd as apss
    V = rows_of_lengths([4, length, 7], 3)
    V.col[V.row_ptr[1] + length - 1] = V.col[V.row_ptr[1]]
    with pytest.raises(apss.ApssError) as e:
        apss.Index.build(V, np.float32(0.5))
    assert e.value.code == apss.APSS_EINVAL
