"""Staging of query rows: sorted in LDS up to 4,096 components, by radix passes past that; checks of every row."""
import numpy as np
import pytest

import oracle
from synth.corpus import Csr, make_corpus, spec_for
from tests.parity import assert_parity
from tests.test_gpu_pairs import csr

pytestmark = pytest.mark.gpu


def on_device(Q):
    import torch
    return Csr(Q.n, Q.m, *(torch.from_numpy(x).cuda() for x in (Q.row_ptr, Q.col, Q.val)))


@pytest.mark.parametrize("length,copies", [(1, 3), (2, 40), (255, 3), (256, 30), (257, 70), (1000, 40), (4095, 2),
                                           (4096, 9), (4097, 2)])
def test_shuffled_rows(length, copies):
    # rows in any order of their dimensions; batches below and above the 128 KB that one copy brings
    import paper_1402_3010_amd as apss
    rng = np.random.default_rng(length)
    m = 9000
    c = rng.choice(m, size=length, replace=False)
    w = rng.lognormal(0, 0.5, size=length)
    rows = [(c, w * rng.lognormal(0, 0.05, size=length)) for _ in range(4)]
    rows += [(rng.choice(m, size=20, replace=False), rng.lognormal(0, 1, size=20)) for _ in range(300)]
    V = csr(rows, m)
    qrows = []
    for k in range(copies):
        p = rng.permutation(length)
        qrows.append((c[p], (w * rng.lognormal(0, 0.05, size=length))[p]))
    Q = csr(qrows, m)
    t = np.float32(0.7)
    ix = apss.Index.build(V, t)
    try:
        a = ix.query(Q, t=t)
        b = apss.query(ix.handle, Q.n, *[getattr(on_device(Q), k) for k in ("row_ptr", "col", "val")], float(t))
        for x, y in zip(a, b):
            assert np.array_equal(x.view(np.uint32), np.asarray(y).view(np.uint32))
        assert len(a[0]) >= 4 * copies
        assert_parity(*a, oracle.query(V, Q, t=float(t)), float(t), Q, V)
    finally:
        ix.close()


@pytest.mark.parametrize("nq,length", [(1, 30), (40, 30), (3, 5000)])
def test_refused_rows(nq, length):
    import paper_1402_3010_amd as apss
    rng = np.random.default_rng(nq)
    V = make_corpus(spec_for("c2", n=3000))
    ix = apss.Index.build(V, np.float32(0.5))
    good = csr([(rng.choice(V.m, size=length, replace=False), rng.lognormal(0, 1, size=length)) for _ in range(nq)], V.m)
    ref = ix.query(good, t=np.float32(0.5))
    at = int(good.row_ptr[nq - 1])
    try:
        for what in ("dim", "negative dim", "nan", "inf", "zero", "norm", "repeat"):
            bad = Csr(nq, V.m, good.row_ptr.copy(), good.col.copy(), good.val.copy())
            if what == "dim":
                bad.col[at] = V.m
            elif what == "negative dim":
                bad.col[at] = -1
            elif what == "repeat":
                bad.col[at] = bad.col[at + 1]
            elif what == "norm":
                bad.val[at:] *= np.float32(1.001)
            else:
                bad.val[at] = {"nan": np.nan, "inf": np.inf, "zero": 0.0}[what]
            for q in (bad, on_device(bad)):
                with pytest.raises(apss.ApssError) as e:
                    ix.query(q, t=np.float32(0.5))
                assert e.value.code == apss.APSS_EINVAL and "row %d" % (nq - 1) in str(e.value) or what == "repeat"
        for rp in ([0] * nq + [-1], [1] + [length] * nq, [0, length + 1] + [length] * (nq - 1) if nq > 1 else [2, 1]):
            bad = Csr(nq, V.m, np.array(rp, np.int64), good.col, good.val)
            for q in (bad, on_device(bad)):
                with pytest.raises(apss.ApssError) as e:
                    ix.query(q, t=np.float32(0.5))
                assert e.value.code == apss.APSS_EINVAL
        # and the index answers as before
        for x, y in zip(ref, ix.query(good, t=np.float32(0.5))):
            assert np.array_equal(x.view(np.uint32), y.view(np.uint32))
        assert ix.join(np.float32(0.9)) is not None
    finally:
        ix.close()
