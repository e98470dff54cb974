"""The few-query kernel against the join kernel and the oracle, at the edges of its row spans and query lengths."""
import numpy as np
import pytest

import oracle
from synth.corpus import Csr, make_corpus, spec_for
from tests.parity import assert_parity
from tests.test_gpu_pairs import csr
from tests.test_gpu_query_screen import query_rows

pytestmark = pytest.mark.gpu


def assert_same(V, Q, t_build, **kw):
    import paper_1402_3010_amd as apss
    got = []
    for opts in ({}, {"variant": 1}):
        ix = apss.Index.build(V, t_build, **opts)
        try:
            got.append((ix.query(Q, **kw), ix.stats()))
        finally:
            ix.close()
    (a, sa), (b, sb) = got
    for x, y in zip(a, b):
        assert np.array_equal(x.view(np.uint32), y.view(np.uint32))
    for k in ("candidates", "matches", "posting_visits"):
        assert sa[k] == sb[k]
    return a


@pytest.mark.parametrize("nq", [1, 2, 16])
@pytest.mark.parametrize("n", [1, 2047, 2048, 2049, 16385, 40001])
def test_row_spans(n, nq):
    rng = np.random.default_rng(n + nq)
    V = make_corpus(spec_for("c2", n=n))
    Q = query_rows(V, nq, rng, [V.row(n - 1)])
    tq = rng.uniform(0.5, 0.95, size=nq).astype(np.float32)
    a = assert_same(V, Q, np.float32(0.5), t_per_row=tq)
    assert n - 1 in a[1]
    assert_parity(*a, oracle.query(V, Q, t_per_row=tq.astype(np.float64)), None, Q, V, per_row_t=tq.astype(np.float64))


@pytest.mark.parametrize("length", [1, 511, 512, 513, 1024, 1025, 3000])
def test_query_lengths(length):
    # more dense dimensions than the 32,768 with block offsets, so that both kinds of lists are met
    rng = np.random.default_rng(length)
    m, rows = 90000, []
    c = np.sort(rng.choice(m, size=length, replace=False))
    w = rng.lognormal(0.0, 0.7, size=length)
    rows += [(c, w * rng.lognormal(0.0, 0.1 * k, size=length)) for k in range(6)]
    rows += [(np.sort(rng.choice(m, size=60, replace=False)), rng.lognormal(0, 1, size=60)) for _ in range(5000)]
    V = csr(rows, m)
    Q = csr([rows[0], rows[100], rows[3]], m)
    t = np.float32(0.6)
    a = assert_same(V, Q, t, t=t)
    assert len(a[0]) >= 6
    assert_parity(*a, oracle.query(V, Q, t=float(t)), float(t), Q, V)


def test_empty_queries_and_all_rows_alike():
    V = csr([make_corpus(spec_for("c1", n=1)).row(0)] * 5000, spec_for("c1", n=1).m)
    Q = Csr(3, V.m, np.array([0, 0, V.row_ptr[1], V.row_ptr[1]], np.int64), V.col[:V.row_ptr[1]], V.val[:V.row_ptr[1]])
    a = assert_same(V, Q, np.float32(0.9), t=np.float32(1.0))
    assert a[0].tolist() == [1] * 5000 and a[1].tolist() == list(range(5000))
