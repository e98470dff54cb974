"""Queries by the sketch kernels against the accumulating kernel and the oracle, at the edges of tiles and rows.

Both report the shared rescore of the same pairs, so their outputs are equal bit for bit, and both count the
candidates of the paper's index.
"""
import numpy as np
import pytest

import oracle
from synth.corpus import Csr, make_corpus, spec_for
from tests.parity import assert_parity
from tests.test_gpu_pairs import PROBE_PAIRS, csr

pytestmark = pytest.mark.gpu


def build(V, t, probe):
    import paper_1402_3010_amd as apss
    o = apss.default_opts(apss.current_stream_handle(), variant=-1 if probe else 1)
    o.reserved[0] = PROBE_PAIRS if probe else 0
    return apss.Index(apss.build_index(V.n, V.m, V.row_ptr, V.col, V.val, t, o), V.n, V.m)


def assert_same(V, Q, t_build, **kw):
    out = []
    for probe in (True, False):
        ix = build(V, t_build, probe)
        try:
            out.append((ix.query(Q, **kw), ix.stats()))
        finally:
            ix.close()
    (a, sa), (b, sb) = out
    for x, y in zip(a, b):
        assert np.array_equal(x.view(np.uint32), y.view(np.uint32))
    assert sa["candidates"] == sb["candidates"] and sa["matches"] == sb["matches"]
    assert sa["posting_visits"] == 0 < sb["posting_visits"]
    return a


def query_rows(V, nq, rng, extra=()):
    """Perturbed corpus rows, random rows, and `extra`; some over dimensions that the corpus lacks."""
    rows = list(extra)
    while len(rows) < nq:
        r = int(rng.integers(0, V.n))
        c, w = V.row(r)
        if rng.random() < 0.5 and len(c):
            rows.append((c, w * rng.lognormal(0.0, 0.15, size=len(c))))
        else:
            k = int(rng.integers(1, 80))
            rows.append((np.sort(rng.choice(V.m, size=k, replace=False)).astype(np.int32), rng.lognormal(0, 1, size=k)))
    return csr(rows[:nq], V.m)


@pytest.mark.parametrize("nq", [2, 31, 32, 33, 63, 64, 65, 257])
@pytest.mark.parametrize("n", [63, 65, 256, 4097])
def test_tile_edges(n, nq):
    rng = np.random.default_rng(1000 * n + nq)
    V = make_corpus(spec_for("c2", n=n))
    Q = query_rows(V, nq, rng)
    tq = rng.uniform(0.5, 0.95, size=nq).astype(np.float32)
    a = assert_same(V, Q, np.float32(0.5), t_per_row=tq)
    assert_parity(*a, oracle.query(V, Q, t_per_row=tq.astype(np.float64)), None, Q, V, per_row_t=tq.astype(np.float64))


@pytest.mark.parametrize("length", [256, 257, 1025, 3000])
def test_long_rows(length):
    rng = np.random.default_rng(length)
    m, rows = 6000, []
    for _ in range(4):
        c = np.sort(rng.choice(m, size=length, replace=False))
        w = rng.lognormal(0.0, 0.7, size=length)
        rows += [(c, w * rng.lognormal(0.0, rng.uniform(0.05, 0.5), size=length)) for _ in range(8)]
    rows += [(np.sort(rng.choice(m, size=30, replace=False)), rng.lognormal(0, 1, size=30)) for _ in range(400)]
    V = csr(rows, m)
    Q = query_rows(V, 70, rng, [rows[k] for k in range(0, 32, 3)])
    t = np.float32(0.75)
    a = assert_same(V, Q, t, t=t)
    assert len(a[0]) >= 40
    assert_parity(*a, oracle.query(V, Q, t=float(t)), float(t), Q, V)


def test_empty_rows_and_whole_corpus():
    # rows without components among the queries, the corpus against itself, and more pairs than the first buffers hold
    V = make_corpus(spec_for("c1", n=1200))
    rp = np.concatenate([[0, 0], V.row_ptr[1:], [V.row_ptr[-1]] * 2]).astype(np.int64)
    Q = Csr(len(rp) - 1, V.m, rp, V.col, V.val)
    t = np.float32(0.5)
    a = assert_same(V, Q, t, t=t)
    assert set(range(V.n)) <= {int(i) - 1 for i, j in zip(a[0], a[1]) if int(i) - 1 == int(j)}
    same = csr([V.row(0)] * 300, V.m)
    b = assert_same(same, csr([V.row(0)] * 300, V.m), t, t=t)
    assert len(b[0]) == 300 * 300


def test_host_device_and_server_agree():
    import torch

    import paper_1402_3010_amd as apss
    rng = np.random.default_rng(3)
    V = make_corpus(spec_for("c2", n=9000))
    Q = query_rows(V, 130, rng)
    t = np.float32(0.6)
    ix = build(V, np.float32(0.5), True)
    try:
        ref = ix.query(Q, t=t)
        out = [torch.zeros(len(ref[0]) + 8, dtype=d, device="cuda") for d in (torch.int32, torch.int32, torch.float32)]
        D = Csr(Q.n, Q.m, *(torch.from_numpy(x).cuda() for x in (Q.row_ptr, Q.col, Q.val)))
        cnt = ix.query_device(D, *out, t=t)
        assert cnt == len(ref[0])
        for x, y in zip(out, ref):
            assert np.array_equal(x[:cnt].cpu().numpy().view(np.uint32), y.view(np.uint32))
        with apss.Server(ix, slots=2, pairs_per_query=1) as srv:
            ids = [srv.submit(Q, t=float(t)) for _ in range(6)]
            for r in ids:
                got = srv.poll(r)
                for x, y in zip(got, ref):
                    assert np.array_equal(x.view(np.uint32), y.view(np.uint32))
    finally:
        ix.close()


def test_more_survivors_than_expected():
    # copies of one row are few pairs of the corpus's and all of the queries': the survivor queue overflows and the
    # accumulating kernel answers
    base = make_corpus(spec_for("c1", n=15000))
    hot = base.row(7)
    V = csr([base.row(k) for k in range(base.n)] + [hot] * 1000, base.m)
    Q = csr([hot] * 150 + [base.row(k) for k in range(10)], base.m)
    t = np.float32(0.9)
    (a, sa), (b, sb) = [(ix.query(Q, t=t), ix.stats()) for ix in (build(V, t, True), build(V, t, False))]
    for x, y in zip(a, b):
        assert np.array_equal(x.view(np.uint32), y.view(np.uint32))
    assert len(a[0]) >= 150 * 1001
    assert sa["candidates"] == sb["candidates"] and sa["posting_visits"] == sb["posting_visits"]


def test_queue_filled_in_turns():
    # a slot's queue holds fewer survivors than its batch has: runs of queries take turns
    import paper_1402_3010_amd as apss
    V = make_corpus(spec_for("c1", n=6000))
    t = np.float32(0.5)
    ix = build(V, t, True)
    try:
        ref = ix.query(V, t=t)
        with apss.Server(ix, slots=1, pairs_per_query=64, max_batch_queries=8192) as srv:
            got = srv.poll(srv.submit(V, t=float(t)))
    finally:
        ix.close()
    for x, y in zip(got, ref):
        assert np.array_equal(x.view(np.uint32), y.view(np.uint32))
