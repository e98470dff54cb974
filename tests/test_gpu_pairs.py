"""The list-pair self-join against the accumulating one and the oracle, at the edges of its lists and rows.

Both report the shared rescore of the same pairs, so their outputs are equal bit for bit, and both count the
candidates of the paper's index.  An index built with an explicit tile variant takes the accumulating kernel; a
reserved option makes one that takes the list-pair kernels whatever their cost rule says.
"""
import numpy as np
import pytest

import oracle
from synth.corpus import Csr, make_corpus, spec_for
from tests.parity import assert_parity

pytestmark = pytest.mark.gpu


PROBE_PAIRS = 0x50414952


def join(V, t, pairs=False, **kw):
    import paper_1402_3010_amd as apss
    o = apss.default_opts(apss.current_stream_handle(), **kw)
    o.reserved[0] = PROBE_PAIRS if pairs else 0
    ix = apss.Index(apss.build_index(V.n, V.m, V.row_ptr, V.col, V.val, t, o), V.n, V.m)
    try:
        out = ix.join(t)
        st = ix.stats()
    finally:
        ix.close()
    return out, st


def assert_same(V, t):
    (a, sa), (b, sb) = join(V, t, pairs=True), join(V, t, variant=1)
    for x, y in zip(a, b):
        assert np.array_equal(np.asarray(x).view(np.uint32), np.asarray(y).view(np.uint32))
    assert sa["candidates"] == sb["candidates"] and sa["matches"] == sb["matches"]
    # the list-pair kernels ran: they meet fewer list entries
    assert sa["posting_visits"] < sb["posting_visits"]
    return a


def csr(rows, m):
    lens = [len(c) for c, _ in rows]
    rp = np.zeros(len(rows) + 1, np.int64)
    np.cumsum(lens, out=rp[1:])
    val = np.concatenate([w / np.sqrt((w * w).sum()) for _, w in rows]).astype(np.float32)
    return Csr(len(rows), m, rp, np.concatenate([c for c, _ in rows]).astype(np.int32), val)


@pytest.mark.parametrize("lens", [(2, 31, 32, 33, 63, 64, 65, 127, 128, 129), (255, 256, 257, 511, 512, 513, 769),
                                  (4095, 4096, 4097, 4353)])
def test_list_lengths(lens):
    # a list of exactly each length: rows that share one dimension of varying weight (and a tail of common
    # dimensions), in shuffled order
    rng = np.random.default_rng(len(lens))
    m, rows = 3000, []
    for g, k in enumerate(lens):
        for _ in range(k):
            c = rng.choice(m - 100, size=12, replace=False) + 100
            w = rng.lognormal(0.0, 1.0, size=12)
            w *= 1.0 / np.sqrt((w * w).sum())
            h = rng.uniform(0.4, 2.0)
            rows.append((np.concatenate([[g], np.sort(c)]), np.concatenate([[h], w])))
    rng.shuffle(rows)
    V = csr(rows, m)
    t = np.float32(0.8)
    a = assert_same(V, t)
    assert len(a[0]) > 0
    assert_parity(*a, oracle.join_plain(V, t), float(t), V)


@pytest.mark.parametrize("length", [128, 129, 256, 257, 512, 1024, 1025, 2048, 2049, 5000])
def test_row_lengths(length):
    # perturbed copies of long rows among short ones: both rows of a pair staged whole, by ranks, or not at all
    rng = np.random.default_rng(length)
    m, rows = 8000, []
    for _ in range(6):
        c = np.sort(rng.choice(m, size=length, replace=False))
        w = rng.lognormal(0.0, 0.7, size=length)
        for _ in range(7):
            rows.append((c, w * rng.lognormal(0.0, rng.uniform(0.05, 0.5), size=length)))
    for _ in range(300):
        k = int(rng.integers(2, 40))
        rows.append((np.sort(rng.choice(m, size=k, replace=False)), rng.lognormal(0.0, 1.0, size=k)))
    rng.shuffle(rows)
    V = csr(rows, m)
    t = np.float32(0.75)
    a = assert_same(V, t)
    assert len(a[0]) >= 6 * 10
    assert_parity(*a, oracle.join_plain(V, t), float(t), V)


@pytest.mark.parametrize("name,n,t", [("c1", 2000, 0.5), ("c2", 4097, 0.6), ("c2", 30011, 0.5), ("c3", 20000, 0.7),
                                      ("c4", 12000, 0.8)])
def test_workload_shapes(name, n, t):
    assert_same(make_corpus(spec_for(name, n=n)), np.float32(t))


def test_above_the_build_threshold():
    import paper_1402_3010_amd as apss
    V = make_corpus(spec_for("c2", n=9000))
    a, b = apss.Index.build(V, np.float32(0.5)), apss.Index.build(V, np.float32(0.5), variant=1)
    try:
        for t in (0.5, 0.65, 0.9, 1.0):
            x, y = a.join(np.float32(t)), b.join(np.float32(t))
            assert all(np.array_equal(p, q) for p, q in zip(x, y))
            assert a.stats()["candidates"] == b.stats()["candidates"]
    finally:
        a.close()
        b.close()


def test_more_survivors_than_the_queue_holds():
    # the allocation-free call queues 2M survivors: what does not fit is decided where it is found
    import torch

    import paper_1402_3010_amd as apss
    V = make_corpus(spec_for("c2", n=40000))
    t = np.float32(0.5)
    ref, st = join(V, t)
    assert st["bound_survivors"] > 0
    ix = apss.Index.build(V, t)
    try:
        out = [torch.zeros(len(ref[0]) + 10, dtype=d, device="cuda") for d in (torch.int32, torch.int32, torch.float32)]
        for _ in range(2):
            cnt = ix.join_device_noalloc(t, *out)
            assert cnt == len(ref[0]) and ix.stats()["candidates"] == st["candidates"]
            assert ix.stats()["verified"] == st["verified"]
            for x, y in zip(out, ref):
                assert np.array_equal(x[:cnt].cpu().numpy().view(np.uint32), np.asarray(y).view(np.uint32))
    finally:
        ix.close()


def test_flat_rows_over_few_dimensions_keep_the_accumulating_kernel():
    # equal weights over 60 dimensions: no sketch tells these rows apart
    rng = np.random.default_rng(7)
    rows = [(np.sort(rng.choice(60, size=45, replace=False)), np.ones(45)) for _ in range(6000)]
    V = csr(rows, 60)
    t = np.float32(0.85)
    (a, sa), (b, sb) = join(V, t), join(V, t, variant=1)
    assert all(np.array_equal(x, y) for x, y in zip(a, b))
    assert sa["candidates"] == sb["candidates"] and sa["posting_visits"] == sb["posting_visits"]


@pytest.mark.parametrize("n,head", [(3000, 64), (20000, 256), (30001, 4096)])
def test_sparse_pass_of_the_screened_join(n, head):
    # pairs that share a dimension past the head, by list pairs and by the accumulating kernel: same pairs, and the
    # same count of pairs that share one
    V = make_corpus(spec_for("c4", n=n))
    t = np.float32(0.6)
    (a, sa), (b, sb) = join(V, t, pairs=True, screen_dims=head), join(V, t, variant=1)
    for x, y in zip(a, b):
        assert np.array_equal(np.asarray(x).view(np.uint32), np.asarray(y).view(np.uint32))
    rank, _, _ = oracle.prefix_index(V, t)
    import scipy.sparse as sp
    tail = rank[V.col] >= head
    row = np.repeat(np.arange(V.n), np.diff(V.row_ptr))[tail]
    A = sp.csr_matrix((np.ones(len(row), np.int32), (row, V.col[tail])), shape=(V.n, V.m))
    shared = (A @ A.T).tocsr()
    assert sa["candidates"] == (shared.nnz - np.count_nonzero(shared.diagonal())) // 2


@pytest.mark.parametrize("lens", [(2,) * 40, (32, 33, 31), (3, 5, 30, 2, 2, 32, 34), (33, 2, 33, 2, 64, 1, 1, 32)])
def test_tiny_lists_share_tiles(lens):
    # lists of exactly these lengths one after another (each of rows with a dimension of their own), from every offset
    for lead in (0, 1, 17, 31):
        rng = np.random.default_rng(len(lens) + lead)
        m, rows = 2000, []
        for g, k in enumerate((lead,) + lens):
            w = rng.uniform(0.9, 1.1, size=8)
            rows += [(np.concatenate([[g], np.sort(rng.choice(900, size=7, replace=False)) + 1000]),
                      np.concatenate([[4.0], w[1:]])) for _ in range(k)]
        rng.shuffle(rows)
        V = csr(rows, m)
        t = np.float32(0.7)
        (a, sa), (b, sb) = join(V, t, pairs=True), join(V, t, variant=1)
        for x, y in zip(a, b):
            assert np.array_equal(np.asarray(x).view(np.uint32), np.asarray(y).view(np.uint32))
        assert sa["candidates"] == sb["candidates"]
        assert_parity(*a, oracle.join_plain(V, t), float(t), V)


@pytest.mark.parametrize("n", [3001, 5000])
def test_replays_of_a_captured_join(n):
    # pairs and counters of every replay are the eager call's
    import torch

    import paper_1402_3010_amd as apss
    V = make_corpus(spec_for("c2", n=n))
    t = np.float32(0.6)
    ref, st = join(V, t)
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    ix = apss.Index.build(V, t, stream=stream.cuda_stream, graph=True)
    try:
        out = [torch.zeros(len(ref[0]) + 3, dtype=d, device="cuda") for d in (torch.int32, torch.int32, torch.float32)]
        for k in range(5):
            for o in out:
                o.zero_()
            torch.cuda.synchronize()
            assert ix.join_device(t, *out) == len(ref[0])
            for x, y in zip(out, ref):
                assert np.array_equal(x[:len(y)].cpu().numpy().view(np.uint32), np.asarray(y).view(np.uint32))
            now = ix.stats()
            for key in ("candidates", "bound_survivors", "verified", "band", "matches", "posting_visits"):
                assert now[key] == st[key], key
    finally:
        ix.close()


@pytest.mark.parametrize("lens", [(1, 63, 64, 65, 128, 129), (1,) * 15 + (1100,), (1500, 2, 64, 700), (64,) * 33])
def test_count_of_few_rows_by_pieces(lens):
    # rows around multiples of 64 components, long ones among short, and workgroups of fewer than 16 rows
    rng = np.random.default_rng(sum(lens))
    m, n = 2000, 2 * 4096 + 17
    rows = []
    for k in range(n):
        c = np.sort(rng.choice(m, size=min(lens[k % len(lens)] if k % 97 < 33 else 5, m), replace=False))
        rows.append((c, rng.lognormal(0.0, 1.0, size=len(c))))
    V = csr(rows, m)
    t = np.float32(0.8)
    (a, sa), (b, sb) = join(V, t, pairs=True), join(V, t, variant=1)
    assert all(np.array_equal(np.asarray(x).view(np.uint32), np.asarray(y).view(np.uint32)) for x, y in zip(a, b))
    assert sa["candidates"] == sb["candidates"]
