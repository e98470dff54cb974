"""Paths of the list-pair and sketch kernels that a corpus reaches only by its size or its skew."""
import numpy as np
import pytest

import oracle
from synth.corpus import Csr, make_corpus, spec_for
from tests.parity import assert_parity
from tests.test_gpu_pairs import PROBE_PAIRS, csr, join
from tests.test_gpu_query_rows import on_device
from tests.test_gpu_query_screen import build

pytestmark = pytest.mark.gpu


def wide_units(entries):
    blocks = -(-entries // 256)
    k = blocks // 16
    return 16 * k * (k + 1) // 2 + (blocks - 16 * k) * (k + 1)


def test_survivors_that_the_sample_missed():
    # every eighth work unit is sampled, and all pairs lie in four units between: 499,500 survivors for a queue of
    # 65,536, decided where they are found
    n, same = 265_000, 1000
    lone = wide_units(n)
    units = lone + wide_units(same) + ((2 * n + same + 31) // 32) // 64
    every = units // 4096
    at = lone % every
    while at == 0 or at + wide_units(same) > every:
        n += 256
        lone = wide_units(n)
        units = lone + wide_units(same) + ((2 * n + same + 31) // 32) // 64
        every = units // 4096
        at = lone % every
    # rows of a dimension that all share, too little for a pair, and one of their own; rows of one dimension
    m = n + 2
    rp = np.concatenate([2 * np.arange(n + 1), 2 * n + 1 + np.arange(same)]).astype(np.int64)
    col = np.concatenate([np.stack([np.zeros(n, np.int64), 2 + np.arange(n)], 1).ravel(), np.ones(same, np.int64)])
    val = np.concatenate([np.tile([0.92, np.sqrt(1 - 0.92 ** 2)], n), np.ones(same)])
    V = Csr(n + same, m, rp, col.astype(np.int32), val.astype(np.float32))
    (i, j, s), st = join(V, np.float32(0.9), pairs=True)
    a, b = np.triu_indices(same, 1)
    assert np.array_equal(i, n + a) and np.array_equal(j, n + b) and np.all(s == 1.0)
    assert st["bound_survivors"] == len(a) > 4 * 65536
    assert st["candidates"] == len(a) + n * (n - 1) // 2


def test_sparse_count_over_several_spans():
    # one bit per corpus row holds 516,096 rows at a time: more rows than that, in lists of one to thousands of entries
    n, head, m = 530_000, 64, 60_000
    rng = np.random.default_rng(11)
    tail = (head + np.minimum((m - head) * rng.random(n) ** 2.5, m - head - 1).astype(np.int64)).astype(np.int32)
    first = rng.integers(0, head - 1, size=n).astype(np.int32)
    second = np.minimum(first + 1 + rng.integers(0, 3, size=n), head - 1).astype(np.int32)
    w = np.stack([rng.uniform(0.3, 0.5, size=n), rng.uniform(0.3, 0.5, size=n), np.full(n, 0.7)], 1)
    w /= np.sqrt((w * w).sum(1, keepdims=True))
    V = Csr(n, m, 3 * np.arange(n + 1, dtype=np.int64), np.stack([first, second, tail], 1).ravel().astype(np.int32),
            w.ravel().astype(np.float32))
    t = np.float32(0.995)
    (a, sa), (b, sb) = join(V, t, pairs=True, screen_dims=head), join(V, t, variant=1)
    assert len(a[0]) > 10_000
    for x, y in zip(a, b):
        assert np.array_equal(np.asarray(x).view(np.uint32), np.asarray(y).view(np.uint32))
    # the head is the densest dimensions: the others' lists are the sparse pass's
    cnt = np.bincount(V.col, minlength=m)
    rank = np.empty(m, np.int64)
    rank[np.lexsort((np.arange(m), -cnt))] = np.arange(m)
    assert np.array_equal(np.sort(rank[:head]), np.arange(head))
    held = np.bincount(tail, minlength=m).astype(np.int64)
    assert held.max() > 5000
    assert sa["candidates"] == int((held * (held - 1) // 2).sum())


def test_several_runs_of_queries():
    # a slot whose queue is smaller than the survivors that its batch has
    import paper_1402_3010_amd as apss
    V = make_corpus(spec_for("c1", n=9000))
    t = np.float32(0.5)
    ix = build(V, t, True)
    try:
        ref = ix.query(V, t=t)
        assert ix.stats()["bound_survivors"] > 2 * 65536 and ix.stats()["posting_visits"] == 0
        with apss.Server(ix, slots=1, pairs_per_query=4, max_batch_queries=9000) as srv:
            for _ in range(2):
                for x, y in zip(srv.poll(srv.submit(V, t=float(t))), ref):
                    assert np.array_equal(x.view(np.uint32), y.view(np.uint32))
    finally:
        ix.close()
    assert_parity(*ref, oracle.query(V, V, t=float(t)), float(t), V, V)


@pytest.mark.parametrize("nq,length", [(1, 30), (40, 30), (3, 5000)])
def test_repeated_dimensions_are_refused(nq, length):
    import paper_1402_3010_amd as apss
    rng = np.random.default_rng(nq)
    V = make_corpus(spec_for("c2", n=3000))
    ix = apss.Index.build(V, np.float32(0.5))
    bad = csr([(rng.choice(V.m, size=length, replace=False), rng.lognormal(0, 1, size=length)) for _ in range(nq)], V.m)
    bad.col[-1] = bad.col[-3]
    try:
        for q in (bad, on_device(bad)):
            with pytest.raises(apss.ApssError) as e:
                ix.query(q, t=np.float32(0.5))
            assert e.value.code == apss.APSS_EINVAL and "repeated dimension" in str(e.value)
    finally:
        ix.close()
