"""Pairs that the allocation-free call holds: as many by list pairs as by the accumulating kernel."""
import numpy as np
import pytest

from synth.corpus import make_corpus, spec_for
from tests.test_gpu_pairs import PROBE_PAIRS, csr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("copies", [2900, 3170])  # 4.20 and 5.02 million pairs of equal rows
def test_pairs_near_the_scratch_limit(copies):
    import torch

    import paper_1402_3010_amd as apss
    base = make_corpus(spec_for("c1", n=2000))
    rng = np.random.default_rng(copies)
    rows = [base.row(k) for k in range(1, 2000)] + [base.row(0)] * copies
    order = rng.permutation(len(rows))
    V = csr([rows[k] for k in order], base.m)
    t = np.float32(0.9)
    got = []
    for pairs in (True, False):
        o = apss.default_opts(apss.current_stream_handle(), variant=-1 if pairs else 1)
        o.reserved[0] = PROBE_PAIRS if pairs else 0
        ix = apss.Index(apss.build_index(V.n, V.m, V.row_ptr, V.col, V.val, t, o), V.n, V.m)
        try:
            out = [torch.zeros(5_100_000, dtype=d, device="cuda") for d in (torch.int32, torch.int32, torch.float32)]
            cnt = ix.join_device_noalloc(t, *out)
            got.append((cnt, out, ix.stats()))
            with pytest.raises(apss.ApssError) as e:  # a smaller buffer: its size is asked for, whatever fits beside it
                ix.join_device_noalloc(t, *[x[:cnt - 1] for x in out])
            assert e.value.code == apss.APSS_ERANGE and e.value.count == cnt
        finally:
            ix.close()
    (ca, a, sa), (cb, b, sb) = got
    assert ca == cb >= copies * (copies - 1) // 2
    assert sa["candidates"] == sb["candidates"] and sa["verified"] == sb["verified"]
    assert sa["posting_visits"] < sb["posting_visits"]  # (the list-pair kernels ran)
    for x, y in zip(a, b):
        assert torch.equal(x.view(torch.int32), y.view(torch.int32))


def test_more_survivors_than_the_queue_in_turns():
    # the queue is filled and decided several times; one that is not was 5 times slower than the accumulating kernel
    import torch

    import paper_1402_3010_amd as apss
    V = make_corpus(spec_for("c2", n=60000))
    t = np.float32(0.5)
    got = []
    for pairs in (True, False):
        o = apss.default_opts(apss.current_stream_handle(), variant=-1 if pairs else 1)
        o.reserved[0] = PROBE_PAIRS if pairs else 0
        ix = apss.Index(apss.build_index(V.n, V.m, V.row_ptr, V.col, V.val, t, o), V.n, V.m)
        try:
            # (room for five million pairs: the queue is what is left beside them)
            out = [torch.zeros(5_000_000, dtype=d, device="cuda") for d in (torch.int32, torch.int32, torch.float32)]
            ms = []
            for _ in range(3):
                cnt = ix.join_device_noalloc(t, *out)
                ms.append(ix.stats()["ms_candidates"])
            got.append((cnt, out, ix.stats(), min(ms)))
        finally:
            ix.close()
    (ca, a, sa, ma), (cb, b, sb, mb) = got
    assert ca == cb and sa["candidates"] == sb["candidates"]
    for x, y in zip(a, b):
        assert torch.equal(x.view(torch.int32), y.view(torch.int32))
    assert ma < 2 * mb
