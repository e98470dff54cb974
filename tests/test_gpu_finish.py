"""Results of few pairs are sorted and handed over by one kernel: the same pairs as a larger result's sort gives.

Copies of one row make any number of them (k rows: k (k - 1) / 2 pairs).
"""
import numpy as np
import pytest

from synth.corpus import make_corpus, spec_for
from tests.test_gpu_pairs import csr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("copies", [1, 2, 11, 12, 91, 181, 182, 300])
def test_self_join_of_copies(copies):
    import torch

    import paper_1402_3010_amd as apss
    base = make_corpus(spec_for("c1", n=500))
    rng = np.random.default_rng(copies)
    rows = [base.row(k) for k in range(1, 200)] + [base.row(0)] * copies
    order = rng.permutation(len(rows))
    V = csr([rows[k] for k in order], base.m)
    at = np.sort(np.flatnonzero(order >= 199))
    want = [(int(i), int(j)) for x, i in enumerate(at) for j in at[x + 1:]]
    ix = apss.Index.build(V, np.float32(0.95), stream=torch.cuda.current_stream().cuda_stream)
    try:
        i, j, s = ix.join(np.float32(0.95))
        pairs = list(zip(i.tolist(), j.tolist()))
        assert pairs == sorted(set(pairs)) and set(want) <= set(pairs)
        n = len(i)
        for call in (ix.join_device, ix.join_device_noalloc):
            out = [torch.full((n + 5,), -1, dtype=d, device="cuda") for d in (torch.int32, torch.int32, torch.float32)]
            assert call(np.float32(0.95), *out) == n
            for o, p in zip(out, (i, j, s)):
                assert np.array_equal(o[:n].cpu().numpy().view(np.uint32), p.view(np.uint32))
                assert bool((o[n:] == -1).all())
            if n:  # no room: refused, and nothing written
                small = [o[:n - 1].fill_(-1) for o in out]
                with pytest.raises(apss.ApssError) as e:
                    call(np.float32(0.95), *small)
                assert e.value.code == apss.APSS_ERANGE
                assert all(bool((o == -1).all()) for o in small)
    finally:
        ix.close()


@pytest.mark.parametrize("copies", [50, 182])
def test_graph_replays(copies):
    import torch

    import paper_1402_3010_amd as apss
    base = make_corpus(spec_for("c1", n=300))
    V = csr([base.row(k % 200) if k >= copies else base.row(0) for k in range(copies + 200)], base.m)
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    ref = None
    ix = apss.Index.build(V, np.float32(0.9), stream=stream.cuda_stream, graph=True)
    try:
        ref = ix.join(np.float32(0.9))
        out = [torch.zeros(len(ref[0]), dtype=d, device="cuda") for d in (torch.int32, torch.int32, torch.float32)]
        for _ in range(4):
            for o in out:
                o.zero_()
            torch.cuda.synchronize()
            assert ix.join_device(np.float32(0.9), *out) == len(ref[0])
            for o, p in zip(out, ref):
                assert np.array_equal(o.cpu().numpy().view(np.uint32), p.view(np.uint32))
    finally:
        ix.close()
