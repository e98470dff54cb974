"""Memory that ended indexes leave to the next ones: bounded, reused, from several threads, with the same results."""
import threading

import numpy as np
import pytest

from synth.corpus import make_corpus, spec_for

pytestmark = pytest.mark.gpu


def test_indexes_of_many_sizes_in_turn():
    # each reuses what others of other sizes left, and answers as the first of its size did
    import torch

    import paper_1402_3010_amd as apss
    rng = np.random.default_rng(5)
    seen = {}
    free0, total = torch.cuda.mem_get_info()
    for k in rng.integers(0, 6, size=40):
        n = [1, 40, 700, 5000, 20000, 60000][k]
        V = make_corpus(spec_for("c2", n=n))
        ix = apss.Index.build(V, np.float32(0.6))
        try:
            out = [np.asarray(x) for x in ix.join(np.float32(0.6))]
            out += [np.asarray(x) for x in ix.query(V.take_rows(np.arange(min(n, 40))), t=np.float32(0.7))]
            out += [np.asarray(x) for x in ix.export()]
        finally:
            ix.close()
        for a, b in zip(seen.setdefault(n, out), out):
            assert np.array_equal(a.view(np.uint32), b.view(np.uint32))
    assert free0 - torch.cuda.mem_get_info()[0] <= total // 32 + (256 << 20)


def test_threads_build_and_close():
    import torch

    import paper_1402_3010_amd as apss
    corpora = [make_corpus(spec_for("c2", n=n)) for n in (3000, 3100, 9000)]
    ref, bad = [], []
    for V in corpora:
        ix = apss.Index.build(V, np.float32(0.6))
        ref.append(ix.join(np.float32(0.6)))
        ix.close()

    def work(w):
        stream = torch.cuda.Stream()
        for k in range(8):
            V, want = corpora[(w + k) % 3], ref[(w + k) % 3]
            ix = apss.Index.build(V, np.float32(0.6), stream=stream.cuda_stream)
            got = ix.join(np.float32(0.6))
            ix.close()
            if not all(np.array_equal(a.view(np.uint32), b.view(np.uint32)) for a, b in zip(got, want)):
                bad.append((w, k))

    th = [threading.Thread(target=work, args=(w,)) for w in range(4)]
    for x in th:
        x.start()
    for x in th:
        x.join()
    assert not bad
