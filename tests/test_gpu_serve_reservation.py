"""A server's slot holds no more device memory than the largest reservation, also of rows of a few components."""
import numpy as np
import pytest

from synth.corpus import make_corpus, spec_for
from tests.test_gpu_pairs import PROBE_PAIRS, csr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nq,length,pairs_per_query", [(16384, 3, 16), (16384, 5, 16), (4096, 300, 16), (4096, 3, 96),
                                                       (16384, 40, 4), (2000, 5000, 40)])
def test_slot_holds_its_reservation(nq, length, pairs_per_query):
    import paper_1402_3010_amd as apss
    rng = np.random.default_rng(nq + length)
    V = make_corpus(spec_for("c2", n=3000))
    rows = [V.row(int(r)) for r in rng.choice(V.n, size=40, replace=False)]
    for _ in range(100):
        rows.append((np.sort(rng.choice(V.m, size=length, replace=False)), rng.lognormal(0.0, 0.5, size=length)))
    Q = csr([rows[40 + k % 100] for k in range(nq - 40)] + rows[:40], V.m)
    t = np.float32(0.8)
    o = apss.default_opts(apss.current_stream_handle())
    o.reserved[0] = PROBE_PAIRS  # (batches take the sketch kernels where they may)
    ix = apss.Index(apss.build_index(V.n, V.m, V.row_ptr, V.col, V.val, t, o), V.n, V.m)
    try:
        ref = ix.query(Q, t=t)
        assert 40 <= len(ref[0]) <= pairs_per_query * nq
        with apss.Server(ix, slots=1, max_batch_queries=nq, pairs_per_query=pairs_per_query) as srv:
            for _ in range(2):
                got = srv.poll(srv.submit(Q, t=float(t)))
                for x, y in zip(got, ref):
                    assert np.array_equal(x.view(np.uint32), y.view(np.uint32))
            st = srv.stats()
    finally:
        ix.close()
    assert st["regrows"] == 0
    print("slot", st["device_bytes"][0], "reserved", st["peak_reserved_bytes"])
    assert 0 < st["device_bytes"][0] <= st["peak_reserved_bytes"]
