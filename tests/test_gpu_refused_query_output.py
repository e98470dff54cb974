"""A refused batch of queries leaves the caller's device buffers as they were."""
import numpy as np
import pytest

from synth.corpus import Csr, make_corpus, spec_for
from tests.test_gpu_query_rows import on_device
from tests.test_gpu_pairs import PROBE_PAIRS

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nq", [2, 40])
def test_nothing_is_written(nq):
    # all rows but the last are copies of corpus rows, which have pairs
    import torch

    import paper_1402_3010_amd as apss
    V = make_corpus(spec_for("c1", n=3000))
    for probe, variant in ((0, -1), (PROBE_PAIRS, -1), (0, 1)):
        o = apss.default_opts(apss.current_stream_handle(), variant=variant)
        o.reserved[0] = probe
        ix = apss.Index(apss.build_index(V.n, V.m, V.row_ptr, V.col, V.val, np.float32(0.5), o), V.n, V.m)
        try:
            Q = V.take_rows(np.arange(nq))
            bad = Csr(nq, V.m, Q.row_ptr, Q.col.copy(), Q.val.copy())
            bad.val[-1] = np.nan
            out = [torch.full((4096,), -1, dtype=d, device="cuda") for d in (torch.int32, torch.int32, torch.float32)]
            assert ix.query_device(Q, *out, t=np.float32(0.5)) >= nq
            for q in (bad, on_device(bad)):
                for x in out:
                    x.fill_(-1)
                with pytest.raises(apss.ApssError) as e:
                    ix.query_device(q, *out, t=np.float32(0.5))
                assert e.value.code == apss.APSS_EINVAL and "row %d" % (nq - 1) in str(e.value)
                assert all(bool((x == -1).all()) for x in out)
        finally:
            ix.close()
