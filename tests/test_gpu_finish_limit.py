"""The one-launch end of a call at its limit of 32,768 pairs, with keys of more and of fewer than 32 bits."""
import numpy as np
import pytest

from synth.corpus import make_corpus, spec_for
from tests.test_gpu_pairs import csr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("copies", [255, 256, 257])  # 32,385, 32,640 and 32,896 pairs
@pytest.mark.parametrize("others", [100, 70000])     # 18 and 34 key bits
def test_pairs_at_the_limit(copies, others):
    import paper_1402_3010_amd as apss
    base = make_corpus(spec_for("c1", n=200))
    rng = np.random.default_rng(copies + others)
    # (single dimensions, three rows to each, so that the rest has pairs too)
    rows = [base.row(0)] * copies + [(np.array([k // 3 % base.m], np.int32), np.ones(1)) for k in range(others)]
    order = rng.permutation(len(rows))
    V = csr([rows[k] for k in order], base.m)
    ix = apss.Index.build(V, np.float32(0.95))
    try:
        i, j, s = ix.join(np.float32(0.95))
    finally:
        ix.close()
    group = np.where(order < copies, -1, (order - copies) // 3 % base.m)
    want = set()
    for g in np.unique(group):
        at = np.flatnonzero(group == g)
        want.update((int(a), int(b)) for x, a in enumerate(at) for b in at[x + 1:])
    pairs = list(zip(i.tolist(), j.tolist()))
    assert pairs == sorted(pairs) and set(pairs) == want and len(pairs) == len(want)
    assert np.all(np.abs(s - 1.0) <= 1e-5)
