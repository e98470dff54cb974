"""Rows of a million components, with weights whose plain float sum falls short of their product by more than the slack.

A wave adds 64 chains of products, longest first from the rare end; each weight is chosen so that its step of the
chains rounds down by almost half a unit.  The pair's similarity is just over the threshold.
"""
import numpy as np
import pytest

import oracle
from synth.corpus import Csr
from tests.parity import assert_parity
from tests.test_gpu_pairs import PROBE_PAIRS

pytestmark = pytest.mark.gpu


def short_falling_row(length):
    """Weights by position (64 equal ones to a step of the chains), and the plain sum's shortfall."""
    steps = length // 64
    w = np.empty(steps, np.float32)
    s, exact, goal = np.float32(0.0), 0.0, 1.000004 / length
    for k in range(steps):
        # (half a unit past a whole number of them, as many as keep to the goal)
        unit = np.spacing(np.float32(max(float(s) + goal, 1e-30)))
        want = goal * (k + 1) - exact
        p = (np.round(want / unit - 0.499) + 0.499) * unit if float(unit) * 8 < want else want
        w[k] = np.float32(np.sqrt(p))
        p = np.float64(w[k]) ** 2
        s = np.float32(np.float64(s) + p)
        exact += p
    # chains go through chunks of 256 from the last on, four steps in each
    by_position = np.concatenate([w[4 * c:4 * c + 4] for c in range(steps // 4)][::-1])
    return np.repeat(by_position, 64), 64.0 * (exact - float(s))


@pytest.mark.parametrize("length", [1 << 20])
def test_plain_sum_does_not_drop_a_pair(length):
    import paper_1402_3010_amd as apss
    w, short = short_falling_row(length)
    assert short > 2e-4 and 1.0 <= np.sum(w.astype(np.float64) ** 2) <= 1.00001
    V = Csr(2, length, np.array([0, length, 2 * length], np.int64), np.tile(np.arange(length, dtype=np.int32), 2),
            np.concatenate([w, w]))
    t = np.float32(1.0)
    got = []
    for pairs in (True, False):
        o = apss.default_opts(apss.current_stream_handle(), variant=-1 if pairs else 1)
        o.reserved[0] = PROBE_PAIRS if pairs else 0
        ix = apss.Index(apss.build_index(V.n, V.m, V.row_ptr, V.col, V.val, t, o), V.n, V.m)
        try:
            got.append((ix.join(t), ix.query(V, t=t)))
        finally:
            ix.close()
    for a, b in zip(*got):
        for x, y in zip(a, b):
            assert np.array_equal(x.view(np.uint32), y.view(np.uint32))
    assert len(got[0][0][0]) == 1 and len(got[0][1][0]) == 4
    assert_parity(*got[0][0], oracle.join_plain(V, t), float(t), V)
