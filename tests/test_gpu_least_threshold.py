"""Thresholds so small that they round to no sketch product: rows without components are still nobody's survivors.

(A survivor's rows are read from their first component on; the last rows here have none.)
"""
import numpy as np
import pytest

from synth.corpus import Csr, make_corpus, spec_for
from tests.test_gpu_query_screen import assert_same

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("t", [1e-9, 6e-8, 1e-4])
def test_empty_rows_at_a_tiny_threshold(t):
    V = make_corpus(spec_for("c1", n=512))
    empty = Csr(V.n + 100, V.m, np.concatenate([V.row_ptr, np.full(100, V.row_ptr[-1])]), V.col, V.val)
    a = assert_same(empty, empty, np.float32(t), t=np.float32(t))
    assert len(a[0]) > 512 and max(a[0]) < V.n and max(a[1]) < V.n
