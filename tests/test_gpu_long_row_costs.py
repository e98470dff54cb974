"""Corpora of long rows over many dimensions keep the accumulating kernel: the list pairs' count and decisions are slower,
in self-joins and in the sparse pass of the screened join."""
import numpy as np
import pytest

from synth.corpus import Csr
from tests.test_gpu_pairs import join

pytestmark = pytest.mark.gpu


def corpus(n, mean, seed=5, m=1_000_000, s=0.9):
    rng = np.random.default_rng(seed)
    cum = np.cumsum(np.arange(1, m + 1, dtype=np.float64) ** -s)
    lens = np.clip(rng.lognormal(np.log(mean) - 0.245, 0.7, size=n).astype(np.int64), 50, 9000)
    cols, vals, rp = [], [], [0]
    for k in lens:
        c = np.unique(np.searchsorted(cum, rng.random(k) * cum[-1]).clip(0, m - 1))
        w = rng.lognormal(0.0, 1.0, size=len(c))
        cols.append(c)
        vals.append(w / np.sqrt((w * w).sum()))
        rp.append(rp[-1] + len(c))
    return Csr(n, m, np.array(rp, np.int64), np.concatenate(cols).astype(np.int32), np.concatenate(vals).astype(np.float32))


@pytest.mark.parametrize("n,mean,t,pairs", [(2000, 1500, 0.8, False), (5000, 1500, 0.8, False), (6000, 120, 0.7, True),
                                            (2000, 120, 0.7, True)])
def test_kernels_of_long_rows(n, mean, t, pairs):
    V = corpus(n, mean)
    (a, sa), (b, sb) = join(V, np.float32(t)), join(V, np.float32(t), variant=1)
    for x, y in zip(a, b):
        assert np.array_equal(x, y)
    assert sa["candidates"] == sb["candidates"]
    assert (sa["posting_visits"] < sb["posting_visits"]) == pairs


@pytest.mark.parametrize("n,mean,t,head,pairs", [(2000, 1500, 0.8, 64, False), (2000, 1500, 0.8, 4096, False),
                                                 (8000, 1500, 0.6, 512, False), (20000, 120, 0.6, 4096, True),
                                                 (20000, 120, 0.5, 512, True)])
def test_kernels_of_the_sparse_pass(n, mean, t, head, pairs):
    V = corpus(n, mean)
    (a, sa), (b, sb), (c, _) = [join(V, np.float32(t), screen_dims=head, pairs=p) for p in (False, True)] + [
        join(V, np.float32(t), variant=1)]
    for x, y, z in zip(a, b, c):
        assert np.array_equal(x, y) and np.array_equal(x, z)
    # (visits of the accumulating kernel are list entries, those of the list pairs fewer pairs)
    assert (sa["posting_visits"] == sb["posting_visits"]) == pairs
