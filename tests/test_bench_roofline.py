"""The benchmark's roofline names the kernels that ran and reports only counters taken on them (CPU)."""
import argparse
import json
import os

import pytest

from tests.test_bench_host import ROOT, bench  # noqa: F401 (fixture)


def test_unit_that_binds(bench):  # noqa: F811
    with open(os.path.join(ROOT, "profiles", "list_pairs_c3_counters.json")) as fh:
        rec = json.load(fh)
    full, part = argparse.Namespace(config="c3", n=None), argparse.Namespace(config="c3", n=300000)
    pairs = dict(matches=21_614_295, posting_visits=17_174_720_604, candidates=304_336_462_582)
    lists = dict(matches=21_614_295, posting_visits=1_400_000_000_000, candidates=304_336_462_582)
    r = bench.roofline_of(full, rec["t"], 119_932_728, pairs, 290.0)
    if rec["source_hash"] == bench.pair_source_hash():
        assert r["bound"] == "l1 address units" and r["frac"] == pytest.approx(rec["l1_accesses"] / 0.29 / 614.4e9)
        assert r["frac_dram"] == pytest.approx(rec["traffic_bytes"] / 0.29 / 8e12) and 0 < r["frac"] < 1
        assert r["issue"]["ta_busy_frac"] == rec["ta_busy_frac"] and "k_count" in r["binding_unit"]
    else:
        assert r["bound"] == "hbm" and r["traffic"] is None and r["binding_unit"] is None
    assert r["pairs_tested"] == pairs["posting_visits"] and "k_count" in r["kernel"]
    assert r["counters_source"] == "profiles/list_pairs_c3_counters.md"
    # other sizes and thresholds, and the accumulating kernel, have none of these counters
    for args, t, st in ((part, rec["t"], pairs), (full, rec["t"] + 0.1, pairs), (full, rec["t"], lists)):
        r = bench.roofline_of(args, t, 119_932_728, st, 290.0)
        assert r["bound"] == "hbm" and r["frac"] == pytest.approx(r["algorithmic_bytes"] / 0.29 / 8e12)
    assert r["kernel"] == "k_join" and r["pairs_tested"] is None
