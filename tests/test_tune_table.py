"""The committed schedule table is what the autotuner's rules make of the
measurements recorded with it."""
import json
import os

import pytest

from paper_2506_17357_amd import autotune

TABLE = os.path.join(os.path.dirname(autotune.__file__), "tune_table.json")


@pytest.fixture(scope="module")
def table():
    with open(TABLE) as f:
        return json.load(f)


def test_entries_follow_the_measurements(table):
    bounds = dict(zip(autotune.BUCKETS, autotune.bucket_bounds(autotune.BUCKETS)))
    entries = {(e["kind"], e["n_max"]): e for e in table["entries"]}
    groups = [m for m in table["measurements"] if "mix" not in m]
    mix, = [m["mix"] for m in table["measurements"] if "mix" in m]
    mix_rows = {(g.split("/")[0], int(g.split("/")[1])): r for g, r in mix["rows"].items()}
    assert len(groups) == len(entries) == 2 * len(autotune.BUCKETS)
    for m in groups:
        e = entries[m["kind"], bounds[m["n"]]]
        plain = {int(k): v for k, v in m["plain_us_per_step"].items()}
        assert plain[e["plain_rows"]] == min(plain.values()), m["n"]  # (recorded to a tenth of a microsecond)
        times = {int(k): v for k, v in m["batched_us_per_eval_launch"].items()}
        assert e["item_rows"] == autotune.choose_item_rows(m["kind"], m["n"], times, mix_rows, 0.03), (m["kind"], m["n"])


def test_item_rows_rule():
    times = {0: 100.0, 16: 98.0, 32: 90.0}
    assert autotune.choose_item_rows("cvrp", 500, times, None, 0.03) == 32
    assert autotune.choose_item_rows("cvrp", 500, {0: 100.0, 32: 98.0}, None, 0.03) == 0
    assert autotune.choose_item_rows("cvrp", 500, times, {("cvrp", 500): 16}, 0.03) == 16
    assert autotune.choose_item_rows("cvrp", 10000, times, {("cvrp", 500): 16}, 0.03) == 0  # not in the mix
