"""The benchmark's result line: tables of timings leave it for the log."""
import json

import bench


def test_long_tables_leave_the_line():
    table = {f"lambda/t{k}": 0.5 * k for k in range(40)}
    extra = {"probes": {"copy": {"best_GBps": 5.6, "GBps": table}}, "by_map": table,
             "batch": {"ms": 2.7, "tiles": [64, 64]}, "few": {"a": 1, "b": 2.5}}
    line, tables = bench.split_tables(extra)
    assert line == {"probes": {"copy": {"best_GBps": 5.6}}, "batch": {"ms": 2.7, "tiles": [64, 64]},
                    "few": {"a": 1, "b": 2.5}}
    assert tables == {"probes/copy/GBps": table, "by_map": table}
    assert json.loads(json.dumps(line)) == line
    assert extra["by_map"] == table  # the argument is left as it was
