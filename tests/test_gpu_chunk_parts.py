"""Classify with chunks on both sides of the size from which each block takes one
contiguous part per step (as many records as threads: 131,072 for traces below
524,288 records), for records of 12, 16 and 20 bytes (three, four and a run-time
count of words per record)."""
import numpy as np
import pytest

from oracle.run import evaluate_workload
from paper_1411_2239_amd import lib
from paper_1411_2239_amd import workloads as W

from _util import prop_workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [131_071, 131_072, 131_073, 300_001])
@pytest.mark.parametrize("record", [12, 16, 20])
def test_batch(n, record):
    if record == 12:
        wl = W.gen_sockets(n, n_sockets=40, seed=n)
    else:
        levels = 1 if record == 16 else 3
        wl = prop_workload(n, levels, [9, 5, 4][:levels], seed=n, n_props=3)
    assert wl.layout.record_bytes == record
    rng = np.random.default_rng(n)
    offsets = np.sort(np.concatenate([[0, 0, n, n], rng.integers(0, n, 120), 1024 * rng.integers(0, n // 1024, 20)]))
    print(f"[case] {n} records of {record} bytes, {len(offsets) - 1} traces", flush=True)
    ctx, ids, rec = lib.open_workload(wl)
    v, c = ctx.eval_batch(rec, offsets, ids)
    for t in range(len(offsets) - 1):
        o = evaluate_workload(wl, records=wl.records[offsets[t]:offsets[t + 1]])
        assert np.array_equal(v[t], o.root_verdict), t
        assert np.array_equal(c[t], o.root_counts.astype(np.int64)), t
    ctx.close()
