"""The chunk of a record, found by moving forward from the previous one:
traces of 0, 1, 63, 64, 65 and more events, runs of empty traces longer than
the forward steps, traces that begin inside a wave; below and above the size
at which a block takes one contiguous part per step (524,288 records)."""
import numpy as np
import pytest

from oracle.run import evaluate_workload
from paper_1411_2239_amd import lib
from paper_1411_2239_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("big", [5_000, 530_000])
def test_chunk_of_every_record(big):
    rng = np.random.default_rng(big)
    lens = np.concatenate([rng.choice([0, 0, 1, 2, 63, 64, 65, 200], size=150), np.zeros(40, np.int64), [big],
                           np.zeros(9, np.int64), rng.choice([0, 1, 4096, 4097], size=30)]).astype(np.int64)
    offsets = np.concatenate([[0], np.cumsum(lens)])
    n = int(offsets[-1])
    wl = W.gen_prop_trace(n, 50, 1.1, seed=big, key_space_bits=8, props=W.batch_properties(2))
    print(f"[case] {len(lens)} traces, {n} events", flush=True)
    ctx, ids, rec = lib.open_workload(wl)
    v, c = ctx.eval_batch(rec, offsets, ids)
    for t in range(len(lens)):
        o = evaluate_workload(wl, records=wl.records[offsets[t]:offsets[t + 1]])
        assert np.array_equal(v[t], o.root_verdict), (t, int(lens[t]))
        assert np.array_equal(c[t], o.root_counts.astype(np.int64)), (t, int(lens[t]))
    ctx.close()
