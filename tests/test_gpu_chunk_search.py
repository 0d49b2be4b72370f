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


@pytest.mark.parametrize("traces", [223, 224])
def test_trace_table_in_the_launch_or_copied(traces):
    wl = W.gen_prop_trace(40 * traces, 20, 1.1, seed=traces, key_space_bits=8, props=W.batch_properties(3))
    offsets = np.arange(traces + 1) * 40
    print(f"[case] {traces} traces", flush=True)
    ctx, ids, rec = lib.open_workload(wl)
    for _ in range(2):
        v, c = ctx.eval_batch(rec, offsets, ids)
    for t in range(0, traces, 7):
        o = evaluate_workload(wl, records=wl.records[offsets[t]:offsets[t + 1]])
        assert np.array_equal(v[t], o.root_verdict) and np.array_equal(c[t], o.root_counts.astype(np.int64))
    ctx.close()


@pytest.mark.parametrize("chunks", [1, 111, 112])
@pytest.mark.parametrize("pointers", [True, False])
def test_chunk_table_in_the_launch_or_copied(chunks, pointers):
    S, size = 5, 70
    wl = W.gen_user_requests(n_events=2 * chunks * size, n_users=9, seed=chunks)
    print(f"[case] {chunks} chunks, pointers={pointers}", flush=True)
    ctx, ids, rec = lib.open_workload(wl)
    grp = lib.StreamGroup(ctx, ids, S, 4096, chunks * size)
    streams = [(3 * i) % S for i in range(chunks)]
    at = [[] for _ in range(S)]
    for push in range(2):
        first = push * chunks
        if pointers:
            grp.push_chunks([rec.data_ptr() + 16 * size * (first + i) for i in range(chunks)], [size] * chunks, streams)
        else:
            grp.push(rec[16 * size * first:16 * size * (first + chunks)], np.arange(chunks + 1) * size, streams)
        for i, st in enumerate(streams):
            at[st].append(np.arange(size * (first + i), size * (first + i + 1)))
        verdict, counts, bindings = grp.read()
        for st in range(S):
            if not at[st]:
                continue
            o = evaluate_workload(wl, records=wl.records[np.concatenate(at[st])])
            assert np.array_equal(verdict[st], o.root_verdict), (push, st)
            assert np.array_equal(counts[st], o.root_counts.astype(np.int64)), (push, st)
            assert bindings[st] == o.inst_keys.shape[0]
    grp.close()
    ctx.close()


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
