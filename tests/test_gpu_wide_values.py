"""Event keys wider than declared: ltl4c_wait reports LTL4C_ERANGE, the value is
taken cut to its declared width, and nothing else changes for it: the event
keeps its stream or trace, its kind (own or parent event) and its place, and
the other events their results.  Bits above a key of the top level would
otherwise reach the parent kind, the exclusion bit or the stream id."""
import numpy as np
import pytest

from oracle.run import evaluate_workload
from paper_1411_2239_amd import lib

from _util import compare_full, prop_workload
from test_gpu_parent_events import parent_workload

pytestmark = pytest.mark.gpu


def _cut(wl, records=None):
    """The same records with every key cut to its declared width."""
    r = (wl.records if records is None else records).copy()
    for m, b in enumerate(wl.layout.key_bits):
        r[f"k{m}"] &= np.uint32((1 << b) - 1)
    return r


def _widen(wl, seed, bits, own=True):
    """A few events get one bit of key 0 above its width set (bits: how far above)."""
    t = wl.records["type"]
    at = np.flatnonzero(t < 8 if own else (t >= 8) & (t < 16))
    at = np.random.default_rng(seed).choice(at, min(5, at.size), replace=False)
    wl.records["k0"][at] |= np.uint32(1 << (wl.layout.key_bits[0] + bits))


def _raises_range(call):
    with pytest.raises(lib.LTL4CError) as e:
        call()
    assert e.value.status == lib.ERANGE


@pytest.mark.parametrize("bits", [0, 1, 2, 20])
@pytest.mark.parametrize("own", [True, False])
def test_parent_events(bits, own):
    import torch
    wl = parent_workload(30_000, 2, [40, 300], seed=5 + bits, n_props=3)
    _widen(wl, bits, bits, own)
    print(f"[case] parent events, {bits} bits above, own {own}", flush=True)
    ctx, ids, rec = lib.open_workload(wl)
    n = wl.n_events
    r = ctx.alloc_result(len(ids), n, instances=True, nodes=True)
    ctx.eval_into(rec, n, ids, r, ctx.workspace(n, ids))
    _raises_range(ctx.wait)
    torch.cuda.synchronize()
    compare_full(r, evaluate_workload(wl, records=_cut(wl)), len(ids), 2, key_bits=wl.layout.key_bits)
    ctx.close()


@pytest.mark.parametrize("bits", [0, 1, 20])
@pytest.mark.parametrize("excluded", [False, True])
def test_timeline_and_instances(bits, excluded):
    import torch
    wl = prop_workload(20_000, 2, [40, 30], seed=15 + bits, n_props=2)
    if excluded:
        wl.records["type"][::7] = 200                # carries no key: joins no cluster
    _widen(wl, bits, bits)
    print(f"[case] plain, {bits} bits above, excluded {excluded}", flush=True)
    ctx, ids, rec = lib.open_workload(wl)
    n = wl.n_events
    out = []
    for records in (wl.records, _cut(wl)):
        rec = torch.from_numpy(np.ascontiguousarray(records).view(np.uint8).reshape(-1)).to("cuda:0")
        r = ctx.alloc_result(len(ids), n, instances=True, nodes=True, timeline=True, n_events=n)
        ctx.eval_into(rec, n, ids, r, ctx.workspace(n, ids))
        if not out:
            _raises_range(ctx.wait)
        else:
            ctx.wait()
        out.append(r)
    o = evaluate_workload(wl, records=_cut(wl))
    for r in out:
        compare_full(r, o, len(ids), 2, key_bits=wl.layout.key_bits)
    k = int(out[0].sizes[0].item())
    assert torch.equal(out[0].event_verdict, out[1].event_verdict)
    assert torch.equal(out[0].inst_conclusive.view(len(ids), -1)[:, :k], out[1].inst_conclusive.view(len(ids), -1)[:, :k])
    ctx.close()


def test_other_traces_of_a_batch():
    wl = prop_workload(12_000, 1, [60], seed=31, n_props=3)
    _widen(wl, 3, 1)                                 # the lowest bits of the trace id
    wl.records["type"][::5] = 200
    offsets = [0, 1000, 1000, 5000, 8000, 12_000]
    print("[case] batch", flush=True)
    import torch
    ctx, ids, rec = lib.open_workload(wl)
    P, T = len(ids), len(offsets) - 1
    v = torch.empty(T * P, dtype=torch.uint8, device="cuda:0")
    c = torch.empty(T * P * 6, dtype=torch.int64, device="cuda:0")
    ctx.eval_batch_into(rec, offsets, ids, v, c, ctx.batch_workspace(wl.n_events, T, ids))
    _raises_range(ctx.wait)
    cut = _cut(wl)
    for t in range(T):
        o = evaluate_workload(wl, records=cut[offsets[t]:offsets[t + 1]])
        assert np.array_equal(v.cpu().numpy().reshape(T, P)[t], o.root_verdict)
        assert np.array_equal(c.cpu().numpy().reshape(T, P, 6)[t], o.root_counts.astype(np.int64))
    ctx.close()


@pytest.mark.parametrize("bits", [0, 1, 2, 8])
def test_other_streams_of_a_group(bits):
    import torch
    from test_gpu_serving import _stream_traces
    S, n = 4, 3000
    traces = _stream_traces("users", S, n, 77)
    lay = traces[0].layout
    whole = [t.records.copy() for t in traces]
    print(f"[case] stream group, {bits} bits above", flush=True)
    ctx, ids, _ = lib.open_workload(traces[0])
    grp = lib.StreamGroup(ctx, ids, max_streams=S, max_bindings=4096, max_batch=S * n)
    for push in range(2):
        a, b = push * n // 2, (push + 1) * n // 2
        if push == 1:
            whole[1]["k0"][a + 10:a + 13] |= np.uint32(1 << (lay.key_bits[0] + bits))
        raw = np.concatenate([np.ascontiguousarray(w[a:b]).view(np.uint8).reshape(-1) for w in whole])
        dev = torch.from_numpy(raw).to("cuda:0")
        grp.push(dev, np.arange(S + 1) * (b - a), list(range(S)))
        if push == 1:
            _raises_range(grp.read)
        verdict, counts, bindings = grp.read()
        for s in range(S):
            o = evaluate_workload(traces[s], records=_cut(traces[s], whole[s][:b]))
            assert np.array_equal(verdict[s], o.root_verdict), (push, s)
            assert np.array_equal(counts[s], o.root_counts.astype(np.int64)), (push, s)
            assert bindings[s] == o.inst_keys.shape[0], (push, s)
    grp.close()
    ctx.close()
