"""The radix pass whose tile is fitted to the trace (variant 6): sizes at the
edges of its tiles, of its groups of 16 tiles, of its rounds of 256 tiles and of
its grouped look-back, with 8- and 9-bit digits; and workspaces: one planned
for a size serves every smaller size."""
import numpy as np
import pytest

from oracle.run import evaluate_workload
from paper_1411_2239_amd import lib
from paper_1411_2239_amd import workloads as W

from _util import compare_full

pytestmark = pytest.mark.gpu

SIZES = [1, 2047, 2049, 15 * 2048, 16 * 2048, 16 * 2048 + 1, 33 * 2048 - 1, 256 * 2048, 256 * 2048 + 1,
         256 * 4096 + 1, 256 * 6144 + 1, 256 * 8192 + 1, 256 * 10240 + 1, 256 * 12288 + 1, 256 * 13312 + 1]


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("bits", [32, 36])
def test_sort_shapes(n, bits):
    if bits == 32:       # four 8-bit passes
        wl = W.gen_prop_trace(n, max(1, n // 7), 0.8, seed=n, props=W.timeline_properties())
    else:                # four 9-bit passes; some events excluded
        wl = W.gen_user_requests(n_events=max(n, 40), n_users=12, seed=n)
        wl.records = wl.records[:n]
        wl.records["type"][::17] = 300
        wl.layout.key_bits = [14, 22]
    print(f"[case] {n} events, {bits} key bits", flush=True)
    ctx = lib.Context(0, use_tuned=False)
    ctx.set_layout(wl.layout)
    ids = [ctx.add_spec(p) for p in wl.props]
    import torch
    rec = torch.from_numpy(np.ascontiguousarray(wl.raw())).to("cuda:0")
    r = ctx.eval(rec, ids, instances=True, nodes=bits == 36)
    compare_full(r, evaluate_workload(wl), len(ids), wl.layout.n_keys, check_nodes=bits == 36)
    ctx.close()


def test_beyond_the_grouped_look_back():
    wl = W.gen_prop_trace(4 * 256 * 16384 + 1, 1000, 1.0, seed=3, key_space_bits=10, props=W.timeline_properties()[:1])
    print(f"[case] {wl.n_events} events", flush=True)
    ctx, ids, rec = lib.open_workload(wl)
    r = ctx.eval(rec, ids, instances=True, capacity=1024)
    compare_full(r, evaluate_workload(wl), 1, 1)
    ctx.close()


def test_workspace_serves_smaller_traces():
    wl = W.gen_user_requests(n_events=100, n_users=5, seed=1)
    ctx = lib.Context(0, use_tuned=False)
    ctx.set_layout(wl.layout)
    ids = [ctx.add_spec(p) for p in wl.props]
    edges = sorted({1024 * i * 256 * r + d for i in (2, 4, 6, 8, 10, 12, 13, 14, 16) for r in (1, 2, 3, 4) for d in (0, 1)})
    need = [ctx.workspace_bytes(n, ids) for n in edges]
    assert need == sorted(need)
    ctx.close()


def test_small_workspace_takes_the_largest_tiles():
    import torch
    wl = W.gen_user_requests(n_events=1_500_000, n_users=300, seed=8)
    ctx = lib.Context(0, use_tuned=False)
    ctx.set_layout(wl.layout)
    ids = [ctx.add_spec(p) for p in wl.props]
    rec = torch.from_numpy(np.ascontiguousarray(wl.raw())).to("cuda:0")
    n = wl.n_events
    full = ctx.workspace_bytes(n, ids)
    ctx.set_option(lib.OPT_SORT_TILE, 1)
    less = ctx.workspace_bytes(n, ids)
    ctx.set_option(lib.OPT_SORT_TILE, -1)
    assert less < full
    ws = torch.empty(less, dtype=torch.uint8, device="cuda:0")
    r = ctx.alloc_result(len(ids), n, instances=True)
    ctx.eval_into(rec, n, ids, r, ws)
    ctx.wait()
    compare_full(r, evaluate_workload(wl), len(ids), 2, check_nodes=False)
    with pytest.raises(lib.LTL4CError):
        ctx.eval_into(rec, n, ids, r, ws[:less // 2])
    ctx.close()
