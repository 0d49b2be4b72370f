"""The states and maps prepared for every entry of the parent array: runs whose
ends fall on, before and after the edges of a thread's 8 entries, a wave's 512
and a block's 2,048, runs over several blocks, and what preparing them costs
where a parent has many parent events."""
import numpy as np
import pytest

from oracle.run import evaluate_workload
from paper_1411_2239_amd import lib
from paper_1411_2239_amd import workloads as W

from _util import compare_full
from test_gpu_parent_events import BIG, parent_workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("runs", [[2048], [2047, 2], [2049, 1], [2048, 2048], [1, 2047, 2048, 2049, 7], [511, 1, 512, 513],
                                  [7, 8, 9, 1, 2023], [5000], [1, 9000, 1], [3] * 700, [6143, 2, 2047]])
@pytest.mark.parametrize("props", [1, 5])
def test_run_edges(runs, props):
    import torch
    own = 12                                         # own events of every parent, among its parent events
    n = sum(runs) + own * len(runs)
    wl = parent_workload(n, 2, [len(runs) + 1, 3], seed=n, n_props=props, p_parent=0.0, p_other=0.0,
                         formulas=(BIG + ["G(a -> F b)"])[-props:])
    rng = np.random.default_rng(n)
    parent = np.repeat(np.arange(len(runs), dtype=np.uint32), np.array(runs) + own)
    kind = np.concatenate([rng.permutation(np.repeat(np.uint32([8, 0]), [r, own])) for r in runs])
    at = rng.permutation(n)                          # parents interleaved in the trace
    wl.records["k0"], wl.records["type"] = parent[at], (wl.records["type"] & 7) | kind[at]
    print(f"[case] runs {runs[:6]} props {props}", flush=True)
    ctx, ids, rec = lib.open_workload(wl)
    r = ctx.eval(rec, ids, instances=True, nodes=True)
    torch.cuda.synchronize()
    compare_full(r, evaluate_workload(wl), props, 2, key_bits=wl.layout.key_bits)
    ctx.close()


@pytest.mark.parametrize("own", [0, 1])
def test_preparation_of_long_runs_is_linear(own):
    """2M parent events of one parent and 16 properties, with as many own events
    of one instance or none: at most 40 ps per parent event and property, twenty
    times the 17 bytes it has to move at 8 TB/s (a walk over the segment tree per
    entry took 106 ps)."""
    import torch
    n = 4_000_000 if own else 2_000_000
    lay = W.prop_layout(3, 2, [1, 10])
    lay.class_of_type[8:16], lay.key_present[8:16], lay.parent_events = np.arange(8), 1, True
    ctx = lib.Context(0)
    ctx.set_layout(lay)
    ids = [ctx.add_spec(W.PropertySpec(s.formula, s.quants * 2, s.name)) for s in W.batch_properties(16)]
    g = torch.Generator(device="cuda:0")
    g.manual_seed(1)
    rec = torch.zeros((n, 4), dtype=torch.int32, device="cuda:0")
    rec[:, 1] = torch.randint(0, 8, (n,), generator=g, device="cuda:0", dtype=torch.int32) + 8
    if own:
        rec[::2, 1] -= 8
    rec = rec.view(torch.uint8).reshape(-1)
    r, ws = ctx.alloc_result(16), ctx.workspace(n, ids)
    print(f"[case] 2M parent events, own events {n // 2 if own else 0}", flush=True)
    ctx.eval_into(rec, n, ids, r, ws)
    ctx.wait()
    ctx.profile(True)
    ctx.profile_reset()
    for _ in range(5):
        ctx.eval_into(rec, n, ids, r, ws)
    us = 1e3 * ctx.profile_read()["parent"][0] / 5
    ctx.profile(False)
    ctx.wait()
    ctx.close()
    assert us * 1e6 <= 40 * 2_000_000 * 16, us
