"""An empty trace whose keys are wider than the sort word: the ranking has
nothing to count, whatever the workspace held before."""
import numpy as np
import pytest

from paper_1411_2239_amd import lib

from _util import prop_workload

pytestmark = pytest.mark.gpu


def test_empty_trace_of_wide_keys():
    import torch
    got = []
    for bits in (10, 32):                     # 32 + 32 bits are ranked, 10 + 10 are not
        wl = prop_workload(0, 2, [50, 40], seed=1, n_props=2, key_bits=[bits, bits])
        print(f"[case] no events, {bits}-bit keys", flush=True)
        ctx = lib.Context(0)
        ctx.set_layout(wl.layout)
        ids = [ctx.add_spec(p) for p in wl.props]
        ws = torch.full((ctx.workspace_bytes(0, ids),), 255, dtype=torch.uint8, device="cuda:0")
        r = ctx.alloc_result(2, 1)
        ctx.eval_into(torch.empty(16, dtype=torch.uint8, device="cuda:0"), 0, ids, r, ws)
        ctx.wait()
        got.append([t.cpu().numpy() for t in (r.root_verdict, r.root_counts, r.sizes)])
        ctx.close()
    for narrow, wide in zip(*got):
        assert np.array_equal(narrow, wide)
