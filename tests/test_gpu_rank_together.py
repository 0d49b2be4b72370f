"""Keys wider than the sort word: all levels ranked in the same launches, and one
level after the other when the workspace has no room for that; edges of the
radix and ranking tiles."""
import numpy as np
import pytest

from oracle.run import evaluate_workload
from paper_1411_2239_amd import lib

from _util import prop_workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2047, 2049, 4096, 4097, 60_001])
@pytest.mark.parametrize("levels", [2, 4])
def test_levels_together_and_apart(n, levels):
    import torch
    wl = prop_workload(n, levels, [7, 30, 5, 9][:levels], seed=n + levels, n_props=2, key_bits=[32] * levels)
    for m in range(levels):      # distinct, spread 32-bit values
        wl.records[f"k{m}"] = (wl.records[f"k{m}"].astype(np.uint64) * 0x9E3779B1 + 77 * m).astype(np.uint32)
    print(f"[case] {n} events, {levels} levels", flush=True)
    ctx, ids, rec = lib.open_workload(wl)
    o = evaluate_workload(wl)
    need = ctx.workspace_bytes(n, ids)
    for size in (need, need - 1):                 # the second has no room for all levels at once
        ws = torch.empty(size, dtype=torch.uint8, device="cuda:0")
        r = ctx.alloc_result(len(ids), max(n, 1), instances=True, nodes=True, key_values=True)
        ctx.eval_into(rec, n, ids, r, ws)
        ctx.wait()
        k = int(r.sizes[0].item())
        assert k == o.inst_keys.shape[0]
        assert np.array_equal(r.root_verdict.cpu().numpy(), o.root_verdict)
        assert np.array_equal(r.root_counts.cpu().numpy().reshape(-1, 6), o.root_counts.astype(np.int64))
        assert np.array_equal(r.inst_verdict.view(len(ids), -1)[:, :k].cpu().numpy(), o.inst_verdict)
        values = r.inst_key_values.view(-1, levels)[:k].cpu().numpy().view(np.uint32)
        assert np.array_equal(values, o.inst_keys.astype(np.uint32))
    ctx.close()
