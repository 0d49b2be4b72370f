"""The packed verdicts after every event: sizes around the 8 events a thread
unpacks and the 16 words a thread scans, rows that start at odd bytes, one to
two scan launches of 2- and 4-byte packs, excluded events, and 16-state
monitors."""
import numpy as np
import pytest

from oracle.run import evaluate_workload
from paper_1411_2239_amd import lib
from paper_1411_2239_amd import workloads as W

from _util import compare_full

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 7, 8, 9, 15, 17, 4095, 4097, 20_001])
@pytest.mark.parametrize("props", [1, 4, 5, 9, 16])
def test_event_pack(n, props):
    wl = W.gen_prop_trace(n, max(1, n // 9), 0.9, seed=n + props, key_space_bits=16, props=W.batch_properties(props)[::-1])
    wl.records["type"][np.random.default_rng(n).random(n) < 0.2] = 300      # events of no instance
    print(f"[case] {n} events, {props} properties", flush=True)
    ctx, ids, rec = lib.open_workload(wl)
    r = ctx.eval(rec, ids, instances=True, events=True)
    o = evaluate_workload(wl)
    compare_full(r, o, props, 1)
    assert np.array_equal(r.event_verdict.cpu().numpy().reshape(props, -1), o.event_verdict)
    ctx.close()
