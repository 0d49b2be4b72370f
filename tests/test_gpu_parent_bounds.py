"""Parent events merged into the map scan: parts of the parent array around the
2,048 entries a block copies to LDS, own events around a block's 4,096 and a
thread's 16, runs of exactly 8 and 9 parent entries (the short gap), and scan
launches of one to five properties with small and 16-state monitors."""
import numpy as np
import pytest

from oracle.run import evaluate_workload
from paper_1411_2239_amd import lib

from _util import compare_full
from test_gpu_parent_events import BIG, parent_workload

pytestmark = pytest.mark.gpu


def _check(n_own, n_par, keys, props, seed):
    import torch
    n = n_own + n_par
    wl = parent_workload(n, 2, keys, seed, n_props=props, p_parent=0.0, p_other=0.0,
                         formulas=(BIG + ["G(a -> F b)"])[-props:])
    at = np.random.default_rng(seed).permutation(n)[:n_par]
    wl.records["type"][at] |= 8                      # exactly n_par parent events
    print(f"[case] own {n_own} parent {n_par} keys {keys} props {props}", flush=True)
    ctx, ids, rec = lib.open_workload(wl)
    r = ctx.eval(rec, ids, instances=True, nodes=True)
    torch.cuda.synchronize()
    compare_full(r, evaluate_workload(wl), props, 2, key_bits=wl.layout.key_bits)
    ctx.close()


@pytest.mark.parametrize("n_par", [1, 63, 64, 65, 2047, 2048, 2049, 4097])
def test_one_parent(n_par):
    _check(9000, n_par, [1, 700], 2, n_par)


@pytest.mark.parametrize("n_own", [1, 15, 16, 17, 4095, 4096, 4097])
@pytest.mark.parametrize("props", [1, 5])
def test_own_events(n_own, props):
    _check(n_own, 300, [5, 30], props, n_own)


@pytest.mark.parametrize("run", [8, 9])
def test_runs_at_the_short_gap(run):
    _check(20_000, 500 * run, [500, 20], 3, run)
