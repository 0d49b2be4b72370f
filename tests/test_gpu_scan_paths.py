"""The map scan's ways through a tile: pairs of symbols (classes of at most 3
bits) or single words, ends found one by one (fewer than 256 heads in a tile of
4,096 words) or by stepping every word, runs with and without heads, the last
tile's remainder; launches of one to eight maps of 8 and of 16 states."""
import numpy as np
import pytest

from oracle.run import evaluate_workload
from paper_1411_2239_amd import lib
from paper_1411_2239_amd import workloads as W

from _util import compare_full

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("length", [1, 3, 15, 16, 17, 4096, 9000])
@pytest.mark.parametrize("props", [1, 2, 4, 8, 16])
@pytest.mark.parametrize("letters", [3, 4])        # 8 classes, 16 classes
@pytest.mark.parametrize("scan", [4, 5])
def test_scan_paths(length, props, letters, scan):
    n = 3 * 8192 + 37
    wl = W.gen_prop_trace(n, 2, 1.0, p_props=(0.3, 0.6, 0.4, 0.5)[:letters], seed=length + props, key_space_bits=16,
                          props=W.batch_properties(props))
    wl.records["k0"] = np.arange(n) // length      # instances of exactly `length` words
    print(f"[case] length {length} props {props} letters {letters} scan {scan}", flush=True)
    ctx, ids, rec = lib.open_workload(wl)
    ctx.set_option(lib.OPT_SCAN_TILE, scan)
    r = ctx.eval(rec, ids, instances=True)
    compare_full(r, evaluate_workload(wl), props, 1)
    ctx.close()
