"""10-bit radix digits (a thread per bucket): key widths where they save a pass,
and one bit more, at the edges of tiles and of groups of 16 tiles, with excluded
events; and ranked keys, which take fewer bits than the workspace was sized for."""
import numpy as np
import pytest

from oracle.run import evaluate_workload
from paper_1411_2239_amd import lib

from _util import compare_full, prop_workload

pytestmark = pytest.mark.gpu


def _check(wl):
    print(f"[case] {wl.n_events} events, key bits {wl.layout.key_bits}", flush=True)
    import torch
    ctx = lib.Context(0, use_tuned=False)
    ctx.set_layout(wl.layout)
    ids = [ctx.add_spec(p) for p in wl.props]
    rec = torch.from_numpy(np.ascontiguousarray(wl.raw())).to("cuda:0")
    r = ctx.eval(rec, ids, instances=True, nodes=True)
    compare_full(r, evaluate_workload(wl), len(ids), wl.layout.n_keys)
    ctx.close()


@pytest.mark.parametrize("n", [1, 2048, 2049, 16 * 2048 + 1, 256 * 2048 + 1, 256 * 6144 + 1, 256 * 13312 + 1])
@pytest.mark.parametrize("bits", [[10], [11], [10, 10], [14, 16], [20, 20], [19, 22]])
def test_wide_digits(n, bits):
    # (both ends of the key range are taken, so that the last buckets fill)
    wl = prop_workload(n, len(bits), [1 << b for b in bits], seed=n + sum(bits), n_props=2, key_bits=bits)
    for m, b in enumerate(bits):
        wl.records[f"k{m}"][::5] = (1 << b) - 1
        wl.records[f"k{m}"][1::5] = 0
    wl.records["type"][3::7] = 300
    wl.layout.type_bytes = 2
    _check(wl)


@pytest.mark.parametrize("n,keys", [(5000, 1000), (1_060_000, 1 << 20)])
def test_ranked_keys_of_fewer_bits(n, keys):
    # sized for two levels of bits_for(n) bits (13, 21), ranked to 10 or 20 bits each
    wl = prop_workload(n, 2, [keys, keys], seed=n, n_props=1, key_bits=[32, 32])
    for k in ("k0", "k1"):
        wl.records[k] = (wl.records[k].astype(np.uint64) * 0x9E3779B1 % (1 << 32)).astype(np.uint32)
    print(f"[case] {n} events, {keys} values a level", flush=True)
    ctx, ids, rec = lib.open_workload(wl)
    r = ctx.eval(rec, ids, instances=True, key_values=True)
    o = evaluate_workload(wl)
    r.key_bits = None                 # packed ranks: compared through their values
    compare_full(r, o, 1, 2, check_nodes=False)
    k = int(r.sizes[0].item())
    assert np.array_equal(r.inst_key_values.cpu().numpy().view(np.uint32).reshape(-1, 2)[:k], o.inst_keys)
    ctx.close()
