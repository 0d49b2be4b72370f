"""ltl4c_wait after the context moved to another stream: errors of work since the
last wait on the stream before (the null stream, which a blocking copy follows)
are reported, and its results are complete."""
import pytest

from paper_1411_2239_amd import lib
from paper_1411_2239_amd import workloads as W

pytestmark = pytest.mark.gpu


def test_error_of_the_stream_before():
    import torch
    n = 100_000_000                                  # some milliseconds of work
    ctx = lib.Context(0)
    ctx.set_layout(W.prop_layout(3, 1, [10]))
    ids = [ctx.add_spec(W.PropertySpec("G a", [("A", ">=", "1/2")], "p"))]
    rec = torch.zeros((n, 4), dtype=torch.int32, device="cuda:0")
    rec[:, 1] = 1
    rec[-1, 2] = 1 << 10                             # the last event's key is one bit too wide
    small = rec[:1000].clone()
    out = [ctx.alloc_result(1), ctx.alloc_result(1)]
    ws = [torch.empty(max(256, ctx.workspace_bytes(k, ids)), dtype=torch.uint8, device="cuda:0") for k in (n, 1000)]
    out[0].root_counts.zero_()
    side = torch.cuda.Stream()
    ctx.eval_into(small, 1000, ids, out[1], ws[1])   # (every kernel loaded)
    with torch.cuda.stream(side):
        ctx.eval_into(small, 1000, ids, out[1], ws[1])
    ctx.wait()
    torch.cuda.synchronize()
    print("[case] wait on a side stream after work on the null stream", flush=True)
    ctx.eval_into(rec.view(torch.uint8).reshape(-1), n, ids, out[0], ws[0])
    with torch.cuda.stream(side):
        ctx.eval_into(small, 1000, ids, out[1], ws[1])
        with pytest.raises(lib.LTL4CError) as e:
            ctx.wait()
        assert e.value.status == lib.ERANGE
    with torch.cuda.stream(side):                    # no wait of torch's own before this read
        counts = out[0].root_counts.to("cpu")
    assert int(counts.sum()) == 1                    # one instance: the wide key cut to 0
    ctx.wait()                                       # reported once
    ctx.close()
