"""A no-allocation evaluation and the wait that completes it allocate nothing,
the first ones of a context included: a child process runs them with the HIP
runtime's own log of API calls, which is searched for allocations."""
import os
import re
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

CHILD = """
import os
import torch
from paper_1411_2239_amd import lib, workloads as W
torch.cuda.init()
rec = torch.zeros(16 * 1000, dtype=torch.uint8, device="cuda:0")
ctx = lib.Context(0)
ctx.set_layout(W.prop_layout(3, 1, [10]))
ids = [ctx.add_spec(W.PropertySpec("G a", [("A", ">=", "1/2")], "p"))]
r = ctx.alloc_result(1)
torch.cuda.synchronize()
os.write(2, b"\\nBEGIN\\n")
for _ in range(2):
    ctx.eval_noalloc_into(rec, 1000, ids, r)
    ctx.wait()
os.write(2, b"\\nEND\\n")
"""


def test_first_wait_allocates_nothing():
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    print("[case] allocations of eval_noalloc and wait, from the runtime's log", flush=True)
    p = subprocess.run([sys.executable, "-c", CHILD], cwd=root, env=dict(os.environ, AMD_LOG_LEVEL="3"),
                       capture_output=True, text=True, errors="replace", timeout=100)
    assert p.returncode == 0, p.stderr[-2000:]
    log = p.stderr[p.stderr.index("\nBEGIN\n"):p.stderr.index("\nEND\n")]
    calls = re.findall(r"\b(hip[A-Z]\w*)\s*\(", log)
    assert "hipStreamSynchronize" in calls           # the log is on
    assert not [c for c in calls if re.search("Malloc|HostAlloc|HostRegister", c)], sorted(set(calls))


def test_error_words_of_many_contexts():
    """More contexts at a time than the page of host words has room for, some
    closed and made again, two threads at it: every context reports its own
    errors and no other's."""
    import threading

    import torch
    from paper_1411_2239_amd import lib, workloads as W
    good = torch.zeros((64, 4), dtype=torch.int32, device="cuda:0")
    bad = good.clone()
    bad[5, 2] = 1 << 12                              # a key wider than declared
    good, bad = good.view(torch.uint8).reshape(-1), bad.view(torch.uint8).reshape(-1)

    def make():
        ctx = lib.Context(0)
        ctx.set_layout(W.prop_layout(3, 1, [10]))
        ids = [ctx.add_spec(W.PropertySpec("G a", [("A", ">=", "1/2")], "p"))]
        return ctx, ids, ctx.alloc_result(1), ctx.workspace(64, ids)

    failures = []

    def work(k):
        try:
            all_ctx = [make() for _ in range(40)]
            for ctx, *_ in all_ctx[::3]:
                ctx.close()
            all_ctx = [make() if i % 3 == 0 else c for i, c in enumerate(all_ctx)]
            for i, (ctx, ids, r, ws) in enumerate(all_ctx):
                ctx.eval_into(bad if (i + k) % 2 else good, 64, ids, r, ws)
            for i, (ctx, *_) in enumerate(all_ctx):
                try:
                    ctx.wait()
                    got = lib.OK
                except lib.LTL4CError as e:
                    got = e.status
                if got != (lib.ERANGE if (i + k) % 2 else lib.OK):
                    failures.append((k, i, got))
                ctx.close()
        except Exception as e:                       # (a thread's failure would be lost)
            failures.append((k, repr(e)))

    print("[case] 80 contexts in two threads", flush=True)
    threads = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not failures, failures[:5]
