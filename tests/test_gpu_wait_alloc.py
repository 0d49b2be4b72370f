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
