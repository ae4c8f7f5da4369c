"""The first call that needs scratch words, made while another stream is being captured."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

PROGRAM = """
import numpy as np, torch
import paper_2504_17307_amd as pkg
from synth.layout import DESC, NO_FORWARD
n, C = 3072, 64                                     # no chunk size given: streamed in destination order
g = np.random.default_rng(1)
d = np.zeros(n, dtype=DESC)
d["seq"] = g.permutation(n)
d["src_off"], d["dst_off"], d["out_off"], d["len"] = np.arange(n) * C, d["seq"].astype(np.uint64) * C, NO_FORWARD, C
assert pkg.uccl_launch_ordered(n) == 1
recv = torch.randn(n * C // 4, device="cuda")
acc, bits, recs = torch.zeros_like(recv), torch.zeros(n // 32, dtype=torch.int32, device="cuda"), torch.from_numpy(d.view(np.uint8)).cuda()
x, y = torch.ones(1 << 16, device="cuda"), torch.zeros(1 << 16, device="cuda")
other, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
torch.cuda.synchronize()
with torch.cuda.graph(graph):
    y.add_(x)
    pkg.uccl_chunk_apply(acc, None, recv, recs, n, bits, pkg.UCCL_F32, pkg.UCCL_SUM, stream=other)   # eager, on another stream
    y.add_(x)
other.synchronize()
want = np.zeros(n * C // 4, dtype=np.float32).reshape(n, -1)
want[d["seq"]] = recv.cpu().numpy().reshape(n, -1)
assert np.array_equal(acc.cpu().numpy().reshape(n, -1), want) and bool((bits == -1).all())
for k in range(3):
    graph.replay()
    torch.cuda.synchronize()
    assert bool((y == 2.0 * (k + 1)).all())
assert pkg.uccl_claim_timeouts() == 0
print("FIRST CALL OK")
"""


def test_first_call_beside_a_capture(gpu_lib):
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", PROGRAM], cwd=root, capture_output=True, text=True, timeout=110)
    assert r.returncode == 0 and "FIRST CALL OK" in r.stdout, r.stdout[-1000:] + r.stderr[-3000:]
