"""Contexts created and stepped while a stream is being captured: nothing they
do may invalidate the capture, and every replay of the graph leaves the
results of the same calls made eagerly.  Each case runs in a process of its
own, because what the library allocates once per process it must be able to
allocate there."""
import os
import subprocess
import sys

import pytest

from tests.gpu_util import announce, need_gpu

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CASE = """
import sys
import torch
import paper_1911_12954_amd as trg
d, dcut, steps, method = int(sys.argv[1]), int(sys.argv[2]), int(sys.argv[3]), sys.argv[4]

def run(stream):
    ctx = trg.trg_init_ising(0.2, 1e-3, d, dcut=dcut, method=method, stream=stream, workspace_bytes=1 << 28)
    for n in range(steps):
        (ctx.atrg_step if method == "atrg" else ctx.hotrg_step)(n % d, dcut)
    return ctx

x = torch.zeros(4, device="cuda")
torch.cuda.synchronize()
graph, stream = torch.cuda.CUDAGraph(), torch.cuda.Stream()
with torch.cuda.graph(graph, stream=stream):
    x.add_(1.0)
    captured = run(stream)
eager = run(torch.cuda.current_stream())
ref = eager.free_energy()
for n in range(3):
    graph.replay()
    torch.cuda.synchronize()
    x.mul_(2.0)     # eager work between the replays
    got = captured.free_energy()
    assert got == ref, (n, got, ref)
assert x.tolist() == [14.0] * 4, x.tolist()
print("replays agree", ref)
"""


@pytest.mark.parametrize("d,dcut,steps,method", [(2, 4, 4, "hotrg"), (2, 14, 8, "hotrg"), (4, 4, 5, "hotrg"),
                                                 (2, 8, 4, "atrg")])
def test_first_context_inside_a_capture(d, dcut, steps, method):
    need_gpu()
    announce("first context inside a capture", d, dcut, steps, method)
    r = subprocess.run([sys.executable, "-u", "-c", CASE, str(d), str(dcut), str(steps), method], cwd=ROOT,
                       capture_output=True, text=True, timeout=100)
    print(r.stdout[-2000:], r.stderr[-2000:], flush=True)
    assert r.returncode == 0 and "replays agree" in r.stdout
