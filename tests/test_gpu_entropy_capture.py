"""GPU: `entropy_argmax` under graph capture.  Small eager calls take one launch and count arrivals in words that carry the
call's number; a captured call, whose number would be frozen, takes two launches and uses no such state."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

# Runs in a process of its own: the very first call of a process is the captured one (it may allocate, hence the relaxed mode,
# but neither clear memory nor synchronise).
CHILD = """
import ctypes, sys
import torch
import paper_2502_06833_amd as ead
rows, V, dt = int(sys.argv[1]), int(sys.argv[2]), getattr(torch, sys.argv[3])
xs = [(torch.randn(r, v, generator=torch.Generator().manual_seed(r)) * 3).to(dt).cuda() for r, v in ((rows, V), (1, 128256), (3, 8))]
out = torch.zeros(rows, device="cuda"), torch.zeros(rows, dtype=torch.int32, device="cuda")
torch.cuda.synchronize()
graph = torch.cuda.CUDAGraph(keep_graph=True)
with torch.cuda.graph(graph, capture_error_mode="relaxed"):
    ead.entropy_argmax(xs[0], out=out)
path = next(l.split()[-1] for l in open("/proc/self/maps") if "libamdhip64" in l)
nodes = ctypes.c_size_t(0)
assert ctypes.CDLL(path).hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(nodes)) == 0
assert nodes.value == 2, nodes.value
ref = [tuple(t.clone() for t in ead.entropy_argmax(x, static=True)) for x in xs]
p = xs[0].double().softmax(-1)
assert (ref[0][0] + (p * p.log()).sum(-1)).abs().max() < 1e-4 and (ref[0][1] == xs[0].argmax(-1)).all()
for _ in range(4):
    out[0].zero_(); out[1].zero_()
    graph.replay()
    torch.cuda.synchronize()
    assert torch.equal(out[0], ref[0][0]) and torch.equal(out[1], ref[0][1])
    for x, (h, a) in zip(xs, ref):
        h1, a1 = ead.entropy_argmax(x)
        assert torch.equal(h1, h) and torch.equal(a1, a)
    torch.cuda.synchronize()
print("capture ok", flush=True)
"""


@pytest.mark.parametrize("rows,V,dtype", [(1, 128256, "bfloat16"), (16, 50264, "float32"), (64, 512, "bfloat16")])
def test_first_call_of_a_process_can_be_captured(rows, V, dtype):
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", CHILD, str(rows), str(V), dtype], cwd=root, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and "capture ok" in r.stdout, r.stderr[-2000:]
