"""A process loads a kind's kernels with the first call of one, also where that call is captured into a graph: every replay as the eager call after it."""
import subprocess
import sys

import pytest

from conftest import ROOT

pytestmark = pytest.mark.gpu

CHILD = """
import torch
import paper_2103_14949_amd as hago

g = torch.Generator(device="cuda:0")
g.manual_seed(5)
codes = lambda *shape: torch.randint(-127, 128, shape, generator=g, device="cuda:0", dtype=torch.int8)
q = hago.QType(hago.I8)

def requant(n, kind):
    if kind == "raw":
        return None
    mult = torch.randint(2 ** 30, 2 ** 31 - 1, (n,), generator=g, device="cuda:0", dtype=torch.int64).to(torch.int32)
    return hago.Requant(mult, torch.full((n,), 9, dtype=torch.int32, device="cuda:0"), q, *((-100, 90) if kind == "clipped" else (None, None)))

def calls(kind):
    found = []
    for M, K, N in ((2048, 768, 3072), (2048, 768, 768)):
        a, w, rq = codes(M, K), codes(N, K), requant(N, kind)
        found.append(lambda a=a, w=w, rq=rq: hago.qdense(a, q, w, q, None, hago.I32, rq))
    for C, H, O, k, s in ((64, 28, 64, 3, 1), (3, 64, 64, 7, 2)):
        a, w, rq = codes(2, C, H, H), codes(O, C, k, k), requant(O, kind)
        found.append(lambda a=a, w=w, rq=rq, k=k, s=s: hago.qconv2d(a, q, w, q, None, hago.NCHW, (s, s), (k // 2, k // 2), 1, hago.I32, rq))
    return found

for call in calls("whole"):
    call()
first = calls("raw") + calls("clipped")
torch.cuda.synchronize()
stream, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
with torch.cuda.stream(stream), torch.cuda.graph(graph, stream=stream):
    captured = [call() for call in first]
for replay in range(3):
    for out in captured:
        out.zero_()
    torch.cuda.synchronize()
    graph.replay()
    torch.cuda.synchronize()
    for i, (out, call) in enumerate(zip(captured, first)):
        want = call()
        torch.cuda.synchronize()
        assert torch.equal(out, want) and int(out.count_nonzero()) > 0, (replay, i)
print("captured: ok")
"""


def test_first_calls_of_other_kinds_of_results():
    r = subprocess.run([sys.executable, "-c", CHILD], cwd=ROOT, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and "captured: ok" in r.stdout, r.stdout + r.stderr
