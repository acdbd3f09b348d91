"""Bernoulli calls that sample nothing, or everything, captured and replayed
(GPU): every replay writes the count, beside the program's own work."""
import ctypes

import pytest

from tests.gpu_util import announce, dcs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("edges", [False, True])
@pytest.mark.parametrize("p,count", [(0.0, 0), (1.0, 45)])
def test_captured_extremes(edges, p, count):
    import torch
    m = dcs()
    announce(f"captured Bernoulli p={p} edges={edges}")
    out = torch.zeros(64, dtype=torch.int64, device="cuda")
    cnt = torch.zeros(1, dtype=torch.int64, device="cuda")

    def call():
        if edges:
            m.sample_edges_gnp(10, p, 3, out=out.view(torch.int32).view(-1, 2), count=cnt)
        else:
            m.sample_bernoulli(p, 45, 3, out=out, count=cnt)

    call()
    torch.cuda.synchronize()
    want = out.clone()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call()
    for i in range(5):
        cnt.fill_(1000 + i)
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert int(cnt) == count and torch.equal(out, want)


def test_nothing_sampled_records_no_memset():
    """What a call with p = 0 records is a kernel: a node of another kind
    (a memset) may write something else on later replays."""
    import torch
    m = dcs()
    hip = ctypes.CDLL("libamdhip64.so")
    cnt = torch.zeros(1, dtype=torch.int64, device="cuda")
    out = torch.zeros(8, dtype=torch.int64, device="cuda")
    m.sample_bernoulli(0.0, 45, 3, out=out, count=cnt)
    torch.cuda.synchronize()
    stream = torch.cuda.Stream()
    graph = ctypes.c_void_p()
    announce("nodes of a captured Bernoulli p=0")
    with torch.cuda.stream(stream):
        handle = ctypes.c_void_p(stream.cuda_stream)
        assert hip.hipStreamBeginCapture(handle, 1) == 0  # thread local
        m.sample_bernoulli(0.0, 45, 3, out=out, count=cnt)
        assert hip.hipStreamEndCapture(handle, ctypes.byref(graph)) == 0
    n = ctypes.c_size_t(0)
    assert hip.hipGraphGetNodes(graph, None, ctypes.byref(n)) == 0
    nodes = (ctypes.c_void_p * n.value)()
    assert hip.hipGraphGetNodes(graph, nodes, ctypes.byref(n)) == 0
    kinds = []
    for node in nodes:
        kind = ctypes.c_int(-1)
        assert hip.hipGraphNodeGetType(ctypes.c_void_p(node), ctypes.byref(kind)) == 0
        kinds.append(kind.value)
    assert hip.hipGraphDestroy(graph) == 0
    assert kinds == [0]  # hipGraphNodeTypeKernel
