"""The launch counts the library reports are those it issues: the nodes of a captured graph of each call,
for every path of epl_layout_dispatch, its two phases and epl_layout."""
import ctypes

import pytest
import torch

from paper_2607_06202_amd import epl
from tests.gpu_util import device

pytestmark = pytest.mark.gpu


def _launches(fn):
    """Kernel launches of fn: it runs once eagerly, then into a graph, whose nodes are counted."""
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        fn()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        fn()
    n = ctypes.c_size_t()
    assert epl._hip_runtime().hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(n)) == 0
    return n.value


@pytest.mark.parametrize("R,E,k,Tr,payload,launches", [
    (4, 16, 2, 128, "bf16", 1), (16, 64, 8, 30, "fp8", 1), (1024, 1024, 2, 3, "bf16", 1),
    (4, 64, 1, 4096, "bf16", 2), (2, 6, 1, 1500, "fp8", 2), (512, 1024, 2, 14, "bf16", 2),
    (64, 256, 8, 40, "bf16", 3), (16, 64, 8, 1024, "bf16", 3), (64, 256, 8, 40, "fp8", 3),
    (64, 512, 8, 64, "bf16", 4), (16, 512, 4, 300, "fp8", 4)])
def test_reported_launches_are_issued(R, E, k, Tr, payload, launches):
    dev = device()
    H = 2048 if (R, payload) == (2, "fp8") else 128
    cfg = epl.config(R, E, k, H, Tr, payload)
    idx = torch.randint(0, E, (cfg.T, k), dtype=torch.int32, device=dev)
    x = torch.randn(cfg.T, H, device=dev).to(torch.bfloat16)
    L = epl.alloc_layout(cfg, dev)
    recv, scale = epl.alloc_recv(cfg, dev)
    assert epl.layout_dispatch_launches(cfg) == launches
    assert _launches(lambda: epl.layout_dispatch(cfg, idx, x, out=L, recv=recv, recv_scale=scale)) == launches
    assert _launches(lambda: epl.layout_counts(cfg, idx, out=L)) == max(launches - 1, 1)
    assert _launches(lambda: epl.dispatch_rows(cfg, idx, x, L, recv, scale)) == 1
    assert _launches(lambda: epl.layout(cfg, idx, out=L)) == epl.layout_launches(cfg)
