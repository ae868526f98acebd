"""Calls captured into a graph without a caller's workspace: what they record,
and replays beside eager calls that take and return the kept workspaces."""
import ctypes
import sys

import numpy as np
import pytest

import mmp_inputs as gen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
mmp = pytest.importorskip("paper_2601_07508_amd")

KERNEL_NODE = 0  # hipGraphNodeTypeKernel
P36, P50 = 68719476731, 1125899906842597


def say(*a):
    print(*a, file=sys.stderr, flush=True)


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def problem(seed, p, m, n, k):
    A = gen.random_matrix(seed, 1, m, k, p)
    B = gen.random_matrix(seed, 2, k, n, p)
    want = torch.from_numpy(oracle.mm_modp(p, A, B).astype(np.float64)).cuda()
    return (torch.from_numpy(A.astype(np.float64)).cuda(), torch.from_numpy(B.astype(np.float64)).cuda(),
            torch.full((m, n), -1.0, dtype=torch.float64, device="cuda"), p, want)


def capture(call):
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(g, stream=s):
        call(s)
    g.instantiate()
    return g


def node_types(g):
    """The node types of a captured graph, by the runtime that the library is linked with."""
    hip = mmp.lib()
    graph, count = ctypes.c_void_p(g.raw_cuda_graph()), ctypes.c_size_t()
    assert hip.hipGraphGetNodes(graph, None, ctypes.byref(count)) == 0
    nodes = (ctypes.c_void_p * count.value)()
    assert hip.hipGraphGetNodes(graph, nodes, ctypes.byref(count)) == 0
    kinds = []
    for node in nodes:
        kind = ctypes.c_int(-1)
        assert hip.hipGraphNodeGetType(ctypes.c_void_p(node), ctypes.byref(kind)) == 0
        kinds.append(kind.value)
    return kinds


def test_batch_on_fp64_words_records_kernels_alone():
    # four of 512^3: on INT8 words when run eagerly, with a workspace that no product's plan calls for
    items = [problem(i, P36, 512, 512, 512) for i in range(4)]
    jobs = [(A, B, C, p, 0, 0) for A, B, C, p, _ in items]
    assert all(mmp.plan(P36, 512, 512, 512, splits=1)["workspace_bytes"] == 0 for _ in items)
    assert mmp.workspace_batched(jobs) > 0
    g = capture(lambda s: mmp.mm_modp_batched(jobs, stream=s))
    kinds = node_types(g)
    say("batch capture", kinds)
    assert kinds and set(kinds) == {KERNEL_NODE}
    for rep in range(3):
        for *_, C, _p, _w in items:
            C.fill_(-2.0)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(C, want) for _, _, C, _, want in items)
        for *_, C, _p, _w in items:
            C.fill_(-3.0)
        mmp.mm_modp_batched(jobs)  # eager, on INT8 words
        torch.cuda.synchronize()
        assert all(torch.equal(C, want) for _, _, C, _, want in items)
