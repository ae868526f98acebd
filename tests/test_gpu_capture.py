"""Calls captured into a graph without a caller's workspace: what they record,
and replays beside eager calls that take and return the kept workspaces."""
import ctypes
import sys
import threading

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


def test_products_that_need_a_workspace_beside_eager_calls():
    # a captured call allocates for its graph alone; eager calls of the same sizes take
    # and return kept workspaces between the replays, on the same stream and others
    items = [problem(40, P50, 90, 70, 9000), problem(41, P36, 300, 200, 700)]
    kws = [{}, {"form": mmp.FORM_INT8_WORDS}]
    streams = [torch.cuda.Stream() for _ in range(2)]

    def eager(rounds):
        for r in range(rounds):
            for (A, B, C, p, _), kw in zip(items, kws):
                mmp.mm_modp_async(A, B, C, p, stream=streams[r % 2], **kw)
        for s in streams:
            s.synchronize()

    eager(2)
    graphs = []
    for (A, B, C, p, want), kw in zip(items, kws):
        assert mmp.plan(p, *C.shape, A.shape[1], **kw)["workspace_bytes"] > 0
        g = capture(lambda s: mmp.mm_modp_async(A, B, C, p, stream=s, **kw))
        say("product capture", node_types(g))
        graphs.append(g)
    for rep in range(3):
        for g, (A, B, C, p, want) in zip(graphs, items):
            say("replay", rep)
            C.fill_(-2.0)
            torch.cuda.synchronize()
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(C, want)
        for *_, C, _p, _w in items:
            C.fill_(-3.0)
        torch.cuda.synchronize()
        eager(4)
        assert all(torch.equal(C, want) for _, _, C, _, want in items)


def test_another_threads_calls_during_a_capture():
    # a capture in global mode refuses what other threads must not do meanwhile; calls
    # that query, take and return kept workspaces are not among it
    A, B, C, p, want = problem(50, P50, 256, 256, 512)
    X, Y, _, q, expect = problem(51, P36, 300, 200, 700)
    streams = [torch.cuda.Stream() for _ in range(2)]
    outs = [torch.full_like(expect, -1.0) for _ in range(24)]
    ws = torch.empty(1 << 26, dtype=torch.uint8, device="cuda")
    busy = torch.randn(2048, 2048, device="cuda")
    dst = torch.empty_like(busy)
    torch.cuda.synchronize()
    errors = []

    def calls():
        try:
            for i, D in enumerate(outs):
                mmp.mm_modp_async(X, Y, D, q, stream=streams[i % 2], form=mmp.FORM_INT8_WORDS)
            mmp.release_workspaces()
        except Exception as e:  # reported below, in the test's own thread
            errors.append(e)

    with torch.cuda.stream(streams[0]):
        for _ in range(20):
            torch.mm(busy, busy, out=dst)

    def body(s):
        t = threading.Thread(target=calls)
        mmp.mm_modp_async(A, B, C, p, workspace=ws, stream=s)
        t.start()
        t.join()
        mmp.mm_modp_async(A, B, C, p, workspace=ws, stream=s)

    say("another thread during a capture")
    g = capture(body)
    torch.cuda.synchronize()
    assert not errors, errors
    assert all(torch.equal(D, expect) for D in outs)
    for rep in range(3):
        C.fill_(-2.0)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(C, want)
