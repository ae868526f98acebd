"""Workspaces kept between calls: results stay exact when calls of different
sizes share them over several streams and threads (beside a graph capture:
test_gpu_capture.py), and they stay within their bounds."""
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

# products that need a workspace: digit planes, residue planes, split-K residues
SHAPES = [(4503599627370449, 90, 70, 9000, {}), (1125899906842597, 513, 520, 2048, {}),
          (68719476731, 300, 200, 700, {"form": mmp.FORM_INT8_WORDS}),
          (8388593, 64, 64, 40000, {"form": mmp.FORM_FP64_WORDS})]


def say(*a):
    print(*a, file=sys.stderr, flush=True)


@pytest.fixture(scope="module")
def problems():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    out = []
    for i, (p, m, n, k, kw) in enumerate(SHAPES):
        A = gen.random_matrix(i, 1, m, k, p)
        B = gen.random_matrix(i, 2, k, n, p)
        want = torch.from_numpy(oracle.mm_modp(p, A, B).astype(np.float64)).cuda()
        out.append((p, torch.from_numpy(A.astype(np.float64)).cuda(), torch.from_numpy(B.astype(np.float64)).cuda(),
                    want, kw))
    torch.cuda.synchronize()
    return out


def rounds(problems, streams, count, first, bad):
    outs = []
    for r in range(count):
        p, A, B, want, kw = problems[(first + r) % len(problems)]
        s = streams[r % len(streams)]
        C = torch.empty_like(want)
        mmp.mm_modp_async(A, B, C, p, stream=s, **kw)
        outs.append((C, want))
    for s in streams:
        s.synchronize()
    bad.extend(i for i, (C, want) in enumerate(outs) if not torch.equal(C, want))
    torch.cuda.synchronize()


@pytest.mark.parametrize("nstreams", [1, 3])
def test_streams_share_kept_workspaces(problems, nstreams):
    bad = []
    streams = [torch.cuda.Stream() for _ in range(nstreams)]
    say("streams", nstreams)
    rounds(problems, streams, 60, 0, bad)
    assert not bad


def test_threads_share_kept_workspaces(problems):
    bad = []
    threads = [threading.Thread(target=rounds, args=(problems, [torch.cuda.Stream(), torch.cuda.Stream()], 30, t, bad))
               for t in range(4)]
    say("threads", len(threads))
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad


def used_memory():
    """Bytes taken from the device's default memory pool (hipMemPoolAttrUsedMemCurrent), the workspaces' own."""
    hip, pool, value = mmp.lib(), ctypes.c_void_p(), ctypes.c_uint64()
    assert hip.hipDeviceGetDefaultMemPool(ctypes.byref(pool), 0) == 0
    assert hip.hipMemPoolGetAttribute(pool, 7, ctypes.byref(value)) == 0
    return value.value


def test_kept_blocks_fit_what_they_serve():
    # digit planes of some 137 MB, then of 0.2 MB: neither takes a block much larger
    p = 1125899906842597
    say("block sizes")
    torch.cuda.synchronize()
    for m, n, k in ((4800, 16, 4096), (64, 64, 200)):
        A = torch.ones((m, k), dtype=torch.float64, device="cuda")
        B = torch.ones((k, n), dtype=torch.float64, device="cuda")
        C = torch.empty((m, n), dtype=torch.float64, device="cuda")
        need = mmp.plan(p, m, n, k, form=mmp.FORM_INT8_WORDS, splits=1)["workspace_bytes"]
        before = used_memory()
        mmp.mm_modp_async(A, B, C, p, form=mmp.FORM_INT8_WORDS, splits=1)
        torch.cuda.synchronize()
        assert bool((C == k).all())
        grown = used_memory() - before
        say(m, n, k, need, grown)
        assert grown <= max(1 << 20, need + need // 4)
        mmp.mm_modp_async(A, B, C, p, form=mmp.FORM_INT8_WORDS, splits=1)  # and takes it again
        torch.cuda.synchronize()
        assert used_memory() - before == grown


def test_kept_blocks_are_bounded_and_given_back():
    # eleven streams, each behind work of its own, take blocks of some 240 MB: the
    # last ones find 2 GiB taken, and a later small block makes room for itself
    p, m, n, k = 1125899906842597, 8192, 4, 4096
    A = torch.randint(0, p, (m, k), dtype=torch.int64, device="cuda").double()
    B = torch.randint(0, p, (k, n), dtype=torch.int64, device="cuda").double()
    want = torch.from_numpy(oracle.mm_modp(p, A.cpu().numpy().astype(np.uint64),
                                           B.cpu().numpy().astype(np.uint64)).astype(np.float64)).cuda()
    busy = torch.randn(4096, 4096, device="cuda")
    streams = [torch.cuda.Stream() for _ in range(11)]
    outs = [torch.full((m, n), -1.0, dtype=torch.float64, device="cuda") for _ in streams]
    torch.cuda.synchronize()
    mmp.release_workspaces()
    start = used_memory()
    assert mmp.plan(p, m, n, k, form=mmp.FORM_INT8_WORDS, splits=1)["workspace_bytes"] > 224 << 20
    say("eleven streams")
    for s, C in zip(streams, outs):
        with torch.cuda.stream(s):
            for _ in range(20):
                busy @ busy
        mmp.mm_modp_async(A, B, C, p, form=mmp.FORM_INT8_WORDS, splits=1, stream=s)
    torch.cuda.synchronize()
    assert all(torch.equal(C, want) for C in outs)
    held = used_memory() - start
    say("held", held)
    assert 7 * (224 << 20) < held <= 2 << 30
    small = torch.ones((64, 64), dtype=torch.float64, device="cuda")
    for _ in range(2):
        for shape in ((8192, 4, 2000), (64, 64, 64)):
            X = torch.ones((shape[0], shape[2]), dtype=torch.float64, device="cuda")
            Y = torch.ones((shape[2], shape[1]), dtype=torch.float64, device="cuda")
            C = torch.empty((shape[0], shape[1]), dtype=torch.float64, device="cuda")
            mmp.mm_modp_async(X, Y, C, p, form=mmp.FORM_INT8_WORDS, splits=1)
            torch.cuda.synchronize()
            assert bool((C == shape[2]).all())
            assert used_memory() - start <= 2 << 30
    assert used_memory() > start
    mmp.release_workspaces()
    assert used_memory() == start
    C.copy_(small)
    mmp.mm_modp_async(small, small, C, p, form=mmp.FORM_INT8_WORDS)
    torch.cuda.synchronize()
    assert bool((C == 64).all())


def test_callers_pending_error_is_not_swallowed(problems):
    # a kept block whose event is still pending on another stream, queried and passed over
    p, A, B, want, kw = problems[2]
    hip = mmp.lib()
    first, second = torch.cuda.Stream(), torch.cuda.Stream()
    C, D = torch.empty_like(want), torch.empty_like(want)
    busy = torch.randn(4096, 4096, device="cuda")
    torch.cuda.synchronize()
    with torch.cuda.stream(first):
        for _ in range(20):
            busy @ busy
    mmp.mm_modp_async(A, B, C, p, stream=first, **kw)
    assert hip.hipSetDevice(4096) != 0  # refused by the host: the caller's error
    say("pending error")
    try:
        mmp.mm_modp_async(A, B, D, p, stream=second, **kw)
        seen = False
    except mmp.MmpError as e:
        seen = "EHIP" in str(e)
    seen = hip.hipGetLastError() != 0 or seen
    torch.cuda.synchronize()
    assert seen
    mmp.mm_modp_async(A, B, D, p, stream=second, **kw)
    torch.cuda.synchronize()
    assert torch.equal(C, want) and torch.equal(D, want)
