"""GPU parity of the INT8 product's residue form against the exact oracle
(tolerance 0), at the edges of its tiles, k-ranges and int32 range.

Products large enough for the planner to take the form; the launch phases say
that it ran.
"""
import sys

import numpy as np
import pytest

import mmp_inputs as gen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
mmp = pytest.importorskip("paper_2601_07508_amd")

P52, P31, P50 = 4503599627370449, 2147483647, 1125899906842597


def say(*a):
    print(*a, file=sys.stderr, flush=True)


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def timed(call):
    """The launch phases of one call."""
    mmp.timers_read(reset=True)
    mmp.timers_enable(True)
    call()
    torch.cuda.synchronize()
    mmp.timers_enable(False)
    return mmp.timers_read(reset=True)


def strided(x, pad, shift):
    """A device copy of x with leading dimension cols + pad, `shift` entries into its storage."""
    rows, cols = x.shape
    flat = torch.full((rows * (cols + pad) + shift + 1,), float("nan"), dtype=torch.float64, device="cuda")
    view = flat[shift:shift + rows * (cols + pad)].view(rows, cols + pad)[:, :cols]
    view.copy_(torch.from_numpy(x.astype(np.float64)))
    return view


# tile edges (128 and 256), 16-row blocks, 64-k stages, 4-stage ring, one digit-count
# boundary and p on both sides of 2^31 (the one- and two-word conversions)
@pytest.mark.parametrize("p,m,n,k,pad,shift", [
    (P52, 512, 512, 2048, 0, 0), (P52, 513, 511, 2049, 1, 1), (P50, 257, 640, 3073, 0, 1), (P52, 255, 257, 4159, 3, 0),
    (P52, 385, 1025, 1985, 2, 0), (P31, 2561, 2545, 4033, 1, 0), (8589934583, 1537, 2050, 2111, 0, 0),
    (P52, 1040, 2064, 1088, 5, 1),
])
def test_edges(p, m, n, k, pad, shift):
    A = gen.random_matrix(m, 1, m, k, p)
    B = gen.random_matrix(n, 2, k, n, p)
    say("residue form", p, m, n, k, pad, shift)
    dA, dB = strided(A, pad, shift), strided(B, pad, shift)
    store = torch.full((m + 1, n + pad), -1.0, dtype=torch.float64, device="cuda")
    phases = timed(lambda: mmp.mm_modp_async(dA, dB, store[:m, :n], p))
    assert "rns_gemm" in phases, phases
    got = store.cpu().numpy()
    want = oracle.mm_modp(p, A, B).astype(np.float64)
    assert np.array_equal(got[:m, :n], want) and not np.signbit(got[:m, :n]).any()
    assert (got[m:] == -1.0).all() and (got[:, n:] == -1.0).all()


@pytest.mark.parametrize("p,k", [(P52, 65536), (P52, 65600), (P31, 65536)])
def test_extreme_sums(p, k):
    # whole k-ranges of 1024 stages with every residue at an end of its range:
    # x = 128 makes the residue mod 256 -128 in every term; x = (p +- 1) / 2 is
    # the largest centered entry of either sign
    m, n = 2048, 2064
    for x, y in ((128, 128), ((p - 1) // 2, (p - 1) // 2), ((p - 1) // 2, (p + 1) // 2), (p - 128, 128)):
        say("extreme", p, k, x, y)
        A = torch.full((m, k), float(x), dtype=torch.float64, device="cuda")
        B = torch.full((k, n), float(y), dtype=torch.float64, device="cuda")
        C = torch.empty((m, n), dtype=torch.float64, device="cuda")
        phases = timed(lambda: mmp.mm_modp_async(A, B, C, p))
        assert "rns_gemm" in phases, phases
        assert bool((C == float(x * y * k % p)).all())


@pytest.mark.parametrize("n", [512, 770])
def test_long_k_ranges(n):
    # few tiles, long k: several k-ranges, the last one shorter
    p, m, k = P52, 260, 40000
    A = gen.random_matrix(8, 1, m, k, p)
    B = gen.random_matrix(9, 2, k, n, p)
    say("ranges", n)
    dA, dB = strided(A, 0, 0), strided(B, 0, 0)
    C = torch.empty((m, n), dtype=torch.float64, device="cuda")
    phases = timed(lambda: mmp.mm_modp_async(dA, dB, C, p))
    assert "rns_gemm" in phases, phases
    assert np.array_equal(C.cpu().numpy(), oracle.mm_modp(p, A, B).astype(np.float64))


def test_workspace_of_the_digit_planes_is_enough():
    # a caller workspace of the plan's size: too small for the residue planes,
    # so the digit form runs, with the same result
    p, m, n, k = P52, 512, 520, 2048
    A = gen.random_matrix(3, 1, m, k, p)
    B = gen.random_matrix(4, 2, k, n, p)
    dA, dB = strided(A, 0, 0), strided(B, 0, 0)
    ws = torch.empty(mmp.plan(p, m, n, k)["workspace_bytes"], dtype=torch.uint8, device="cuda")
    big = torch.empty(1 << 28, dtype=torch.uint8, device="cuda")
    want = oracle.mm_modp(p, A, B).astype(np.float64)
    for w, phase in ((ws, "int8_gemm"), (big, "rns_gemm")):
        C = torch.full((m, n), -1.0, dtype=torch.float64, device="cuda")
        phases = timed(lambda: mmp.mm_modp_async(dA, dB, C, p, workspace=w))
        assert phase in phases, phases
        assert np.array_equal(C.cpu().numpy(), want)
    C = torch.full((m, n), -1.0, dtype=torch.float64, device="cuda")
    phases = timed(lambda: mmp.mm_modp_static(dA, dB, C, p))
    assert "rns_gemm" in phases and np.array_equal(C.cpu().numpy(), want)


def test_captured_in_a_graph():
    p, m, n, k = P50, 640, 520, 1500
    dA = strided(gen.random_matrix(5, 1, m, k, p), 0, 0)
    dB = strided(gen.random_matrix(6, 2, k, n, p), 0, 0)
    C = torch.empty((m, n), dtype=torch.float64, device="cuda")
    ws = torch.empty(1 << 28, dtype=torch.uint8, device="cuda")
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    call = lambda: mmp.mm_modp_async(dA, dB, C, p, workspace=ws, stream=s)
    phases = timed(call)
    assert "rns_gemm" in phases, phases
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        call()
    for rep in range(3):
        A = gen.random_matrix(20 + rep, 1, m, k, p)
        B = gen.random_matrix(30 + rep, 2, k, n, p)
        dA.copy_(torch.from_numpy(A.astype(np.float64)))
        dB.copy_(torch.from_numpy(B.astype(np.float64)))
        C.fill_(-1.0)
        ws.zero_()
        say("replay", rep)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(C.cpu().numpy(), oracle.mm_modp(p, A, B).astype(np.float64))


def exact_mod(A, B, p):
    """A B mod p of Python-integer-sized entries, row by row (the oracle reduces them first)."""
    return oracle.mm_modp(p, A, B).astype(np.float64)


# limbs: one (8-bit entries) to several; a prime of 5 forces the narrow base;
# k beyond one int32 block of the digit form; more than 64 primes; odd and
# line-aligned leading dimensions
@pytest.mark.parametrize("m,n,k,bits,small,count,pad", [
    (130, 257, 520, 62, [], 3, 0), (300, 200, 1000, 62, [5, 7], 6, 1), (260, 140, 4000, 8, [], 3, 0),
    (64, 48, 30000, 60, [], 4, 0), (96, 80, 70000, 62, [11], 3, 1), (200, 144, 900, 33, [], 66, 0),
    (513, 257, 1400, 47, [], 9, 0), (100, 90, 140000, 20, [], 3, 0),
])
def test_multi_modular(m, n, k, bits, small, count, pad):
    primes = small + gen.crt_primes(count=count - len(small))
    A = gen.uniform_bits(m, 1, m * k, bits).reshape(m, k)
    B = gen.uniform_bits(n, 2, k * n, bits).reshape(k, n)
    A[0, :] = B[:, 0] = (1 << bits) - 1  # the largest sum
    A[1, :] = 0
    say("multi-modular", m, n, k, bits, count, pad)
    dA = torch.from_numpy(A.astype(np.int64)).cuda()
    dB = torch.from_numpy(B.astype(np.int64)).cuda()
    stores = [torch.full((m + 1, n + pad), -1.0, dtype=torch.float64, device="cuda") for _ in primes]
    outs = [s[:m, :n] for s in stores]
    phases = timed(lambda: mmp.mm_modp_crt(dA, dB, primes, outs, bits))
    say(sorted(phases))
    for p, s in zip(primes, stores):
        got = s.cpu().numpy()
        assert np.array_equal(got[:m, :n], exact_mod(A, B, p)), p
        assert (got[m:] == -1.0).all() and (got[:, n:] == -1.0).all()
    if (m, k) in ((130, 520), (300, 1000), (64, 30000), (96, 70000), (100, 140000)):
        assert "rns_crt_combine" in phases, phases


def batch_jobs(seed, count):
    """Uneven products: large and small tiles, one and several k-ranges, every conversion."""
    shapes = [(P52, 2060, 1800, 1500), (P50, 300, 200, 9000), (P31, 700, 1200, 900), (65537, 500, 260, 3000),
              (P52, 140, 129, 2100), (251, 70, 90, 100), (P50, 64, 1000, 65)]
    out = []
    for i in range(count):
        p, m, n, k = shapes[i] if i < len(shapes) else (P52, 33 + i, 65 - i // 2, 70 + i)
        A = gen.random_matrix(seed + i, 1, m, k, p)
        B = gen.random_matrix(seed + i, 2, k, n, p)
        C = torch.full((m, n + 1), -1.0, dtype=torch.float64, device="cuda")[:, :n]
        out.append((p, A, B, strided(A, i % 3, i % 2), strided(B, i % 2, 0), C))
    return out


def check_batch(items):
    for p, A, B, dA, dB, C in items:
        assert np.array_equal(C.cpu().numpy(), oracle.mm_modp(p, A, B).astype(np.float64)), (p, A.shape, B.shape)
        assert bool((C._base[:, -1] == -1.0).all())


def test_batch():
    items = batch_jobs(50, 70)  # more than one launch's table
    jobs = [(dA, dB, C, p, 0, 0) for p, A, B, dA, dB, C in items]
    jobs[4] = jobs[4][:4] + (2, 3)  # forced binary64 words keep their own launch
    say("residue batch")
    phases = timed(lambda: mmp.mm_modp_batched(jobs))
    assert phases["fp64_words"][0] == 1 and phases["rns_batch_convert"][0] >= 1, phases
    check_batch(items)
    # a workspace of the queried size, and one too small for the shared launches
    need = mmp.workspace_batched(jobs)
    own = sum(mmp.plan(j[3], *j[2].shape, j[0].shape[1], j[4], j[5], splits=1)["workspace_bytes"] + 256 for j in jobs)
    assert own < need
    for size, shared in ((need, True), (own, False)):
        for *_, C in items:
            C.fill_(-2.0)
        ws = torch.empty(size, dtype=torch.uint8, device="cuda")
        phases = timed(lambda: mmp.mm_modp_batched(jobs, workspace=ws))
        assert ("rns_batch_gemm" in phases) == shared, phases
        check_batch(items)


def test_small_batch_on_digits():
    items = batch_jobs(150, 10)[4:]
    jobs = [(dA, dB, C, p, 0, 0) for p, A, B, dA, dB, C in items]
    phases = timed(lambda: mmp.mm_modp_batched(jobs))
    assert set(phases) == {"int8_batch_digitize", "int8_batch_gemm"}, phases
    check_batch(items)


def test_batch_in_a_graph():
    items = batch_jobs(250, 9)
    jobs = [(dA, dB, C, p, 0, 0) for p, A, B, dA, dB, C in items]
    ws = torch.empty(mmp.workspace_batched(jobs), dtype=torch.uint8, device="cuda")
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    call = lambda: mmp.mm_modp_batched(jobs, workspace=ws, stream=s)
    assert "rns_batch_gemm" in timed(call)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        call()
    for rep in range(3):
        for *_, C in items:
            C.fill_(-2.0)
        ws.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        check_batch(items)


# AUTO calls that the plan gives to FP64 words and measured times to INT8 words: a
# short and a long k, odd strides, few digits, and (last) a small one that stays
@pytest.mark.parametrize("p,m,n,k,pad,form", [
    (P52, 3100, 2306, 37, 0, "int8"), (P52, 1031, 2306, 65, 1, "int8"), (137438953447, 139, 200, 1969, 0, "int8"),
    (P50, 300, 333, 800, 3, "int8"), (P31, 700, 1025, 333, 0, "int8"), (65537, 60, 70, 150, 0, "fp64_words"),
])
def test_faster_words(p, m, n, k, pad, form):
    plan = mmp.plan(p, m, n, k)
    assert plan["form"] == mmp.FORM_FP64_WORDS
    A = gen.random_matrix(m, 1, m, k, p)
    B = gen.random_matrix(n, 2, k, n, p)
    A[0, :] = B[:, 0] = p - 1
    say("faster words", p, m, n, k, pad)
    dA, dB = strided(A, pad, 0), strided(B, pad, 0)
    want = oracle.mm_modp(p, A, B).astype(np.float64)
    store = torch.full((m + 1, n + pad), -1.0, dtype=torch.float64, device="cuda")
    C = store[:m, :n]

    def run(call):
        store.fill_(-1.0)
        phases = timed(call)
        got = store.cpu().numpy()
        assert np.array_equal(got[:m, :n], want)
        assert (got[m:] == -1.0).all() and (got[:, n:] == -1.0).all()
        return "fp64_words" if "fp64_words" in phases else "int8"

    assert run(lambda: mmp.mm_modp_async(dA, dB, C, p)) == form
    big = torch.empty(1 << 26, dtype=torch.uint8, device="cuda")
    assert run(lambda: mmp.mm_modp_async(dA, dB, C, p, workspace=big)) == form
    # as planned: a workspace of the plan's size, the call without allocation, words
    # by name, and a capture (below)
    small = torch.empty(max(256, plan["workspace_bytes"]), dtype=torch.uint8, device="cuda")
    assert run(lambda: mmp.mm_modp_async(dA, dB, C, p, workspace=small)) == "fp64_words"
    assert run(lambda: mmp.mm_modp_static(dA, dB, C, p)) == "fp64_words"
    assert run(lambda: mmp.mm_modp_async(dA, dB, C, p, form=mmp.FORM_FP64_WORDS)) == "fp64_words"
    if plan["splits"] == 1:  # no workspace: a capture without one holds the FP64 launch alone
        s = torch.cuda.Stream()
        s.wait_stream(torch.cuda.current_stream())
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            mmp.mm_modp_async(dA, dB, C, p, stream=s)
        for _ in range(3):
            store.fill_(-1.0)
            torch.cuda.synchronize()
            g.replay()
            torch.cuda.synchronize()
            assert np.array_equal(store.cpu().numpy()[:m, :n], want)
