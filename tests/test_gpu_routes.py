"""Which kernels a call runs on, where the plan alone does not say (the launch phases do)."""
import sys

import numpy as np
import pytest

import mmp_inputs as gen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
mmp = pytest.importorskip("paper_2601_07508_amd")


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


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float64)).cuda()


def test_strict_reductions_keep_fp64_words():
    # planned on FP64 words, estimated faster on INT8 words: an option that asks for
    # the words' complete reductions is not passed over
    p, m, n, k = 1125899906842597, 300, 333, 800
    assert mmp.plan(p, m, n, k, strict_fmod=True)["form"] == mmp.FORM_FP64_WORDS
    A, B = gen.random_matrix(1, 1, m, k, p), gen.random_matrix(1, 2, k, n, p)
    dA, dB, C = dev(A), dev(B), torch.empty((m, n), dtype=torch.float64, device="cuda")
    want = oracle.mm_modp(p, A, B).astype(np.float64)
    for strict in (False, True):
        C.fill_(-1.0)
        say("strict", strict)
        phases = timed(lambda: mmp.mm_modp_async(dA, dB, C, p, strict_fmod=strict))
        assert ("fp64_words" in phases) == strict, phases
        assert np.array_equal(C.cpu().numpy(), want)


P_MAX = (1 << 52) // 3


def wide_primes(count):
    out, x = [], P_MAX + 1
    while len(out) < count:
        x = gen.prev_prime(x)
        out.append(x)
    return out


# the contraction from 5 moduli on, up to 48 and while their constants' digits fit the
# kernel arguments (48 of the job's primes do, 43 of the widest too, 44 do not); any entries
@pytest.mark.parametrize("moduli,contraction", [
    (gen.crt_primes(count=4), False), (gen.crt_primes(count=5), True), (wide_primes(8), True), (wide_primes(9), True),
    (wide_primes(40), True), (gen.crt_primes(count=48), True), (gen.crt_primes(count=49), False),
    (wide_primes(43), True), (wide_primes(44), False), ([2, 3, 5, 7, 11], True),
], ids=lambda v: f"{len(v)}x{max(v).bit_length()}b" if isinstance(v, list) else str(v))
@pytest.mark.parametrize("m,n", [(1, 1), (65, 33)])
def test_reconstruction_route(moduli, contraction, m, n):
    # one integer in every entry: 1, then M - 1
    M = 1
    for q in moduli:
        M *= q
    say("reconstruction", len(moduli), m, n)
    for X in (1, M - 1):
        R = [torch.full((m, n), float(X % q), dtype=torch.float64, device="cuda") for q in moduli]
        out = []
        phases = timed(lambda: out.append(mmp.crt_reconstruct(R, moduli)))
        assert ("crt_reconstruct" in phases) == contraction, phases
        limbs = out[0].cpu().numpy().view(np.uint64)
        for w in range(limbs.shape[0]):
            assert (limbs[w] == np.uint64((X >> (64 * w)) & ((1 << 64) - 1))).all()


# the residue form's conversion of integers, rows of A and of B further apart than they
# are long and starting anywhere on 8 bytes
@pytest.mark.parametrize("m,n,k,bits,count,pa,pb,shift", [
    (300, 200, 1000, 62, 6, 3, 5, 1), (130, 257, 520, 62, 3, 1, 2, 0), (64, 48, 30000, 60, 3, 7, 0, 1),
    (96, 80, 70001, 20, 3, 0, 9, 3),
])
def test_multi_modular_strides(m, n, k, bits, count, pa, pb, shift):
    primes = gen.crt_primes(count=count)
    A = gen.uniform_bits(m, 1, m * k, bits).reshape(m, k)
    B = gen.uniform_bits(n, 2, k * n, bits).reshape(k, n)

    def strided(x, pad):
        rows, cols = x.shape
        flat = torch.full((rows * (cols + pad) + shift,), -1, dtype=torch.int64, device="cuda")
        view = flat[shift:].view(rows, cols + pad)[:, :cols]
        view.copy_(torch.from_numpy(x.astype(np.int64)))
        return view

    dA, dB = strided(A, pa), strided(B, pb)
    outs = [torch.full((m, n), -1.0, dtype=torch.float64, device="cuda") for _ in primes]
    say("multi-modular strides", m, n, k, pa, pb, shift)
    phases = timed(lambda: mmp.mm_modp_crt(dA, dB, primes, outs, bits))
    assert "rns_crt_combine" in phases, phases
    for p, C in zip(primes, outs):
        assert np.array_equal(C.cpu().numpy(), oracle.mm_modp(p, A, B).astype(np.float64)), p
