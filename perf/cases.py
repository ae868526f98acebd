"""The work that a user of this library has it do, as cases that can be timed.

Each case is one call (or one burst of requests) through the library's Python
entry points, on inputs in device memory.  The sizes are those of the
library's own workloads (the square, tall-skinny, inner-product, unbalanced,
multi-modular, batched and served products) and generic ones around them.
"""

from __future__ import annotations

import math
import random

import torch

import paper_2601_07508_amd as mmp

# ------------------------------------------------------------------ the cases


def listed():
    return [
        # the smallest calls: a ragged block of a blocked algorithm, where launches are most of the time
        dict(name="small_96x80x200_b36", kind="product", m=96, n=80, k=200, bits=36),
        # one binary64 word per entry, the classic small-prime product (Section 2's setting)
        dict(name="sq512_b25_uv11", kind="product", m=512, n=512, k=512, bits=25, u=1, v=1),
        # a square product at a mid-size prime, forms and words left to the planner
        dict(name="sq4096_b36", kind="product", m=4096, n=4096, k=4096, bits=36),
        # the benchmark's default: near-full-mantissa primes on binary64 words
        dict(name="sq8192_b50_uv22", kind="product", m=8192, n=8192, k=8192, bits=50, u=2, v=2),
        # a large product of odd sizes at the same primes, left to the planner
        dict(name="ragged_6001x5003x7013_b50", kind="product", m=6001, n=5003, k=7013, bits=50),
        # outer-product-heavy: the update of a blocked elimination (short k, a large result)
        dict(name="tall16384x256_b23", kind="product", m=16384, n=16384, k=256, bits=23),
        # inner-product-heavy: Gram matrices and projections at the widest primes
        dict(name="inner512x131072_b52", kind="product", m=512, n=512, k=131072, bits=52),
        # the iterated product of block Wiedemann: a fixed A whose digit planes the program keeps
        dict(name="unbal10923x32768x32_b36_kept", kind="product", m=10923, n=32, k=32768, bits=36, kept_a=True),
        # one integer pair against many primes
        dict(name="crt2048_b60_32p", kind="crt", m=2048, n=2048, k=2048, entry_bits=60, primes=32),
        # integers from their residues
        dict(name="reconstruct2048_32p", kind="reconstruct", m=2048, n=2048, primes=32),
        # many uneven products at once, each with its own prime
        dict(name="batch32_64to4096", kind="batch", count=32, lo=64, hi=4096, mix=1),
        # a burst of mixed requests on the server
        dict(name="serve24_64to2048", kind="serve", count=24, lo=64, hi=2048, mix=2),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the ranges above; never dearer than the 8192^3 one."""
    kind = rng.choice(["product"] * 6 + ["words"] * 2 + ["crt", "crt", "reconstruct", "reconstruct", "batch", "serve"])
    while True:
        if kind == "product":
            shape = rng.choice(["any", "any", "square", "tall", "inner", "narrow"])
            if shape == "any":
                m, n, k = (_log_int(rng, 64, 8192) for _ in range(3))
            elif shape == "square":
                m = n = k = _log_int(rng, 64, 8192)
            elif shape == "tall":
                m, n, k = _log_int(rng, 4096, 16384), _log_int(rng, 4096, 16384), _log_int(rng, 32, 512)
            elif shape == "inner":
                m, n, k = _log_int(rng, 64, 768), _log_int(rng, 64, 768), _log_int(rng, 16384, 131072)
            else:
                m, n, k = _log_int(rng, 2048, 16384), _log_int(rng, 8, 64), _log_int(rng, 4096, 32768)
            case = dict(kind="product", m=m, n=n, k=k, bits=rng.randint(20, 52))
            if shape == "narrow":
                case["kept_a"] = rng.random() < 0.5
        elif kind == "words":  # binary64 words, with the longer-block options a caller may choose
            m, n, k = (_log_int(rng, 64, 4096) for _ in range(3))
            case = dict(kind="product", m=m, n=n, k=k, bits=rng.randint(20, 52), words=True)
            option = rng.choice(["", "", "extended_block", "centered_words"])
            if option:
                case[option] = True
        elif kind == "crt":
            m, n, k = (_log_int(rng, 64, 3072) for _ in range(3))
            case = dict(kind="crt", m=m, n=n, k=k, entry_bits=rng.randint(16, 62), primes=_log_int(rng, 3, 48))
        elif kind == "reconstruct":
            case = dict(kind="reconstruct", m=_log_int(rng, 64, 4096), n=_log_int(rng, 64, 2048),
                        primes=_log_int(rng, 3, 48))
        elif kind == "batch":
            case = dict(kind="batch", count=_log_int(rng, 4, 64), lo=64, hi=_log_int(rng, 512, 4096),
                        mix=rng.randint(10, 10**6))
        else:
            case = dict(kind="serve", count=_log_int(rng, 4, 32), lo=64, hi=_log_int(rng, 512, 2048),
                        mix=rng.randint(10, 10**6))
        w = work(case)
        if w["flops"] <= 1e12 and w["bytes"] <= 6e9:
            return case


# ------------------------------------------------------------------ primes and shapes


def _is_prime(n):
    if n < 2:
        return False
    bases = (2, 3, 5, 7, 11, 13, 17, 19, 23, 29, 31, 37)
    for b in bases:
        if n % b == 0:
            return n == b
    d, s = n - 1, 0
    while d % 2 == 0:
        d, s = d // 2, s + 1
    for a in bases:
        x = pow(a, d, n)
        if x in (1, n - 1):
            continue
        for _ in range(s - 1):
            x = x * x % n
            if x == n - 1:
                break
        else:
            return False
    return True


def _prime_below(x):
    x -= 1
    while not _is_prime(x):
        x -= 1
    return x


def _many_primes(count):
    """Distinct primes of 31 to 50 bits, the multi-modular product's."""
    rng, out = random.Random(20260107), []
    while len(out) < count:
        b = 31 + len(out) % 20
        q = _prime_below((1 << (b - 1)) + rng.randrange(1 << 20, 1 << (b - 1)))
        if q not in out:
            out.append(q)
    return out


def _mixed_jobs(case):
    """(m, n, k, p) of a mixed batch: sizes log-uniform, primes of 20 to 52 bits."""
    rng = random.Random(case["mix"])
    out = []
    for _ in range(case["count"]):
        m, n, k = (_log_int(rng, case["lo"], case["hi"]) for _ in range(3))
        out.append((m, n, k, _prime_below(1 << rng.randint(20, 52))))
    return out


def _limbs(primes):
    M = 1
    for q in primes:
        M *= q
    return ((M - 1).bit_length() + 63) // 64


# ------------------------------------------------------------------ inputs


def _uniform(gen, rows, cols, bound):
    return torch.randint(0, bound, (rows, cols), generator=gen, dtype=torch.int64, device="cuda")


def _inputs(case, seed):
    """The case's matrices as int64, from the seed alone."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    if case["kind"] == "product":
        p = _prime_below(1 << case["bits"])
        return p, _uniform(gen, case["m"], case["k"], p), _uniform(gen, case["k"], case["n"], p)
    if case["kind"] == "crt":
        top = 1 << case["entry_bits"]
        return (_many_primes(case["primes"]), _uniform(gen, case["m"], case["k"], top),
                _uniform(gen, case["k"], case["n"], top))
    if case["kind"] == "reconstruct":
        primes = _many_primes(case["primes"])
        # residues of a uniform integer below the primes' product are independent and uniform
        return primes, [_uniform(gen, case["m"], case["n"], q) for q in primes]
    return [(p, _uniform(gen, m, k, p), _uniform(gen, k, n, p)) for m, n, k, p in _mixed_jobs(case)]


class _Serving:
    """A server that is closed with the state that holds it."""

    def __init__(self):
        self.server = mmp.Server(hbm_budget=64 << 30, max_slots=64)

    def __del__(self):
        self.server.close()


def prepare(case, seed):
    kind = case["kind"]
    if kind == "product":
        p, A, B = _inputs(case, seed)
        opts = {o: True for o in ("extended_block", "centered_words") if case.get(o)}
        if case.get("words"):
            opts["form"] = mmp.FORM_FP64_WORDS
        state = dict(kind=kind, p=p, A=A.double(), B=B.double(), u=case.get("u", 0), v=case.get("v", 0), opts=opts)
        if case.get("kept_a"):
            opts["prepared_a"] = mmp.prepare_operand(state["A"], p, 0)
        return state
    if kind == "crt":
        primes, A, B = _inputs(case, seed)
        return dict(kind=kind, primes=primes, A=A, B=B, bits=case["entry_bits"])
    if kind == "reconstruct":
        primes, R = _inputs(case, seed)
        return dict(kind=kind, primes=primes, R=[r.double() for r in R])
    jobs = []
    for p, A, B in _inputs(case, seed):
        C = torch.empty((A.shape[0], B.shape[1]), dtype=torch.float64, device="cuda")
        jobs.append((A.double(), B.double(), C, p, 0, 0))
    state = dict(kind=kind, jobs=jobs)
    if kind == "serve":
        state["serving"] = _Serving()
    return state


def run(state):
    kind = state["kind"]
    if kind == "product":
        return mmp.mm_modp(state["A"], state["B"], state["p"], state["u"], state["v"], **state["opts"])
    if kind == "crt":
        A, B = state["A"], state["B"]
        outs = [torch.empty((A.shape[0], B.shape[1]), dtype=torch.float64, device="cuda") for _ in state["primes"]]
        mmp.mm_modp_crt(A, B, state["primes"], outs, state["bits"])
        return outs
    if kind == "reconstruct":
        return mmp.crt_reconstruct(state["R"], state["primes"])
    if kind == "batch":
        mmp.mm_modp_batched(state["jobs"])
    else:
        server = state["serving"].server
        tickets = [server.submit(A, B, C, p, u, v) for A, B, C, p, u, v in state["jobs"]]
        for t in tickets:
            server.wait(t)
    return [j[2] for j in state["jobs"]]


# ------------------------------------------------------------------ what a pass cannot do without


def work(case):
    kind = case["kind"]
    if kind == "product":
        m, n, k = case["m"], case["n"], case["k"]
        a = (case["bits"] + 7) // 8 if case.get("kept_a") else 8  # bytes an entry of A
        return dict(bytes=a * m * k + 8 * (k * n + m * n), flops=2 * m * n * k)
    if kind == "crt":
        m, n, k = case["m"], case["n"], case["k"]
        # the integer product once, one reduction an output and prime
        return dict(bytes=8 * (m * k + k * n + case["primes"] * m * n), flops=2 * m * n * (k + case["primes"]))
    if kind == "reconstruct":
        mn, primes = case["m"] * case["n"], _many_primes(case["primes"])
        # one multiply-add an entry, prime and limb
        return dict(bytes=8 * mn * (len(primes) + _limbs(primes)), flops=2 * mn * len(primes) * _limbs(primes))
    jobs = _mixed_jobs(case)
    return dict(bytes=sum(8 * (m * k + k * n + m * n) for m, n, k, _ in jobs),
                flops=sum(2 * m * n * k for m, n, k, _ in jobs))


# ------------------------------------------------------------------ exact results in 64 bits


def _exact_product(A, B, p):
    """A B mod p of int64 matrices with entries in [0, p), p < 2^52: products
    of 17-bit limbs, exact in binary64 for k <= 2^19, recombined in int64."""
    w = 17
    limbs = max(1, (p.bit_length() + w - 1) // w)
    mask = (1 << w) - 1
    As = [((A >> (w * i)) & mask).double() for i in range(limbs)]
    Bs = [((B >> (w * i)) & mask).double() for i in range(limbs)]
    acc = None
    for s in range(2 * limbs - 2, -1, -1):
        if acc is not None:  # times 2^17, in two steps below 2^63
            acc = ((acc << 10) % p << 7) % p
        for i in range(max(0, s - limbs + 1), min(s, limbs - 1) + 1):
            t = (As[i] @ Bs[s - i]).long() % p
            acc = t if acc is None else (acc + t) % p
    return acc.double()


def _mulmod(x, y, p):
    """x y mod p for int64 tensors below p < 2^52: a binary64 quotient, then
    the remainder from the products' low 64 bits."""
    q = (x.double() * float(y) / float(p)).long()
    r = x * y - q * p  # wraps, but the true value is small
    return torch.remainder(r, p)


def _exact_reconstruct(R, primes):
    """Garner's mixed-radix digits, then Horner in 24-bit pieces."""
    v = []
    for j, p in enumerate(primes):
        t, weight = R[j], 1  # (r_j - sum_i v_i prod_{h<i} p_h) / prod_{h<j} p_h mod p_j
        for i in range(j):
            t = torch.remainder(t - _mulmod(torch.remainder(v[i], p), weight, p), p)
            weight = weight * primes[i] % p
        v.append(_mulmod(t, pow(weight, -1, p), p) if j else t)
    limbs, piece, mask = _limbs(primes), 24, (1 << 24) - 1
    count = (64 * limbs + piece - 1) // piece
    acc = [torch.zeros_like(v[0]) for _ in range(count)]
    for i in range(len(primes) - 1, -1, -1):
        parts = [(primes[i] >> (piece * h)) & mask for h in range(3)]
        new, carry = [], torch.zeros_like(v[0])
        for c in range(count):
            t = carry + ((v[i] >> (piece * c)) & mask if c < 3 else 0)
            for h in range(3):
                if c >= h and parts[h]:
                    t = t + acc[c - h] * parts[h]
            new.append(t & mask)
            carry = t >> piece
        acc = new
    out = []
    for w in range(limbs):
        word = torch.zeros_like(v[0])
        for c in range(count):
            shift = piece * c - 64 * w
            if -piece < shift < 64:
                word = word | (acc[c] << shift if shift >= 0 else acc[c] >> -shift)
        out.append(word)
    return torch.stack(out)


def exact(case, seed):
    kind = case["kind"]
    if kind == "product":
        p, A, B = _inputs(case, seed)
        return _exact_product(A, B, p)
    if kind == "crt":
        primes, A, B = _inputs(case, seed)
        return [_exact_product(A % q, B % q, q) for q in primes]
    if kind == "reconstruct":
        primes, R = _inputs(case, seed)
        return _exact_reconstruct(R, primes)
    return [_exact_product(A, B, p) for p, A, B in _inputs(case, seed)]
