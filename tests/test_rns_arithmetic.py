"""The residue form's arithmetic, emulated exactly: reductions modulo the
one-byte moduli without a conversion, and the recombination modulo p."""
import math
from fractions import Fraction

import numpy as np
import pytest

MODULI = [256, 255, 253, 251, 247, 241, 239, 233, 229, 227, 223, 217, 211, 199, 197, 193, 191, 181, 179, 173]


def test_moduli_are_pairwise_coprime():
    for i, a in enumerate(MODULI):
        for b in MODULI[:i]:
            assert math.gcd(a, b) == 1


def _inverse_bits(m):
    """fl(1/m) in binary32 as an integer over 2^31 (exact for m <= 256)."""
    v = float(np.float32(1.0) / np.float32(m)) * 2.0**31
    assert v == int(v)
    return int(v)


def _residues(y, m, first):
    """Low bytes of y - c m as the kernels form them: O the first multiple of
    256 m from `first` on, c from one fma of the binary32 O + y."""
    O = -(-first // (256 * m)) * (256 * m)
    F = O + y
    assert F.min() >= 2**23 and F.max() < 2**24  # one ulp is 1: O + y is exact
    magic = 12582912 - O // m
    assert 2**22 <= magic < 2**24
    # fma: F inv + magic rounded to nearest even; results lie in [2^23, 2^24)
    t = F * _inverse_bits(m) + (magic << 31)
    q, r = t >> 31, t & (2**31 - 1)
    q = q + ((r > 2**30) | ((r == 2**30) & (q & 1 == 1)))
    assert q.min() >= 2**23 and q.max() < 2**24
    bits = 0x4B000000 + (F - 2**23)         # pattern of F
    low24 = (0x4B000000 + (q - 2**23)) & 0xFFFFFF  # low 24 bits of the quotient's pattern, positive as int24
    assert low24.max() < 2**23
    low = (bits - low24 * m) & 0xFF
    return np.where(low >= 128, low - 256, low)


@pytest.mark.parametrize("m", MODULI)
def test_conversion_residues(m):
    y = np.arange(-(2**17), 2**17 + 1, dtype=np.int64)
    r = _residues(y, m, 2**23 + 2**17)
    assert ((r - y) % m == 0).all()


@pytest.mark.parametrize("m", MODULI)
def test_product_residues(m):
    # y = hi (2^16 mod m) + lo for hi <= 2^15, lo < 2^16
    w = 65536 % m
    top = 2**15 * w + 65535
    assert top < 2**23 - 2**16
    y = np.arange(0, top + 1, dtype=np.int64)
    r = _residues(y, m, 2**23)
    assert ((r - y) % m == 0).all()
    # the accumulator's bounds: 1024 stages of 64 terms about the bias
    bias = (1 << 30) // m * m
    lo, hi = bias - 65536 * 128 * 127, bias + 65536 * 128 * (128 if m == 256 else 127)
    assert lo >= 0 and hi <= 2**31


def _count(log2_bound):
    total = 0.0
    for n, m in enumerate(MODULI, 1):
        total += math.log2(m)
        if total >= log2_bound + 1.05:
            return n


def _exact(f):
    """A binary64 value that must be an exact integer below 2^53."""
    assert f == int(f) and abs(f) <= 2**53
    return int(f)


def _reduce_near(x, p, q):
    c = math.floor(float(Fraction(x) * Fraction(q) + Fraction(1, 2)))
    return x - c * p


@pytest.mark.parametrize("p", [65537, 16777213, 4294967291, 68719476731, 1125899906842597, 4503599627370449])
@pytest.mark.parametrize("k", [64, 65536, 1 << 20])
@pytest.mark.parametrize("splits", [1, 64])
def test_recombination(p, k, splits):
    half = p // 2
    n = _count(math.log2(k) + 2 * math.log2(half))
    ms = MODULI[:n]
    M = math.prod(ms)
    assert M > 2 * k * half * half
    q = 1.0 / p
    inv, W = [], []
    for m in ms:
        i = pow(M // m, -1, m)
        i = i - m if 2 * i > m else i
        inv.append(i)
        w = i * (M // m) % p
        W.append(w - p if w > half else w)
    Mp = M % p
    Mp = Mp - p if Mp > half else Mp
    hi_lo = [(w >> 26, w - ((w >> 26) << 26)) for w in W]
    mh, ml = Mp >> 26, Mp - ((Mp >> 26) << 26)
    rng = np.random.default_rng(p % 1000 + k % 97)
    top = k * half * half
    cases = [0, 1, -1, top, -top, top - 1, p, -p] + [int(rng.integers(-2**62, 2**62)) * top // 2**62 for _ in range(40)]
    for X in cases:
        # residues within [-128, 127], summed over k-ranges: any representative splits adds up to
        r = []
        for m in ms:
            base = X % m
            base = base - m if base > 127 else base
            r.append(base + m * int(rng.integers(-(splits - 1) // 2, splits // 2 + 1)) if splits > 1 else base)
            assert abs(r[-1]) <= 2**13 + 128
        hi = lo = 0
        g = 0.0
        for t, m in enumerate(ms):
            hi = _exact(float(hi + r[t] * hi_lo[t][0]))
            lo = _exact(float(lo + r[t] * hi_lo[t][1]))
            g = float(Fraction(g) + Fraction(r[t]) * Fraction(inv[t] / m))
        h = round(g)
        assert X == sum(x * i * (M // m) for x, i, m in zip(r, inv, ms)) - h * M
        H, L = _exact(float(hi - h * mh)), _exact(float(lo - h * ml))
        a = _reduce_near(H, p, q)
        assert abs(a) <= half + 2
        b = _reduce_near((1 << 26) * a, p, q)
        assert abs(b) <= half + 2
        t = _exact(float(b + L))
        d = t - math.floor(float(t) * q) * p
        d = d - p if d >= p else d
        d = d + p if d < 0 else d
        assert d == X % p
