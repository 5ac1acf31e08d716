"""The arithmetic of the E2M3 path (residue pass and products) modelled on the
host, for every FP8 modulus: the FP64 steps that reduce large integers, the
FP16 digit splits, the folds between passes and the final symmetric residue."""
from fractions import Fraction

import numpy as np
import pytest

from oracle import ozaki2_ref as ref


def _moduli():
    return sorted({(p, kind, s) for name in ("hybrid", "karatsuba")
                   for p, kind, s in ref.moduli_table(33, name)})


def _sym(v, p):
    h = p // 2
    return (v + h) % p - h


def _f16_fma(a, b, c):
    # FP16 fused multiply-add: operands exact in float64, products of 22 bits, one rounding
    return np.float16(np.asarray(a, np.float64) * np.asarray(b, np.float64) + np.float64(c))


@pytest.mark.parametrize("p,kind,s", _moduli())
def test_fp16_digit_split(p, kind, s):
    u = np.arange(-(p // 2), p // 2 + 1)          # an even p's residues include +p/2
    h = u.astype(np.float16)
    assert np.array_equal(h.astype(np.int64), u)
    rint = lambda x, m: np.float16(_f16_fma(x, m, 1536).astype(np.float64) - 1536)
    if kind == "square":
        x1 = rint(h, np.float16(np.float32(1) / np.float32(s)))
        x2 = _f16_fma(np.float16(-s), x1, h)
        digits = (x1, x2)
    else:
        t = np.float16(h.astype(np.float64) + np.where(np.signbit(h), -7.5, 7.5))
        x1 = rint(t, np.float16(1 / 16))
        x2 = _f16_fma(np.float16(-16), x1, h)
        digits = (x1, x2, np.float16(x1 + x2))
    a, b = x1.astype(np.int64), x2.astype(np.int64)
    assert np.array_equal(s * a + b, u)
    assert all(np.abs(d.astype(np.int64)).max() <= 16 for d in digits)


def _fma(a, b, c):
    """a b + c with one rounding, from exact rationals."""
    return float(Fraction(a) * Fraction(b) + Fraction(c))


@pytest.mark.parametrize("pair", [(1089, 1024), (529, 511), (513, 512), (1089, 1)])
def test_fp64_steps_of_large_integers(pair):
    # integers F 2^t as the residue pass forms them, up to its largest exponent
    R = pair[0] * pair[1]
    rng = np.random.default_rng(R)
    inv = 1.0 / float(R)
    for e in (55, 56, 80, 105, 106, 159):
        steps = 1 if e <= 55 else 2 if e <= 105 else 4
        for _ in range(200):
            F = int(rng.integers(2 ** 52, 2 ** 53))
            X = F << (e - 45) if e > 45 else F >> (45 - e)
            x = float(X)
            assert int(x) == X and X < 2 ** (e + 8)
            for _ in range(steps):
                q = float(np.rint(x * inv))
                y = _fma(-q, float(R), x)
                assert Fraction(y) == Fraction(x) - Fraction(q) * R    # exact
                x = y
            assert (int(x) - X) % R == 0
            assert abs(x) <= R / 2 + 2 ** 12
            f = np.float32(x)
            assert float(f) == x
            p = pair[0]
            u = float(f) - p * float(np.rint(f * (np.float32(1) / np.float32(p))))
            assert abs(u) <= p // 2 and (int(u) - X) % p == 0


def _reduce(x, q):
    """x - rint(x / q) q as the products do it: x in units of 1/64, FP32."""
    x64 = (x / 64.0).astype(np.float32)
    inv = np.float32(np.float32(1) / np.float32(q)) * np.float32(64)
    t = np.rint(x64 * inv).astype(np.float64)
    r = x64.astype(np.float64) - t * (q / 64.0)
    assert np.array_equal(r, r.astype(np.float32))       # one exact fused multiply-add
    return r * 64.0


def _values(limit, q):
    rng = np.random.default_rng(q)
    near = (np.arange(-2000, 2000)[:, None] * q + np.arange(-1, 2)[None, :] + q // 2).ravel()
    far = rng.integers(-limit, limit + 1, 1 << 16)
    edge = np.concatenate([np.arange(limit - 3000, limit + 1), -np.arange(limit - 3000, limit + 1)])
    v = np.concatenate([near, far, edge])
    return v[np.abs(v) <= limit]


@pytest.mark.parametrize("p,kind,s", _moduli())
def test_folds_and_symmetric_residue(p, kind, s):
    if kind == "square":
        muls, last = [(s, s)], 1
    else:
        i = lambda v: pow(v % p, -1, p)
        sym = lambda v: int(_sym(np.int64(v), p))
        if np.gcd(p, 15) == 1:
            a, b, last = sym(15), sym(-16 * i(15)), sym(-15)
        else:
            a, b, last = sym(-16), sym(-15 * i(16)), sym(16)
        muls = [(p, a), (p, b)]
    for q, m in muls:
        x = _values(2 ** 24 if kind == "square" else 2 ** 23 + 2 ** 17, q)
        r = _reduce(x, q)
        assert np.all(np.mod(r - x, q) == 0)
        y = r * m
        assert np.all(np.abs(y) <= 2 ** 17)              # + 2^23 stays below 2^24
        assert np.array_equal(y / 64, (y / 64).astype(np.float32))
    x = _values(2 ** 23 + 2 ** 17, p)
    y = (_reduce(x, p) * last).astype(np.float32)
    inv = np.float32(1) / np.float32(p)
    bias = np.float32(0.25) * inv
    # fused multiply-add, then rint
    t = np.rint((y.astype(np.float64) * np.float64(inv) + np.float64(bias)).astype(np.float32))
    z = y.astype(np.float64) - t.astype(np.float64) * p
    assert np.array_equal(z.astype(np.int64), _sym(x * last, p))


@pytest.mark.parametrize("p,kind,s", _moduli())
def test_short_sums_in_one_step(p, kind, s):
    # up to k = 8192 (squares) and 256 (Karatsuba) the result takes one step from
    # the accumulator times its multiplier; up to 3840 Karatsuba's first fold
    # only multiplies
    if kind == "square":
        last, limit = 1, (s // 2) ** 2 * 8192 + s * (s // 2 + 2)
    else:
        i = lambda v: pow(v % p, -1, p)
        sym = lambda v: int(_sym(np.int64(v), p))
        if np.gcd(p, 15) == 1:
            a, b, last = sym(15), sym(-16 * i(15)), sym(-15)
        else:
            a, b, last = sym(-16), sym(-15 * i(16)), sym(16)
        assert (abs(a) + 1) * 256 * 3840 < 2 ** 24
        x = _values((abs(a) + 1) * 256 * 256, p)
        assert np.abs(_reduce(x, p)).max() <= p // 2
        limit = 256 * 256 + abs(b) * (p // 2)
    x = _values(limit, p)
    halves = (np.arange(max(0, limit // p - 3000), limit // p)[:, None] * p + np.arange(-2, 3)
              + p // 2).ravel()
    x = np.concatenate([x, halves, -halves])
    x = x[np.abs(x) <= limit]
    y = (x * last).astype(np.float32)
    assert np.array_equal(y.astype(np.int64), x * last)
    inv = np.float32(1) / np.float32(p)
    bias = np.float32(0.25) * inv
    t = np.rint((y.astype(np.float64) * np.float64(inv) + np.float64(bias)).astype(np.float32))
    z = y.astype(np.float64) - t.astype(np.float64) * p
    assert np.array_equal(z.astype(np.int64), _sym(x * last, p))


def test_int8_fp64_residues():
    # the products' epilogue: one FP64 step on an INT32 sum, the quotient nudged
    # by 1 / (4 p) so that an even p's half goes to -p / 2
    rng = np.random.default_rng(8)
    top = 2 ** 29 + 2 ** 22
    for p, _, _ in ref.moduli_table(33, "int8"):
        inv = 1.0 / float(p)
        x = np.concatenate([rng.integers(-top, top, 300), np.arange(-2 * p, 2 * p + 1),
                            [-top, top], p * rng.integers(0, top // p, 50) + p // 2])
        for v in x.tolist():
            q = np.rint(_fma(float(v), inv, 0.25 * inv))
            assert _fma(-q, float(p), float(v)) == _sym(v, p), (p, v)


@pytest.mark.parametrize("k", [300, 3840, 4096, 32768, 65536, 98304, 131072, 2 ** 18])
@pytest.mark.parametrize("p,kind,s", _moduli())
def test_sums_of_chunked_passes(p, kind, s, k):
    # A list item's three passes: chunks of 2^15, each but the last reduced modulo
    # p, the last one by the pass's own fold.  Digit products of +-256 throughout
    # (and +-255, for odd sums) keep every FP32 sum at most 2^24 and the residue
    # exact.
    chunk = 2 ** 15
    last = 1
    if kind == "square":
        folds = [(p if k > chunk else 0, 1), (s, s), (p if k > 8192 else 0, 1)]
    else:
        i = lambda v: pow(v % p, -1, p)
        sym = lambda v: int(_sym(np.int64(v), p))
        if np.gcd(p, 15) == 1:
            a, b, last = sym(15), sym(-16 * i(15)), sym(-15)
        else:
            a, b, last = sym(-16), sym(-15 * i(16)), sym(16)
        folds = [(p if k > 3840 else 0, a), (p, b), (p if k > 256 else 0, 1)]
    for prods in [(256, 256, 256), (-256, -256, 256), (255, 256, -255), (256, -255, 256)]:
        acc, exact, top = np.float32(0), 0, 0
        for (q, m), d in zip(folds, prods):
            left = k
            while left:
                n = min(left, chunk)
                # whole chunk at once: the sums on the way lie between its ends
                top = max(top, abs(int(acc)), abs(int(acc) + n * d))
                acc = np.float32(np.float64(acc) + n * d)
                left -= n
                r = q if left == 0 else p
                if r:
                    acc = np.float32(_reduce(np.array([acc], np.float64), r)[0])
            acc = np.float32(acc * np.float32(m))
            # (s X only counts modulo p)
            exact = (exact + k * d) * m % p
        assert top <= 2 ** 24
        assert (int(acc) * last - exact * last) % p == 0
