"""Line maxima and bound operands of whole lines through the C ABI: exponents,
flags, Abar and Bbar (fast mode: the norms' exponents) against the oracle at
the edges of the pass's tiles and on both sides of the rule that picks it, with
values that round at the E4M3 boundaries, subnormal lines and special values."""
import numpy as np
import pytest

from oracle import ozaki2_ref as ref

from gpu_util import run, same_bits

pytestmark = pytest.mark.gpu


def _operand(lines, k, rng):
    """Lines of every scale: entries over 2^-24 .. 1 of the line's maximum, each a
    multiple of an eighth, just above or below one, or arbitrary."""
    m = 1.0 + rng.integers(0, 8, (lines, k)) / 8.0
    step = rng.integers(0, 4, (lines, k))
    m = np.where(step == 1, np.nextafter(m, 4.0), np.where(step == 2, np.nextafter(m, 0.0), m))
    m = np.where(step == 3, rng.uniform(1.0, 2.0, (lines, k)), m)
    x = np.ldexp(m * rng.choice([-1.0, 1.0], (lines, k)), rng.integers(-24, 1, (lines, k)))
    x = np.ldexp(x, rng.integers(-300, 300, lines)[:, None])
    x[rng.random((lines, k)) < 0.1] = 0.0
    return x


@pytest.mark.parametrize("m,n,k", [
    (1, 1, 1), (17, 40, 128), (300, 33, 129), (16, 15, 257), (70, 90, 1024),
    (70, 90, 1025),                    # maxima, then bound operands
    (1800, 20, 1025), (1793, 3, 2048), (1800, 20, 3000), (1800, 20, 8192),
    (1800, 20, 8193),                  # maxima, then bound operands
])
@pytest.mark.parametrize("mode", ["accurate", "fast"])
def test_whole_lines(m, n, k, mode):
    print(f"whole lines {m}x{n}x{k} {mode}", flush=True)
    rng = np.random.default_rng(9600 + k)
    A, B = _operand(m, k, rng), _operand(n, k, rng).T.copy()
    if m > 1:
        A[m // 2] = 0.0                                        # a zero line
        A[1] = np.ldexp(A[1] / np.abs(A[1]).max() if A[1].any() else A[1], -1060)  # subnormal
        A[m - 1, -1] = 5e-324
        B[:, 0] = 0.0
        B[-1, 0] = -1e-320                                     # a subnormal maximum
        A[2, :] = np.ldexp(1.0 + 2.0 ** -52, -1004 - (np.arange(k) % 23))  # subnormal entries
    N = 2
    for ta, tb in (("N", "T"), ("T", "N")):
        r = run(A, B, N, ta, tb, keep_ws=True, mode=mode, pad=(1, 2, 0))
        assert r.status == 0
        C, st = ref.emulate(A, B, N, keep_stages=True, mode=mode)
        EA, EB = r.lines(1)
        assert np.array_equal(EA, st["EA"]) and np.array_equal(EB, st["EB"])
        eA, eB = r.lines(2)
        assert np.array_equal(eA, st["e"]) and np.array_equal(eB, st["f"])
        if mode == "accurate":
            Ab, Bb = r.bar("A"), r.bar("B")
            assert np.array_equal(Ab[:m, :k], ref.e4m3_encode_exact(st["Abar"]))
            assert np.array_equal(Bb[:n, :k], ref.e4m3_encode_exact(st["Bbar"].T))
            assert not Ab[m:].any() and not Ab[:, k:].any()
            assert not Bb[n:].any() and not Bb[:, k:].any()
        assert same_bits(r.C, C)


@pytest.mark.parametrize("mode", ["accurate", "fast"])
def test_flags(mode):
    rng = np.random.default_rng(9700)
    A, B = _operand(40, 300, rng), _operand(21, 300, rng).T.copy()
    A[3, 299] = np.inf
    A[4] = np.nan
    A[5] = 0.0
    B[0, 20] = -np.inf
    B[:, 7] = 0.0
    r = run(A, B, 9, keep_ws=True, mode=mode)
    fA, fB = r.lines(9, np.uint32)
    assert [i for i in range(40) if fA[i] & 1] == [3, 4] and fA[5] & 2 and fA[4] & 2
    assert [j for j in range(21) if fB[j] & 1] == [20] and fB[7] & 2
    assert r.status == 0 and same_bits(r.C, ref.emulate(A, B, 9, mode=mode))
