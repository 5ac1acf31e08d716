"""The E2M3 path of the FP8 lists (more than four output tiles) through the C
ABI: the stored digits, the residue planes and C against the oracle, at the
edges of its tiles, stages and scale range."""
import numpy as np
import pytest
import torch

import paper_2603_10634_amd as oz
from oracle import ozaki2_ref as ref
from workloads import phi_matrix

from gpu_util import run, same_bits, split

pytestmark = pytest.mark.gpu


def _digits(r, which):
    """M x lines x k digits decoded from the documented fragment order."""
    mp, np_, kp, M = (r.pads[q] for q in ("mp", "np", "kp", "M"))
    R = mp if which == "A" else np_
    o = r.off[5 if which == "A" else 6]
    size = R * kp // 4 * 3
    h = np.arange(kp)
    line = np.arange(R)[:, None]
    frag = ((h // 128) * (R // 64) + line // 64) * 4 + line % 4
    lane = (line % 64) // 4 + 16 * ((h % 128) // 32)
    out = []
    for q in range(M):
        b = r.ws[o + q * size:o + (q + 1) * size].reshape(-1, 1536)
        lanes = np.concatenate([b[:, :1024].reshape(-1, 64, 16), b[:, 1024:].reshape(-1, 64, 8)],
                               axis=2)
        bits = np.unpackbits(lanes, axis=2, bitorder="little").reshape(-1, 64, 32, 6)
        code = bits @ (1 << np.arange(6))
        val = np.where(code & 32, -(code & 31), code & 31).astype(np.int8)
        out.append(val[frag, lane, h % 32])
    return np.stack(out)


def _check(A, B, N, ta="N", tb="N", mode="accurate", moduli="hybrid"):
    m, k = A.shape
    n = B.shape[1]
    r = run(A, B, N, ta, tb, keep_ws=True, mode=mode, moduli=moduli, pad=(3, 5, 1))
    assert r.status == 0
    C, st = ref.emulate(A, B, N, keep_stages=True, mode=mode, moduli_set=moduli)
    D = {"A": _digits(r, "A"), "B": _digits(r, "B")}
    P = r.planes(N, [pm["p"] for pm in st["per_modulus"]])
    sl = 0
    for l, pm in enumerate(st["per_modulus"]):
        p, square = pm["p"], pm["kind"] == "square"
        s = int(round(p ** 0.5)) if square else 16
        for which, want, lines in (("A", pm["dA"], m), ("B", [d.T for d in pm["dB"]], n)):
            d = D[which][sl:sl + (2 if square else 3)].astype(np.int64)
            assert np.abs(d).max() <= 16
            assert not d[:, lines:].any() and not d[:, :, k:].any(), "padding"
            u = s * d[0] + d[1]
            w = s * want[0].astype(np.int64) + want[1].astype(np.int64)
            assert not np.any((u[:lines, :k] - w) % p), f"residues of {which} modulo {p}"
            if not square:
                assert np.array_equal(d[2], d[0] + d[1])
        sl += 2 if square else 3
        assert np.array_equal(P[l, :n, :m].T, st["planes"][l]), f"plane {l}"
    assert same_bits(r.C, C)


@pytest.mark.parametrize("m,n,k,N,ta,tb,mode,moduli,phi", [
    (513, 700, 1, 1, "N", "T", "fast", "hybrid", 1.0),        # one k of a stage
    (1280, 64, 257, 6, "T", "N", "accurate", "hybrid", 1.0),  # five tiles, one more 256-block
    (700, 600, 300, 12, "N", "N", "accurate", "hybrid", 0.5),
    (600, 513, 128, 14, "T", "T", "accurate", "hybrid", 2.0),
    (520, 770, 130, 17, "N", "N", "accurate", "hybrid", 4.0),  # a second FP64 step
    (560, 520, 200, 33, "T", "N", "accurate", "hybrid", 6.0),  # the largest exponents
    (600, 600, 500, 13, "N", "T", "accurate", "karatsuba", 1.0),
])
def test_stages(m, n, k, N, ta, tb, mode, moduli, phi):
    print(f"E2M3 {m}x{n}x{k} N={N} {ta}{tb} {mode} {moduli} phi={phi}", flush=True)
    _check(phi_matrix(m, k, phi, 9100 + m), phi_matrix(k, n, phi, 9200 + n), N, ta, tb, mode,
           moduli)


def test_special_lines():
    A = phi_matrix(540, 150, 1.0, 9300)
    B = phi_matrix(150, 700, 1.0, 9301)
    A[7] = 0.0
    A[130, 3] = np.inf
    A[511, 149] = np.nan
    A[200] *= 2.0 ** -1000
    A[201] = 5e-324
    B[:, 64] = 0.0
    B[9, 699] = -np.inf
    B[:, 300] *= 2.0 ** 900
    print("E2M3 special lines", flush=True)
    for N, mode in ((12, "accurate"), (20, "fast")):
        r = run(A, B, N, mode=mode)
        assert r.status == 0 and same_bits(r.C, ref.emulate(A, B, N, mode=mode))


@pytest.mark.parametrize("moduli,N", [("hybrid", 12), ("karatsuba", 5)])
def test_extreme_digit_sums(moduli, N):
    # constant operands whose digits reach 16 x 16 over one accumulation of
    # k = 2^15 (sums of 2^23 per product), rows of both signs, six tiles: every
    # output is the 1 x k x 1 emulation's, up to sign
    k = 32768
    for c in (255, 199, 137, 131):
        a, b = c / 128.0, (c + 1) / 128.0 if c < 255 else c / 128.0
        _, st = ref.emulate(np.full((1, k), a), np.full((k, 1), b), N, keep_stages=True,
                            moduli_set=moduli)
        C1 = ref.emulate(np.full((1, k), a), np.full((k, 1), b), N, moduli_set=moduli)[0, 0]
        top = max(abs(int(x[0, 0]) * int(y[0, 0])) for pm in st["per_modulus"]
                  for x in pm["dA"] for y in pm["dB"])
        print(f"E2M3 sums c={c}: digit products up to {top}", flush=True)
        A = np.full((520, k), a)
        A[1::2] *= -1.0
        B = np.full((k, 260), b)
        with split(1):
            r = run(A, B, N, moduli=moduli)
        want = np.where(np.arange(520)[:, None] % 2, -C1, C1) * np.ones((1, 260))
        assert r.status == 0 and same_bits(r.C, want)


@pytest.mark.parametrize("parts", [1, 3, 8])
def test_split_and_blocked(parts):
    # ragged k parts; blocks of which some have four tiles or fewer
    A, B = phi_matrix(800, 2500, 1.0, 9400), phi_matrix(2500, 700, 1.0, 9401)
    want = ref.emulate(A, B, 12)
    with split(parts):
        assert same_bits(run(A, B, 12).C, want)
        assert same_bits(run(A, B, 12, "T", "T", blocking=(768, 512)).C, want)


@pytest.mark.parametrize("moduli", ["hybrid", "int8"])
@pytest.mark.parametrize("m,n,k", [(1, 1300, 300), (1300, 1, 70), (64, 1409, 513), (65, 1408, 200),
                                   (1345, 129, 256), (1344, 128, 700)])
def test_waves_without_outputs(m, n, k, moduli):
    # tiles of which a wave's 128 (columns) x 64 (rows) is padding, one row or
    # column of it is not, or all of it is used, item after item
    A, B = phi_matrix(m, k, 1.0, 9500 + m), phi_matrix(k, n, 1.0, 9600 + n)
    print(f"padding waves {m}x{n}x{k} {moduli}", flush=True)
    C, st = ref.emulate(A, B, 14, keep_stages=True, moduli_set=moduli)
    r = run(A, B, 14, keep_ws=True, moduli=moduli)
    assert r.status == 0
    P = r.planes(14, [pm["p"] for pm in st["per_modulus"]])
    for l, plane in enumerate(st["planes"]):
        assert np.array_equal(P[l, :n, :m].T, plane), f"plane {l}"
    assert same_bits(r.C, C)


def test_waves_without_outputs_in_a_batch():
    # items of several sizes in one launch, sorted by k only: full, ragged and
    # nearly empty tiles follow one another in a workgroup
    import torch
    rng = np.random.default_rng(9700)
    shapes = [(int(m), int(n), int(k)) for m, n, k in
              zip(rng.choice([1, 63, 64, 65, 129, 256, 300, 513], 40),
                  rng.choice([1, 127, 128, 129, 256, 400], 40), rng.choice([30, 257, 600], 40))]
    As = [phi_matrix(m, k, 1.0, 9701 + q) for q, (m, n, k) in enumerate(shapes)]
    Bs = [phi_matrix(k, n, 1.0, 9801 + q) for q, (m, n, k) in enumerate(shapes)]
    Cs = oz.dgemm_batched([torch.from_numpy(a).cuda() for a in As],
                          [torch.from_numpy(b).cuda() for b in Bs], 12)
    for q, (a, b) in enumerate(zip(As, Bs)):
        assert same_bits(Cs[q].cpu().numpy(), ref.emulate(a, b, 12)), shapes[q]


@pytest.mark.parametrize("k,config", [(65536, 0), (131072, 0), (131072, 1)])
def test_square_cross_sums_over_chunks(k, config):
    # an item of a batch over several chunks of 2^15 (config 1: two k parts of two
    # chunks), residues 544 = 16 x 33 + 16 modulo 1089 on both sides: A1 B2 and
    # A2 B1 sum to 2^23 per chunk, with odd remainders of the chunks before
    one = np.full((1, k), 1.0625)
    sc = ref.scaling(one, one.T.copy(), 12)
    v = _residue_value(int(sc["sA"][0]), 544, 1089)
    w = _residue_value(int(sc["sB"][0]), 544, 1089)
    C1, st = ref.emulate(np.full((1, k), v), np.full((k, 1), w), 12, keep_stages=True)
    pm = next(q for q in st["per_modulus"] if q["p"] == 1089)
    assert [int(d[0, 0]) for d in (*pm["dA"], *pm["dB"])] == [16] * 4
    A, B = np.full((70, k), v), np.full((k, 90), w)
    A[1::2] *= -1.0
    want = np.where(np.arange(70)[:, None] % 2, -C1[0, 0], C1[0, 0]) * np.ones((1, 90))
    print(f"square sums over chunks k={k} config={config} v={v!r} w={w!r}", flush=True)
    assert oz.ozaki2_set_schedule(config) == 0
    try:
        Cs = oz.dgemm_batched([torch.from_numpy(x).cuda() for x in (A, A[:3])],
                              [torch.from_numpy(x).cuda() for x in (B, B[:, :5].copy())], 12)
    finally:
        oz.ozaki2_set_schedule(-1)
    assert same_bits(Cs[0].cpu().numpy(), want)
    assert same_bits(Cs[1].cpu().numpy(), want[:3, :5])


def _residue_value(shift, target, p, base=1.0625):
    """A value just above `base` whose integer trunc(v 2^shift) is congruent to
    `target` modulo p."""
    g = max(shift - 52, 0)
    t = int(base * 2.0 ** (shift - g))
    t += (target * pow(2 ** g, -1, p) - t) % p
    return float(np.ldexp(float(t), g - shift))
