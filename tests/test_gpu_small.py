"""The products of few output tiles through the C ABI: every stage against the
oracle at the edges of their tiles, k steps and k parts, and on both sides of
the rules that pick the tile."""
import numpy as np
import pytest

from oracle import ozaki2_ref as ref
from workloads import phi_matrix

from gpu_util import run, check_stages, same_bits, split

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,k,N,moduli,parts", [
    (1, 1, 1, 1, "hybrid", 0),
    (33, 65, 65, 12, "hybrid", 0),
    (97, 31, 449, 33, "hybrid", 0),        # 7 k steps
    (256, 130, 900, 7, "karatsuba", 3),    # k parts of 4, 4 and 7 steps
    (256, 256, 64, 20, "int8", 0),
    (512, 256, 300, 16, "hybrid", 0),      # 512 tiles of 64 x 64: the last of them
    (512, 257, 300, 16, "hybrid", 0),      # 640: tiles of 128 x 128
    (512, 512, 129, 16, "hybrid", 0),      # 256 tiles of 128 x 128
    (512, 512, 129, 17, "hybrid", 0),      # 272: 256 x 256
    (400, 390, 200, 13, "karatsuba", 0),
    (420, 500, 1000, 8, "int8", 2),
])
def test_stages(m, n, k, N, moduli, parts):
    print(f"small tiles {m}x{n}x{k} N={N} {moduli} parts={parts}", flush=True)
    A, B = phi_matrix(m, k, 1.0, 8100 + m + N), phi_matrix(k, n, 1.0, 8200 + n + k)
    with split(parts):
        r = run(A, B, N, "T", "N", keep_ws=True, moduli=moduli, pad=(1, 0, 3))
    assert r.status == 0
    C, st = ref.emulate(A, B, N, keep_stages=True, moduli_set=moduli)
    check_stages(r, A, B, N, st, moduli=moduli)
    assert same_bits(r.C, C)


@pytest.mark.parametrize("m,n,k", [(1345, 1409, 130), (1409, 1470, 70)])
def test_bound_of_many_tiles(m, n, k):
    # 506 tiles of 64 x 64, and 529
    A, B = phi_matrix(m, k, 0.5, 8300), phi_matrix(k, n, 0.5, 8301)
    r = run(A, B, 3, keep_ws=True)
    assert r.status == 0
    C, st = ref.emulate(A, B, 3, keep_stages=True)
    e, f = r.lines(2)
    assert np.array_equal(e, st["e"]) and np.array_equal(f, st["f"])
    assert same_bits(r.C, C)


@pytest.mark.parametrize("moduli,N,parts", [
    ("hybrid", 12, 5),      # 240 workgroups
    ("hybrid", 12, 6),      # 144 + 144
    ("hybrid", 24, 5),      # 480 (120 + 360 would be three rounds)
    ("karatsuba", 13, 6),
])
def test_rounds_of_tiles(moduli, N, parts):
    # four 256 x 256 tiles whose k parts fill one round of the CUs, or more than
    # one (the squares and the Karatsuba moduli are then launched one after the
    # other where that takes no more rounds)
    A, B = phi_matrix(400, 1700, 1.0, 9900), phi_matrix(1700, 300, 1.0, 9901)
    print(f"rounds of tiles {moduli} N={N} parts={parts}", flush=True)
    with split(parts):
        r = run(A, B, N, "T", "N", keep_ws=True, moduli=moduli)
        assert r.status == 0 and r.parts == parts
        check_stages(r, A, B, N, moduli=moduli)
        assert same_bits(r.C, ref.emulate(A, B, N, moduli_set=moduli))
