"""The CRT kernel's fast path (crt_rn of oz2_crt_math.h), compiled for the host
with the library's tables: whatever it decides is RN(C 2^-t) bit for bit, it
decides nearly every value that is spread over the range, and it leaves exact
ties, out-of-range estimates and subnormal results to the exact path."""
import math
import os
import random
import subprocess

import pytest

from oracle import ozaki2_ref as ref
from test_crt_host import CSRC, LISTS, ROOT, SANITIZE, _bits, _rn, _shift, _smod, _targets


@pytest.fixture(scope="module")
def rn_checker(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("crt_rn") / "crt_rn_host_check")
    cmd = ["g++", "-O1", "-g", *SANITIZE, "-ffp-contract=off", "-std=c++17",
           "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + CSRC,
           os.path.join(ROOT, "tests", "crt_rn_host_check.cpp"),
           os.path.join(CSRC, "oz2_tables.cpp"), "-o", out]
    subprocess.run(cmd, check=True, capture_output=True)
    return out


@pytest.mark.parametrize("moduli", ["hybrid", "karatsuba", "int8"])
def test_decided_values_are_exact(rn_checker, moduli):
    rng = random.Random(8200 + LISTS[moduli])
    for N in range(1, 34):
        mods = [p for p, _, _ in ref.moduli_table(N, moduli)]
        P = math.prod(mods)
        h = P // 2
        spread = [rng.randrange(-h, P - h) // rng.choice([1, 3, 1000, 10 ** 6]) for _ in range(100)]
        near = P.bit_length() - 53
        cases = [(c, _shift(c, P, rng)) for c in _targets(P, rng, 60)]
        cases += [(c, near + rng.randrange(-60, 60)) for c in spread]
        # the kernel's residues after a k split: one beyond the symmetric range
        lines = []
        for c, t in cases:
            us = [_smod(c, p) for p in mods]
            lines.append(" ".join(str(v) for v in [t] + us))
        wide = [" ".join(str(v) for v in [near] + [s * (p // 2 + 1) for p in mods]) for s in (-1, 1)]
        res = subprocess.run([rn_checker, str(N), str(LISTS[moduli])],
                             input="\n".join(lines + wide) + "\n", capture_output=True, text=True,
                             check=True)
        got = [(int(x.split()[0]), int(x.split()[1], 16)) for x in res.stdout.splitlines()]
        assert len(got) == len(lines) + 2
        for ln, (ok, bits), (c, t) in zip(lines, got, cases):
            want = _rn(c, t)
            if ok:
                assert bits == _bits(want), (moduli, N, ln)
            assert not (ok and 0 < abs(want) < 2.0 ** -1022), "subnormal result decided"
        if P.bit_length() > 90:      # (the smallest spread values keep 70 bits)
            decided = sum(ok for ok, _ in got[len(cases) - len(spread):len(cases)])
            assert decided == len(spread), (moduli, N, decided)
        # a residue tuple is some C: the sum of weights times residues mod P
        for s, (ok, bits) in zip((-1, 1), got[len(lines):]):
            c = 0
            for p in mods:
                w = P // p * pow(P // p, -1, p)
                c += w * s * (p // 2 + 1)
            if ok:
                assert bits == _bits(_rn(_smod(c, P), near)), (moduli, N, "wide", s)
