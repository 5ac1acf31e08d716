"""The CRT kernel's sums of doubles for P < 2^96, compiled for the host with the
library's tables: every value away from the ends of the range is decided, ties and
near ties included, and is RN(C 2^-t) bit for bit."""
import math
import os
import random
import subprocess

import pytest

from oracle import ozaki2_ref as ref
from test_crt_host import CSRC, LISTS, ROOT, SANITIZE, _bits, _rn, _smod


@pytest.fixture(scope="module")
def host_crt(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("crt_small") / "crt_small_host_check")
    cmd = ["g++", "-O1", "-g", *SANITIZE, "-ffp-contract=off", "-std=c++17",
           "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + CSRC,
           os.path.join(ROOT, "tests", "crt_small_host_check.cpp"),
           os.path.join(CSRC, "oz2_tables.cpp"), "-o", out]
    subprocess.run(cmd, check=True, capture_output=True)
    return out


@pytest.mark.parametrize("moduli", ["hybrid", "karatsuba", "int8"])
def test_every_value_is_decided(host_crt, moduli):
    rng = random.Random(8300 + LISTS[moduli])
    for N in range(1, 34):
        mods = [p for p, _, _ in ref.moduli_table(N, moduli)]
        P = math.prod(mods)
        if P >= 2 ** 96:
            break
        top = min(int(P * (0.5 - 2.0 ** -8)), P // 2 - 3)    # (crt_fast is 2 below P / 2)
        cases = [0, 1, -1, top, -top] + [rng.randrange(-top, top + 1) for _ in range(200)]
        # ties and their neighbours at every length from 54 bits
        for bits in range(54, top.bit_length()):
            for _ in range(12):
                odd = (1 << 53) + 2 * rng.randrange(1 << 52) + 1        # 54 bits, a tie
                c = (odd << (bits - 54)) + rng.choice([-1, 0, 0, 1] if bits > 54 else [0])
                cases.append(rng.choice([-1, 1]) * c if c <= top else top)
        ts = [rng.randrange(-900, 900) for _ in cases]
        text = "\n".join(" ".join(str(v) for v in [t] + [_smod(c, p) for p in mods])
                         for c, t in zip(cases, ts))
        res = subprocess.run([host_crt, str(N), str(LISTS[moduli])], input=text + "\n",
                             capture_output=True, text=True, check=True)
        got = [x.split() for x in res.stdout.splitlines()]
        assert len(got) == len(cases)
        for (ok, bits), c, t in zip(got, cases, ts):
            assert ok == "1", (moduli, N, c, t)
            assert int(bits, 16) == _bits(_rn(c, t)), (moduli, N, c, t)
