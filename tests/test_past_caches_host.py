"""Which C are stored past the caches: none whose next reader would lose more than the
call gains."""
import os
import subprocess

from test_crt_host import CSRC, ROOT


def test_a_c_that_is_read_next_stays_in_the_caches(tmp_path):
    out = str(tmp_path / "past_caches")
    subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + CSRC, os.path.join(ROOT, "tests", "past_caches_host_check.cpp"),
                    "-o", out], check=True, capture_output=True)
    # (megabytes of C, columns of whole 128-byte lines, batch, past the caches)
    cases = [(1, 1, 0, 0), (48, 1, 0, 0), (72, 1, 0, 1), (128, 1, 0, 1), (64, 0, 0, 0),
             (83, 0, 0, 0), (104, 0, 0, 0), (154, 0, 0, 0), (191, 0, 0, 1), (2048, 0, 0, 1),
             (96, 0, 1, 0), (192, 0, 1, 0), (240, 0, 1, 0), (320, 0, 1, 1)]
    text = "".join("%d %d %d\n" % c[:3] for c in cases)
    got = subprocess.run([out], input=text, capture_output=True, text=True, check=True).stdout
    assert [int(x) for x in got.split()] == [c[3] for c in cases]
