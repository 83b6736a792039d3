"""The rules by which a plan picks kernels and schedules, on the host (tests/host_rules_check.cpp
built with g++ from lgf_host.cpp): no GPU needed."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1402_6081_amd", "csrc")
OUT = os.path.join(ROOT, "tests", "_host_build")
GXX = shutil.which("g++")
pytestmark = pytest.mark.skipif(GXX is None, reason="needs g++")


@pytest.fixture(scope="module")
def ask():
    os.makedirs(OUT, exist_ok=True)
    exe = os.path.join(OUT, "host_rules_check")
    srcs = [os.path.join(CSRC, "lgf_host.cpp"), os.path.join(ROOT, "tests", "host_rules_check.cpp")]
    deps = srcs + [os.path.join(CSRC, "lgf_host.h")]
    if not os.path.exists(exe) or os.path.getmtime(exe) < max(os.path.getmtime(f) for f in deps):
        subprocess.run([GXX, "-std=c++17", "-O1", "-g", "-fsanitize=undefined", "-fno-sanitize-recover",
                        "-I", os.path.join(ROOT, "include"), "-I", CSRC] + srcs + ["-o", exe], check=True,
                       capture_output=True, text=True)

    def run(*queries):
        r = subprocess.run([exe], input="\n".join(queries) + "\n", capture_output=True, text=True, timeout=60)
        assert r.returncode == 0, r.stderr[-2000:]
        return [[int(v) for v in a.split()] for a in r.stdout.strip().split("\n")]

    return run


def test_near_fields_never_refuse_first(ask):
    """The level-0 Prod's bound on the near targets lies at or above the M2L's on the level-1
    intervals, (intervals + 1) items of one chunk below 2^32 bytes, so separate sets with more
    targets than sources are refused by neither before that."""
    for chunks, bytes_ in ((2, 8), (1, 16)):  # FP32: two chunks a wave; FP64: one
        most = 2 ** 32 // (64 * bytes_) - 2  # the most intervals the M2L takes
        assert (most + 1) * 64 * bytes_ < 2 ** 32 <= (most + 2) * 64 * bytes_
        assert ask("fields %d %d %d" % (most, chunks, bytes_), "fields %d %d %d" % (most // 2 + 2, chunks, bytes_),
                   "fields 1 %d %d" % (chunks, bytes_)) == [[1], [1], [1]]
    assert ask("fields %d 2 8" % (2 ** 32 // 512 - 1)) == [[0]]
