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


def test_default_schedule(ask):
    """The schedule (1 three branches, 3 two, 2 one stream) of eager solves and of graphs on both
    sides of the line of small plans: 2^20 coefficients of 16^3-block spectra (17408 each) are 60.2
    blocks, of 8^3-block spectra (2304 each) 455.1.  Few sources do not make a plan small when they
    have many near targets (eager) or evaluation blocks (graphs)."""
    plain = "0 0 0 1"
    for prec in (64, 32):
        assert ask("schedule 16 8 0 %d 3 %s" % (prec, plain), "schedule 16 8 0 %d 4 %s" % (prec, plain),
                   "schedule 8 6 0 %d 7 %s" % (prec, plain), "schedule 8 6 0 %d 8 %s" % (prec, plain)) == [
            [2, 2], [1, 3], [2, 2], [1, 3]]
        # separate sets: 8 sources with 27 near targets, 36 with 84, 41 scattered among 4096, one source
        # in a small set
        assert ask("schedule 16 8 0 %d 10 2 2 2 1" % prec, "schedule 16 8 0 %d 10 6 3 2 1" % prec,
                   "schedule 16 8 0 %d 16 16 16 16 100" % prec, "schedule 16 8 0 %d 3 1 1 1 1" % prec) == [
            [2, 3], [3, 3], [3, 3], [2, 2]]
        # the lattice scheme
        assert ask("schedule 16 17 0 %d 2 %s" % (prec, plain), "schedule 16 17 0 %d 8 %s" % (prec, plain)) == [
            [1, 1], [1, 1]]
        # one level, the all-pairs list its far field (graphs' line: 2^18 coefficients, 113.8 blocks of
        # 8^3); two levels follow the general rule
        eager = 2 if prec == 64 else 3
        assert ask("schedule 16 8 1 %d 5 %s" % (prec, plain), "schedule 8 6 1 %d 4 %s" % (prec, plain),
                   "schedule 8 6 1 %d 5 %s" % (prec, plain), "schedule 16 8 2 %d 5 %s" % (prec, plain)) == [
            [eager, 1], [2, 2], [2, 1], [1, 3]]


def test_m2l_variant(ask):
    """The M2L's default variant counts the waves that a level gives, parents x S / 64 with
    S = 4 p^2 (p + 1), not its parents alone: with the few frequencies of p <= 5, workgroups of 64
    parents leave most of the chip idle.  The lines: 32 and 1024 parents, 1280 waves, blocks of 16^3."""
    S = {p: 4 * p * p * (p + 1) for p in (2, 4, 5, 8)}
    cases = [(31, 8, 8, 2), (32, 8, 8, 4), (35, 8, 8, 4), (36, 8, 8, 8), (35, 8, 16, 8), (64, 8, 8, 8), (64, 5, 8, 4),
             (136, 5, 4, 4), (137, 5, 4, 8), (216, 4, 12, 4), (216, 4, 16, 8), (1023, 2, 4, 4), (1024, 2, 4, 8),
             (31, 2, 16, 2), (512, 8, 16, 8)]
    for F in (8, 16):
        got = ask(*["m2l %d %d %d %d" % (parents, S[p], F, n) for parents, p, n, _ in cases])
        assert got == [[c, {2: 8, 4: 256 // F, 8: 64}[c]] for _, _, _, c in cases]


def test_tuned_schedule_is_for_eager_solves(ask):
    """A schedule that the autotuner chose, or that a later plan inherits, serves eager solves by
    themselves; a graph and a server's solve beside others keep the plan's rule, as without tuning.
    One pinned by hand serves all."""
    for lattice in (0, 1):
        beside = 1 if lattice else 2  # (the lattice scheme keeps its own default, 1 here)
        for overlap in (0, 1, 2, 3):
            tuned = overlap or 1
            # by itself, beside others, as a graph
            assert ask(*["solve %d 1 %d %d %d 1 3" % (overlap, lattice, b, g) for b, g in ((0, 0), (0, 1))]) == [
                [tuned], [3]]
            pinned = overlap or None
            assert ask(*["solve %d 0 %d %d %d 1 3" % (overlap, lattice, b, g) for b, g in ((0, 0), (1, 0), (0, 1))]) \
                == [[pinned or 1], [pinned or beside], [pinned or 3]]
        assert ask("solve 3 1 %d 1 0 1 3" % lattice) == [[3 if lattice else 2]]


def test_field_items(ask):
    """The level-0 field spectra's stride: one item more at multiples of 1024 targets only."""
    assert ask("items 1023", "items 1024", "items 1025", "items 512", "items 4096") == [
        [1023], [1025], [1025], [512], [4097]]


def test_runs_of_towers(ask):
    """Towers of 16, 16, 16, 16, 10 and 5 blocks: 8, 8, 8, 8, 5 and 3 groups of 2^3.  Alone they are
    few groups and every run is one; 25 and 171 copies of them make runs of whole towers, and
    workgroups of four that march in lockstep (8 8 8 8) between such that do not (5 3 8 8), the last
    one not full (tests/test_gpu_near.py solves these)."""
    alone, many, small = ask("runs 8 1 16 16 16 16 10 5", "runs 8 25 16 16 16 16 10 5", "runs 4 171 16 16 16 16 10 5")
    assert alone == [1] * 40 + [0, 40, 0, 10]
    assert many == [8, 8, 8, 8, 5, 3, 0, 150, 13, 25]
    assert small == [8, 8, 8, 8, 5, 3, 0, 1026, 86, 171]
