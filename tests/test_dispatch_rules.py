"""The rules that choose between forms of a kernel, compiled from their headers for
the host.  Each point of the VALU basis conversion (one or three target rows per
workgroup, the digits' inverse columns finished inside it or by a pass of their
own) and of the fused kernels at N = 4096 is a launch whose two forms were timed
(times beside the rules)."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2608_17442_amd", "csrc")


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    d = tmp_path_factory.mktemp("rule")
    src, exe = d / "rule.cpp", d / "rule"
    src.write_text("""
#include <cstdio>
#include "conversion_rule.hpp"
#include "small_ring_rule.hpp"
int main() {
  char kind;
  unsigned a, b, c, d, e;
  while (std::scanf(" %c %u %u %u %u %u", &kind, &a, &b, &c, &d, &e) == 6) {
    if (kind == 'c') {
      const fesc::ValuConversion v = fesc::valu_conversion(a, b, c, d);
      std::printf("%u %d\\n", v.targets, v.fuse);
    } else if (kind == 'u') {
      std::printf("%d\\n", fesc::small_modup_pays(a, b, c, d));
    } else if (kind == 'd') {
      std::printf("%d\\n", fesc::small_moddown_pays(a, b, c, d, e));
    } else if (kind == 'r') {
      std::printf("%d\\n", fesc::small_rescale_pays(a, b, c));
    } else {
      const uint64_t* p = nullptr;
      std::printf("%d\\n", fesc::overlap(p + a, b, p + c, d));
    }
  }
}
""")
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True)

    def run(kind, points):
        text = "\n".join(" ".join(map(str, (kind, *p, *[0] * (5 - len(p))))) for p in points)
        out = subprocess.run([str(exe)], input=text, capture_output=True, text=True, check=True)
        return [tuple(map(int, line.split())) for line in out.stdout.splitlines()]
    return run


@pytest.fixture(scope="module")
def rule(ask):
    return lambda points: ask("c", [(n - 12, d, t, g) for n, d, t, g in points])


# (log N, primes of the longest digit, target rows, digits) of one conversion launch
FUSED = [(13, 1, 4, 4), (14, 1, 12, 12), (16, 1, 4, 2), (14, 2, 16, 8), (16, 2, 8, 4),
         (13, 3, 24, 32), (14, 3, 24, 2), (15, 3, 12, 8), (16, 3, 6, 4), (13, 5, 12, 2),
         (13, 9, 9, 2), (14, 9, 9, 2), (15, 3, 3, 48), (15, 3, 9, 20), (16, 3, 9, 6), (16, 2, 6, 16),
         (14, 9, 4, 32), (15, 9, 3, 40), (16, 10, 2, 16)]
SEPARATE_ONE = [(15, 9, 9, 2), (15, 9, 24, 3), (13, 12, 24, 4), (15, 12, 24, 2), (13, 16, 24, 2),
                (14, 16, 24, 4), (16, 9, 9, 4), (12, 1, 4, 4), (12, 16, 24, 16), (15, 9, 9, 4),
                (16, 12, 3, 6), (16, 16, 3, 6)]
SEPARATE_THREE = [(16, 9, 24, 3), (16, 12, 24, 2), (14, 12, 24, 8), (13, 16, 24, 16), (15, 9, 18, 8),
                  (15, 3, 24, 16), (16, 3, 12, 8), (13, 3, 24, 64), (16, 1, 12, 48),
                  (12, 1, 24, 192), (13, 50, 50, 4096), (14, 3, 24, 20), (15, 3, 12, 20),
                  (16, 3, 12, 8), (15, 9, 6, 24)]


def test_forms(rule):
    assert rule(FUSED) == [(1, 1)] * len(FUSED)
    assert rule(SEPARATE_ONE) == [(1, 0)] * len(SEPARATE_ONE)
    assert rule(SEPARATE_THREE) == [(3, 0)] * len(SEPARATE_THREE)


def test_never_fused_where_there_is_no_pass_to_save(rule):
    points = [(12, d, t, g) for d in (1, 3, 16) for t in (1, 24) for g in (1, 7, 96)]
    assert all(not fuse for _, fuse in rule(points))


def test_more_work_never_returns_to_the_fused_form(rule):
    """Along digit length, rows and batch the fused form is given up once."""
    for log_n in range(13, 17):
        for t in (2, 9, 24, 48):
            for g in (1, 2, 8, 32):
                by_digit = [f for _, f in rule([(log_n, d, t, g) for d in range(1, 17)])]
                assert by_digit == sorted(by_digit, reverse=True)
        for d in (1, 3, 9):
            by_group = [f for _, f in rule([(log_n, d, 12, g) for g in range(1, 129)])]
            assert by_group == sorted(by_group, reverse=True)


def _flags(out):
    return [bool(f) for f, in out]


def test_small_ring_limits(ask):
    """Both sides of every limit: the ring, the primes that are converted (ModDown
    merged with the rescale has one more), the work of the launch."""
    # log N, alpha, sources, level
    assert _flags(ask("u", [(12, 1, 1, 3), (12, 1, 14, 8), (12, 1, 15, 8), (12, 3, 3, 15),
                            (12, 3, 5, 15), (12, 4, 1, 5), (13, 1, 1, 3)])) == \
        [True, True, False, True, False, False, False]
    # log N, alpha, merged, jobs, rows
    assert _flags(ask("d", [(12, 1, 0, 1, 3), (12, 3, 0, 5, 29), (12, 3, 0, 6, 29),
                            (12, 4, 0, 1, 5), (12, 1, 1, 32, 11), (12, 2, 1, 16, 15),
                            (12, 2, 1, 32, 15), (12, 3, 1, 1, 11), (12, 3, 1, 4, 23),
                            (16, 1, 0, 1, 3)])) == \
        [True, True, False, False, True, True, False, False, False, False]
    # log N, ciphertexts, rows
    assert _flags(ask("r", [(12, 1, 1), (12, 16, 32), (12, 16, 33), (12, 15, 34), (12, 16, 47),
                            (13, 1, 2)])) == [True, True, False, True, False, False]


def test_overlap(ask):
    """Word ranges that touch do not meet; a shared word is enough."""
    assert _flags(ask("o", [(0, 8, 8, 4), (8, 4, 0, 8), (0, 9, 8, 4), (8, 4, 0, 9), (0, 20, 5, 2),
                            (5, 2, 0, 20), (3, 4, 3, 4)])) == \
        [False, False, True, True, True, True, True]
