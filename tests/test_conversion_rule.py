"""The choice between the forms of the VALU basis conversion: one or three target
rows per workgroup, the digits' inverse columns finished inside it or by a pass
of their own.  Compiled from its header for the host; each point is a launch
whose two forms were timed and differ (times beside the rule)."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2608_17442_amd", "csrc")


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("rule")
    src, exe = d / "rule.cpp", d / "rule"
    src.write_text("""
#include <cstdio>
#include "conversion_rule.hpp"
int main() {
  unsigned m, d, t, g;
  while (std::scanf("%u %u %u %u", &m, &d, &t, &g) == 4) {
    const fesc::ValuConversion v = fesc::valu_conversion(m, d, t, g);
    std::printf("%u %d\\n", v.targets, v.fuse);
  }
}
""")
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True)

    def ask(points):
        text = "\n".join(f"{n - 12} {d} {t} {g}" for n, d, t, g in points)
        out = subprocess.run([str(exe)], input=text, capture_output=True, text=True, check=True)
        return [tuple(map(int, line.split())) for line in out.stdout.splitlines()]
    return ask


# (log N, primes of the longest digit, target rows, digits) of one conversion launch
FUSED = [(13, 1, 4, 4), (14, 1, 12, 12), (16, 1, 4, 2), (14, 2, 16, 8), (16, 2, 8, 4),
         (13, 3, 24, 32), (14, 3, 24, 2), (15, 3, 12, 8), (16, 3, 6, 4), (13, 5, 12, 2),
         (13, 9, 9, 2), (14, 9, 9, 2)]
SEPARATE_ONE = [(15, 9, 9, 2), (15, 9, 24, 3), (13, 12, 24, 4), (15, 12, 24, 2), (13, 16, 24, 2),
                (14, 16, 24, 4), (16, 9, 9, 4), (12, 1, 4, 4), (12, 16, 24, 16)]
SEPARATE_THREE = [(16, 9, 24, 3), (16, 12, 24, 2), (14, 12, 24, 8), (13, 16, 24, 16), (15, 9, 18, 8),
                  (15, 3, 24, 16), (16, 3, 12, 8), (13, 3, 24, 64), (16, 1, 12, 48),
                  (12, 1, 24, 192), (13, 50, 50, 4096)]


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
