"""The host's launch rules (csrc/launch_rules.h, plain C++) on the CPU.

A small program is compiled against the header; it answers one rule per line
of input, and each answer is checked against what the rule has to guarantee.
"""
import itertools
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2307_00229_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <cstring>
#include "launch_rules.h"
using namespace clair;
static CallSizes sizes(int points, int f) {
  return {points, (f & 1) != 0, (f & 2) != 0, (f & 4) != 0, (f & 8) != 0, (f & 16) != 0};
}
int main() {
  char rule[32];
  long long a, b, c, d, e;
  while (std::scanf("%31s %lld %lld %lld %lld %lld", rule, &a, &b, &c, &d, &e) == 6) {
    if (!std::strcmp(rule, "pick")) {
      const TilePick p = tile_pick((int)a, (int)b, c != 0);
      std::printf("%d %d\n", p.first, p.second);
    } else if (!std::strcmp(rule, "reach")) {
      std::printf("%d 0\n", bin_b_reach((int)a));
    } else if (!std::strcmp(rule, "chunk")) {
      std::printf("%d 0\n", shrunk_chunk((int)a, b, (int)c));
    } else if (!std::strcmp(rule, "hold")) {
      std::printf("%d 0\n", launches_hold(sizes((int)a, (int)b), sizes((int)c, (int)d), e) ? 1 : 0);
    } else {
      return 1;
    }
  }
  return 0;
}
"""


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    src, exe = d / "rules.cpp", d / "rules"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(src), "-o", str(exe)], check=True)

    def run(lines):
        text = "\n".join(" ".join(str(v) for v in (*q, *[0] * (6 - len(q)))) for q in lines) + "\n"
        out = subprocess.run([str(exe)], input=text, capture_output=True, text=True, check=True).stdout.split("\n")
        return [tuple(int(v) for v in r.split()) for r in out if r]

    return run


def test_tile_instances(ask):
    asked = [("pick", p, r, s) for p in range(1, 33) for r in (9, 16, 20, 24, 32) for s in (0, 1) if p <= r]
    for (_, points, reach, sized), (first, second) in zip(asked, ask(asked)):
        assert first in (12, 16, 20, 24, 28, 32) and points <= first < max(points, 9) + 4  # the smallest that holds them
        if sized or first >= reach:
            assert second == 0
        else:
            assert second >= reach and second > first
    reach = [r for r, _ in ask([("reach", p) for p in range(1, 33)])]
    assert reach == [16 if p <= 16 else 20 if p <= 20 else 24 if p <= 24 else 32 for p in range(1, 33)]


def test_sizes_that_launches_serve(ask):
    """A repeated synchronous call keeps its result when its blocks fit what was
    launched (equal or smaller ones, or larger ones of the same tile), and no
    pass was left out that has work."""
    points = [0, 1, 8, 9, 12, 13, 16, 17, 20, 24, 25, 32, 33, 64, 65, 72, 128, 300]
    flags = [0, 1, 3, 7, 15, 31, 4, 9]
    asked = [("hold", h, hf, g, gf, scratch) for h, g in itertools.product(points, points)
             for hf, gf in itertools.product(flags, flags) for scratch in (0, 72 * 72, 304 * 304)]
    for (_, h, hf, g, gf, scratch), (ok, _) in zip(asked, ask(asked)):
        left_out = gf & ~hf
        beyond_tile = max(9, min(g, 32)) > max(12, -(-min(h, 32) // 4) * 4)
        beyond_scratch = g > 64 and g * g > scratch
        assert ok == (0 if left_out or beyond_tile or beyond_scratch else 1), (h, hf, g, gf, scratch)
        if g <= h and not left_out and (g <= 64 or h * h <= scratch):
            assert ok == 1


def test_chunks_of_small_batches(ask):
    """Halved while workgroups are fewer than CUs, never below 64 points."""
    asked = [("chunk", c, n, cus) for c in range(256, 2049, 256) for cus in (64, 256, 304)
             for n in (1, 63, 5000, 20000, 60000, 130000, 262143, 262144, 10**7)]
    for (_, chunk, n, cus), (got, _) in zip(asked, ask(asked)):
        assert got >= 64 and got in [chunk >> k for k in range(6)]
        if got < chunk:  # each halving was for want of workgroups
            assert n < (got * 2) * cus
        if n < got * cus:  # and one more would go below 64
            assert got // 2 < 64
