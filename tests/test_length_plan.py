"""The split lengths a Full call plans from the selected requests' lengths
(csrc/oda_length_plan.h, compiled for the host), against an exhaustive search:
the shortest fitting split is found to within 1/16, whole units are returned
only where nothing shorter fits or the plan's first rules say so, and the
slowest CU's share is bounded by the best that any number of rounds gives."""
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CUS, SHORTEST, ROUND_BLOCKS, ROUNDS, LONG, LONG_SPLIT = 256, 8, 128, 16, 1024, 512

PROGRAM = r"""
#include <cmath>
#include <cstdio>
#include <vector>
#include "oda_length_plan.h"
static unsigned plan_less(unsigned most, int i) { return most < (unsigned)i ? most : (unsigned)i; }
int main(int argc, char**) {
  if (argc > 1) {   // quotients: every c below 2^16 and some above, n around its multiples, inv off by an ulp or two
    unsigned bad = 0, state = 1;
    for (unsigned c = 1; c < (1u << 24); c += c < (1u << 16) ? 1 : 997)
      for (int i = 0; i < 40; ++i) {
        state = state * 1664525u + 1013904223u;
        const unsigned most = oda::plan_min((1u << 26) / c, 1u << 20), k = i < 3 ? most - plan_less(most, i) : state % (most + 1);
        for (int d = -1; d <= 1; ++d) {
          const long long n = (long long)k * c + d;
          if (n < 0 || n > (1 << 26) || n > (1ll << 20) * c) continue;
          for (int u = -2; u <= 2; ++u) {
            float inv = 1.0f / (float)c;
            for (int j = 0; j < (u < 0 ? -u : u); ++j) inv = std::nextafter(inv, u < 0 ? 0.f : 2.f);
            bad += oda::ceil_quotient((unsigned)n, c, inv) != (unsigned)((n + c - 1) / c);
          }
        }
      }
    std::printf("%u\n", bad);
    return 0;
  }
  unsigned units, max_splits, slots, head_dim, pairs, count;
  while (std::scanf("%u %u %u %u %u %u", &units, &max_splits, &slots, &head_dim, &pairs, &count) == 6) {
    std::vector<unsigned> n(count);
    unsigned total = 0, longest = 0, calls = 0;
    for (auto& x : n) {
      std::scanf("%u", &x);
      total += x;
      longest = oda::plan_max(longest, x);
    }
    const auto pairs_of = [&](unsigned c) {
      unsigned s = 0;
      ++calls;
      for (unsigned x : n) s += oda::plan_max(1, (x + c - 1) / c);
      return s;
    };
    const unsigned whole = oda::even_up(oda::plan_max(longest, 2));
    const unsigned fit = oda::shortest_fit(total, count, SHORTEST, whole, pairs, pairs_of);
    const unsigned fit_calls = calls;
    std::printf("%u %u %u\n", fit, fit_calls,
                oda::length_bps(total, longest, count, units, max_splits, slots, head_dim, pairs_of));
  }
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no C++ compiler")
    d = tmp_path_factory.mktemp("plan")
    (d / "plan.cpp").write_text(PROGRAM.replace("SHORTEST", str(SHORTEST)))
    csrc = os.path.join(ROOT, "paper_2609_20734_amd", "csrc")
    subprocess.run([cxx, "-std=c++17", "-O2", "-Wall", "-Werror", "-Wno-unused-result", "-I", csrc, str(d / "plan.cpp"),
                    "-o", str(d / "plan")], check=True)

    def run(cases):
        if cases is None:
            return subprocess.run([str(d / "plan"), "quotients"], capture_output=True, text=True, check=True, timeout=60).stdout
        """(units, max_splits, slots, head_dim, pairs, blocks) -> (shortest_fit, its trials, length_bps)."""
        text = "\n".join(" ".join(map(str, [*c[:5], len(c[5]), *c[5]])) for c in cases)
        out = subprocess.run([str(d / "plan")], input=text, capture_output=True, text=True, check=True, timeout=60).stdout
        return [tuple(map(int, line.split())) for line in out.splitlines()]

    return run


def _pairs(n, c):
    return int(np.maximum(1, -(-np.asarray(n) // c)).sum())


def _exact(n, least, pairs):
    """The shortest even fitting split, and the length of whole units."""
    whole = max(2, (max(n) + 1) & ~1)
    lo, hi = min(whole, least), whole          # _pairs falls as c grows
    while lo < hi:
        mid = ((lo + hi) // 2) & ~1
        if _pairs(n, mid) <= pairs:
            hi = mid
        else:
            lo = mid + 2
    return lo, whole


def _draw(g, kind):
    B = int(g.integers(2, 65))
    n = np.exp(g.uniform(np.log(1), np.log(4096), B)).astype(int)
    if kind == "even":
        lo, hi = sorted(np.exp(g.uniform(np.log(12), np.log(4096), 2)).astype(int))
        n = np.linspace(lo, hi, B).astype(int)
    elif kind == "two":
        n = np.where(g.random(B) < 0.3, n[0], n[1])
    elif kind == "equal":
        n[:] = n[0]
    return np.maximum(n, 0).tolist()


@pytest.mark.parametrize("kind", ["any", "even", "two", "equal"])
def test_random_lengths(plan, kind):
    g = np.random.default_rng(len(kind))
    cases = []
    for _ in range(1500):
        n = _draw(g, kind)
        units, D = int(g.choice([1, 2, 4, 8, 16, 24, 48, 63])), int(g.choice([64, 128]))
        slots = len(n) + int(g.integers(0, 2 * CUS // units + 1))
        cases.append((units, int(g.choice([16, 64])), slots, D, int(g.integers(len(n), 4 * len(n) + 2)), n))
    for (units, max_splits, slots, D, pairs, n), (fit, trials, bps) in zip(cases, plan(cases)):
        best, whole = _exact(n, SHORTEST, pairs)
        assert fit % 2 == 0 and _pairs(n, fit) <= pairs and best <= fit <= best + max(2, best // 16)
        assert trials <= 16
        assert bps % 2 == 0 and max(-(-x // bps) for x in n) <= max_splits and _pairs(n, bps) <= slots
        work, rounds = sum(n) * units, -(-len(n) * units // CUS)
        least = (max(SHORTEST, -(-max(n) // max_splits)) + 1) & ~1
        if bps == whole and (rounds >= 8 or work * 20 >= rounds * whole * CUS * 19
                             or (rounds == 1 and whole * 5 * CUS <= 8 * work + 240 * 128 // D * CUS)
                             or (rounds > 1 and work < ROUND_BLOCKS * (rounds + 1) * CUS)):
            continue
        if work >= LONG * CUS:
            c = min(whole, max(least, LONG_SPLIT))
            if _pairs(n, c) > slots:
                c = _exact(n, least, slots)[0]
            assert c <= bps <= c + max(2, c // 16)
            continue
        # the shares of the rounds it may use; it stops at one within 10% of even
        shares = [m * _exact(n, least, min(CUS * m // units, slots))[0] for m in range(rounds, ROUNDS + 1)
                  if m == rounds or work >= ROUND_BLOCKS * m * CUS]
        share = -(-_pairs(n, bps) * units // CUS) * bps
        assert share <= max(min(shares) * 17 / 16 + 2 * ROUNDS, work / CUS / 0.9 + 2 * ROUNDS), (n, units, slots, bps)


def test_evenly_spread_lengths_are_split(plan):
    """Six requests of 3,622-43,790 positions, two units each: 128 pairs fit
    splits of 74 blocks; a search that gave up after four guesses left them
    whole (402 us instead of 39)."""
    n = [227, 729, 1231, 1733, 2235, 2737]
    (fit, _, bps), = plan([(2, 42, 256, 128, 128, n)])
    assert _exact(n, SHORTEST, 128)[0] == 74 and fit <= 78 and bps <= 78


def test_quotients(plan):
    """ceil_quotient is exact over its range with a reciprocal two units off."""
    assert int(plan(None)) == 0
