"""The electron launch's division of several discharges' work (work_split.h),
compiled for the host: each division covers all units within the room there is
for its ranges, and the busiest workgroup has little more than an equal share,
whatever the sizes and however many discharges there are."""
import os
import random
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1508_02892_amd", "csrc")

PROBE = """
#include <cstdio>
#include <vector>
#include <algorithm>
#include "work_split.h"
// reads "workgroups waves most_rounds D units..." and prints the length of the
// ranges, as the launch finds it
int main() {
  unsigned G, W, rounds, D;
  while (std::scanf("%u %u %u %u", &G, &W, &rounds, &D) == 4) {
    std::vector<uint32_t> u(D);
    uint32_t all = 0, longest = 0, active = 0, asked = 0;
    for (auto& x : u) {
      if (std::scanf("%u", &x) != 1) return 1;
      all += x;
      longest = std::max(longest, x);
      active += x != 0;
    }
    auto number = [&](uint32_t per) {
      uint32_t n = 0;
      ++asked;
      for (uint32_t x : u) n += (x + per - 1) / per;
      return n;
    };
    auto length = [&](uint32_t g) { return hd::range_length(all, std::min(g, 4096u), W); };
    uint32_t per = length(G);
    if (number(per) > G) per = hd::batch_length(all, longest, active, G, rounds, length, number);
    std::printf("%u %u\\n", per, asked);
  }
}
"""

SETUP = 16  # units that a range costs beside its own


def _lengths(tmp_path, cases):
    src, exe = tmp_path / "probe.cpp", tmp_path / "probe"
    src.write_text(PROBE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__host__=", "-D__device__=", "-D__forceinline__=inline",
                    "-I", CSRC, str(src), "-o", str(exe)], check=True, capture_output=True, text=True)
    text = "".join("%d %d %d %d %s\n" % (G, W, rounds, len(u), " ".join(map(str, u)))
                   for G, W, rounds, u in cases)
    out = subprocess.run([str(exe)], input=text, check=True, capture_output=True, text=True).stdout
    return [tuple(map(int, line.split())) for line in out.split("\n") if line]


def _loads(G, per, units):
    """Units of each workgroup, with SETUP for each range it takes."""
    load, v = [0] * G, 0
    for u in units:
        for r in range(0, u, per):
            load[v % G] += min(per, u - r) + SETUP
            v += 1
    return load, v


def _cases():
    rng = random.Random(5)
    cases = []
    for big in (4102, 16390):  # one large discharge among many small ones
        for n, small in ((7, 68), (99, 12), (199, 68), (399, 12), (511, 12), (512, 12), (599, 12), (2000, 12)):
            for G in (512, 256, 64):
                cases.append((G, 8, 2 ** 32 - 1, [big] + [small] * n))
                cases.append((G, 8, 2 ** 32 - 1, [small] * n + [big]))
    cases += [(64, 8, 2 ** 32 - 1, [396] * 24), (512, 8, 2 ** 32 - 1, [68] * 300),
              (512, 8, 2 ** 32 - 1, [0] * 90 + [500] + [0] * 600 + [7] * 3), (512, 16, 2 ** 32 - 1, [2738] * 24)]
    for _ in range(300):
        G = rng.choice([1, 2, 7, 64, 256, 512, 1000, 4096])
        D = rng.choice([2, 3, 24, 64, 65, 200, 700])
        top = rng.choice([10, 100, 1000, 20000])
        cases.append((G, rng.choice([8, 16]), 2 ** 32 - 1,
                      [0 if rng.random() < 0.1 else int(top ** rng.random()) + 1 for _ in range(D)]))
    return cases


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host C++ compiler")
def test_no_workgroup_has_much_more_than_its_share(tmp_path):
    cases = _cases()
    for (G, W, _, units), (per, asked) in zip(cases, _lengths(tmp_path, cases)):
        what = (G, W, per, len(units), max(units))
        assert per >= 1 and all((u + per - 1) // per <= 4096 for u in units), what
        assert asked <= 25, what
        load, n = _loads(G, per, units)
        # an equal share of the units and set-ups of ranges as long as a
        # workgroup has waves, or of one range per discharge
        share = sum(units) / G
        ranges = max(1, -(-sum(1 for u in units if u) // G))
        assert max(load) <= 2.0 * (share + SETUP * ranges) + 2 * W + SETUP, (what, max(load), share, n)


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host C++ compiler")
def test_one_round_where_only_one_is_allowed(tmp_path):
    # a workgroup for every range: as many workgroups as the launch was given
    # and one for every discharge more
    cases = [(G + len(u), W, 1, u) for G, W, _, u in _cases()]
    for (G, W, _, units), (per, _) in zip(cases, _lengths(tmp_path, cases)):
        assert sum((u + per - 1) // per for u in units) <= G, (G, W, per)
        assert all((u + per - 1) // per <= 4096 for u in units)
