"""The electron launch's division of several discharges' work (work_split.h),
compiled for the host: each division is into no more ranges than the launch has
workgroups and a discharge has room for, and the launch takes little longer than
equal shares would, whatever the sizes and however many discharges there are."""
import heapq
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
// reads "groups waves D units..." and prints the workgroups of the launch, the
// length of the ranges, as the launch finds it, and the lengths it tried
int main() {
  unsigned G, W, D;
  while (std::scanf("%u %u %u", &G, &W, &D) == 3) {
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
      for (uint32_t x : u) {
        n += hd::ranges_in(x, per, 1.0f / (float)per);
        if (hd::ranges_in(x, per, 1.0f / (float)per) != (x + per - 1) / per) return ~0u;
      }
      return n;
    };
    auto length = [&](uint32_t g) { return hd::range_length(all, std::min(g, 4096u), W); };
    const uint32_t most = hd::launch_groups(D, G);
    const uint32_t per = std::max(1u, hd::batch_length(all, longest, active, G, most, length, number));
    std::printf("%u %u %u\\n", most, per, asked);
  }
}
"""

SETUP = 16  # units that a range costs beside its own


def _lengths(tmp_path, cases):
    src, exe = tmp_path / "probe.cpp", tmp_path / "probe"
    src.write_text(PROBE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__host__=", "-D__device__=", "-D__forceinline__=inline",
                    "-I", CSRC, str(src), "-o", str(exe)], check=True, capture_output=True, text=True)
    text = "".join("%d %d %d %s\n" % (G, W, len(u), " ".join(map(str, u))) for G, W, u in cases)
    out = subprocess.run([str(exe)], input=text, check=True, capture_output=True, text=True).stdout
    return [tuple(map(int, line.split())) for line in out.split("\n") if line]


def _time(G, per, units):
    """When the last workgroup ends, in units, with SETUP for each range, and the
    number of ranges; G are on the device and the others start as they end."""
    ends, n = [0] * G, 0
    for u in units:
        for r in range(0, u, per):
            heapq.heapreplace(ends, ends[0] + min(per, u - r) + SETUP)
            n += 1
    return max(ends), n


def _cases():
    rng = random.Random(5)
    cases = []
    for big in (4102, 16390):  # one large discharge among many small ones
        for n, small in ((7, 68), (99, 12), (199, 68), (399, 12), (511, 12), (512, 12), (599, 12), (2000, 12)):
            for G in (512, 256, 64):
                cases.append((G, 8, [big] + [small] * n))
                cases.append((G, 8, [small] * n + [big]))
    cases += [(64, 8, [396] * 24), (512, 8, [68] * 300),
              (512, 8, [0] * 90 + [500] + [0] * 600 + [7] * 3), (512, 16, [2738] * 24)]
    for _ in range(300):
        G = rng.choice([1, 2, 7, 64, 256, 512, 1000, 4096])
        D = rng.choice([2, 3, 24, 64, 65, 200, 700])
        top = rng.choice([10, 100, 1000, 20000])
        cases.append((G, rng.choice([8, 16]),
                      [0 if rng.random() < 0.1 else int(top ** rng.random()) + 1 for _ in range(D)]))
    return cases


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host C++ compiler")
def test_no_workgroup_has_much_more_than_its_share(tmp_path):
    cases = _cases()
    for (G, W, units), (most, per, asked) in zip(cases, _lengths(tmp_path, cases)):
        time, n = _time(G, per, units)
        what = (G, W, per, len(units), max(units), n, time)
        assert per >= 1 and n <= most and all((u + per - 1) // per <= 4096 for u in units), what
        assert asked <= 25, what
        # an equal share of the units, and the set-ups of one range per
        # workgroup or, with more discharges than workgroups, per discharge
        share = sum(units) / G
        ranges = max(1, -(-sum(1 for u in units if u) // G))
        assert time <= 2.0 * (share + SETUP * ranges) + 2 * W + SETUP, (what, share)


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host C++ compiler")
def test_ranges_in_is_exact(tmp_path):
    src, exe = tmp_path / "div.cpp", tmp_path / "div"
    src.write_text("""
#include <cstdio>
#include <initializer_list>
#include "work_split.h"
int main() {
  unsigned long bad = 0;
  auto one = [&](uint32_t u, uint32_t per) {
    if (u <= (1u << 24) && per && per <= (1u << 24))
      bad += hd::ranges_in(u, per, 1.0f / (float)per) != (uint32_t)(((uint64_t)u + per - 1) / per);
  };
  for (uint32_t per = 1; per < 3000; ++per)
    for (uint32_t u = 0; u < 3000; ++u) one(u, per);
  for (uint32_t per = 1; per < (1u << 24); per = per * 5 / 4 + 1)
    for (uint32_t u = 1; u <= (1u << 24); u = u + u / 777 + 1)
      for (uint32_t v : {u, u / per * per, u / per * per + 1, u / per * per - 1}) one(v, per);
  std::printf("%lu\\n", bad);
}
""")
    subprocess.run(["g++", "-std=c++17", "-O2", "-D__host__=", "-D__device__=", "-D__forceinline__=inline",
                    "-I", CSRC, str(src), "-o", str(exe)], check=True, capture_output=True, text=True)
    assert subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.strip() == "0"


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host C++ compiler")
def test_ranges_of_one_discharge(tmp_path):
    # all sub-chunks are covered, by no more ranges than workgroups, and the
    # last range has none while there are workgroups enough
    src, exe = tmp_path / "one.cpp", tmp_path / "one"
    src.write_text("""
#include <cstdio>
#include <initializer_list>
#include "work_split.h"
int main() {
  unsigned long bad = 0, alone = 0;
  for (uint32_t G : {1u, 2u, 7u, 64u, 256u, 512u, 4096u})
    for (uint32_t W : {8u, 16u})
      for (uint32_t f : {4u, 8u, 68u, 132u})
        for (uint32_t subs = 0; subs < 70000; subs += 1 + subs / 97) {
          const hd::Ranges x = hd::ranges_of_one(subs, f, G, W);
          const bool few = (uint64_t)G * W > subs + W + f && G > 256;
          const uint32_t start = (x.n - 1) * x.per;  // of the last range
          bad += x.n < 1 || x.n > G || x.per < 1 || (uint64_t)x.n * x.per < subs;
          bad += x.n > 1 && (uint64_t)(x.n - 1) * x.per > subs + f + x.per;
          bad += few && start < subs;
          alone += start >= subs;
        }
  std::printf("%lu %d\\n", bad, alone > 0);
}
""")
    subprocess.run(["g++", "-std=c++17", "-O2", "-D__host__=", "-D__device__=", "-D__forceinline__=inline",
                    "-I", CSRC, str(src), "-o", str(exe)], check=True, capture_output=True, text=True)
    assert subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split() == ["0", "1"]
