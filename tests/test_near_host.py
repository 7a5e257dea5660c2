"""The tables of the small heads' near form that the host makes at every launch: against their definitions, element by element and
candidate by candidate, and how long they take."""
import os
import subprocess

from paper_2512_13368_amd import build

PROGRAM = r"""
#include <chrono>
#include <cstdio>
#include <initializer_list>
#include "near_host.h"
using namespace blossom;

static bool pow2(int x) { return x > 0 && (x & (x - 1)) == 0; }

static int parts_by_trial(int units, int tiles, int waves, int slots)
{
  int best = 0, parts = 0;
  for (int p = 1; p <= (tiles + waves - 1) / waves; ++p) {
    const int rounds = (units * p + slots - 1) / slots, each = (tiles + waves * p - 1) / (waves * p);
    if (each > kMostTiles) continue;
    if (best == 0 || rounds * (2 * each + 1) < best) best = rounds * (2 * each + 1), parts = p;
  }
  return parts;
}

int main()
{
  int wrong = 0;
  for (int window = 1; window <= 17; ++window)
    for (int powers = 0; powers < 2; ++powers)
      for (int key = 0; key < 2; ++key) {
        const NearMasks m(window, powers, key);
        for (int r = 0; r < 4; ++r)
          for (int l = 0; l < 64; ++l) {
            const int x = 4 * (l >> 4) + r - (l & 15), d = key ? x : -x;
            auto seen = [&](int d) { return d >= 0 && (d < window || (powers && pow2(d))); };
            wrong += (m.own[r] >> l & 1) != (unsigned)seen(d) || (m.next[r] >> l & 1) != (unsigned)seen(d + 16);
          }
      }
  std::printf("masks %d\n", wrong);
  wrong = 0;
  for (int tiles = 1; tiles <= 1024; tiles += tiles < 130 ? 1 : 37)
    for (int units = 1; units < 100000; units = units * 5 / 4 + 1)
      for (int slots : {1024, 1280}) wrong += parts_that_end_together(units, tiles, 4, slots) != parts_by_trial(units, tiles, 4, slots);
  std::printf("parts %d\n", wrong);
  unsigned long long sum = 0;
  double best = 1e9;
  for (int run = 0; run < 20; ++run) {
    const auto t0 = std::chrono::steady_clock::now();
    for (int i = 0; i < 1000; ++i) {
      const NearMasks m(1 + i % 17, i & 1, i & 2);
      sum += m.own[i & 3] + m.next[i & 3] + parts_that_end_together(8 + i, 1024, 4, 1280);
    }
    const double ns = std::chrono::duration<double, std::nano>(std::chrono::steady_clock::now() - t0).count() / 1000;
    best = ns < best ? ns : best;
  }
  std::printf("ns %.0f (%d)\n", best, (int)(sum & 1));
}
"""


def test_tables_of_a_launch(tmp_path):
    src, exe = tmp_path / "near.cpp", tmp_path / "near"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-O2", "-std=c++17", "-I" + build.CSRC, str(src), "-o", str(exe)], check=True)
    out = dict(line.split(" ")[:2] for line in subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.splitlines())
    print(out)
    assert out["masks"] == "0" and out["parts"] == "0"
    assert int(out["ns"]) < 1000  # masks and a plan: 340 here, element by element and candidate by candidate 1700
