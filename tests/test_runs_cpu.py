"""The stream-K cut's closed forms (csrc/runs.h), built for the host: run
starts and the run of a chunk against the definition in 64-bit integers."""

import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2608_00814_amd", "csrc")

PROGRAM = r"""
#define __host__
#define __device__
#define __forceinline__ inline
#include <stdio.h>
#include <random>
#include "runs.h"
static long long wrong = 0, seen = 0;
static void check(long long C, int cus, int KC, bool spread) {
  const int B = C < cus ? (int)C : cus;
  const ooo::Runs u = ooo::cut_runs(C, B, KC, spread);
  const auto lo = [&](long long b) { return spread ? C * b / B : C / B * b + (b < C % B ? b : C % B); };
  for (int b = 0; b < B; ++b) {
    wrong += u.lo(b) != lo(b) || u.lo(b + 1) != lo(b + 1);
    const long long last = lo(b + 1) - 1, probe[3] = {lo(b), (lo(b) + last) / 2, last};
    for (long long x : probe) wrong += u.of((int)x) != b;
    wrong += last / KC - lo(b) / KC + 1 > u.seg;  // tiles the run touches
    ++seen;
  }
}
int main() {
  std::mt19937 rng(1);
  for (int spread = 0; spread < 2; ++spread)
    for (int cus : {1, 7, 240, 255, 256, 304}) {
      for (int C = 1; C < 4000; ++C) check(C, cus, 1 + C % 37, spread);
      for (int tiles : {1, 2, 8, 24, 40, 216})
        for (int KC : {1, 16, 64, 80, 144, 192, 257, 432}) check((long long)tiles * KC, cus, KC, spread);
      for (int i = 0; i < 500; ++i) check(1 + rng() % 2147483647u, cus, 1 + (int)(rng() % 4096), spread);
      check(2147483647, cus, 4096, spread);
    }
  printf("%lld %lld\n", seen, wrong);
}
"""


def test_run_cut_closed_forms(tmp_path):
    src, exe = tmp_path / "runs.cpp", tmp_path / "runs"
    src.write_text(PROGRAM)
    try:
        subprocess.run(["g++", "-O2", "-std=c++17", f"-I{CSRC}", str(src), "-o", str(exe)], check=True)
    except FileNotFoundError:
        pytest.skip("no host compiler")
    seen, wrong = map(int, subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout.split())
    assert seen > 1_000_000 and wrong == 0
