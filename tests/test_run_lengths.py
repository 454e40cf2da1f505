"""The choice of run lengths for packed calls of the generic path: the same runs as a search tile by tile
finds, for a number of passes over the sequences that grows with the logarithm of the longest one."""
import os
import subprocess


CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2602_12128_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <random>
#include <vector>
#include "hla_runs.h"

int main() {
  std::mt19937_64 rng(1);
  const int64_t tok = 64;
  for (int trial = 0; trial < 3000; ++trial) {
    const int nseq = 1 + rng() % (trial % 3 ? 6 : 200);
    const int64_t heads = 1 + rng() % 40, cap = trial % 2 ? 504 : 254;
    std::vector<int64_t> len(nseq);
    int64_t longest = 1;
    for (auto& n : len) n = rng() % 4 ? rng() % 400 : rng() % 100000;  // empty ones among them
    for (auto n : len) longest = std::max(longest, (n + tok - 1) / tok);
    int64_t calls = 0;
    auto count = [&](int64_t per) {
      ++calls;
      int64_t c = 0;
      for (auto n : len) c += (n + per * tok - 1) / (per * tok);
      return c;
    };
    int64_t want = std::max<int64_t>(1, count(1) * heads / cap);
    while (count(want) * heads > cap && count(want) > nseq) ++want;
    calls = 0;
    const int64_t got = hla::tiles_per_run(heads, nseq, cap, count);
    int64_t log2 = 0;
    while ((int64_t{1} << log2) < longest) ++log2;
    if (got != want || calls > 2 * log2 + 3) {
      std::printf("trial %d: %lld tiles, want %lld; %lld counts, longest %lld\n", trial, (long long)got, (long long)want,
                  (long long)calls, (long long)longest);
      return 1;
    }
  }
  // 64 sequences of 12 heads, one of 32760 tokens
  int64_t calls = 0;
  auto count = [&](int64_t per) {
    ++calls;
    return 63 + (32760 + per * tok - 1) / (per * tok);
  };
  hla::tiles_per_run(12, 64, 254, count);
  std::printf("%lld\n", (long long)calls);
  return 0;
}
"""


def test_run_lengths_match_the_linear_search(tmp_path):
    src = tmp_path / "runs.cpp"
    src.write_text(PROGRAM)
    exe = str(tmp_path / "runs")
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", CSRC, str(src), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
    assert int(r.stdout) <= 21
    print(r.stdout)
