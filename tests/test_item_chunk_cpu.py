"""The length of a full bin's items in an untuned batch: never below the batch's,
equal to it where the bin is small, and the bin's serial time (its items' products,
then those that join its partials, which take half as long each) within 1.6 times
the best over the doublings of the batch's length."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HARNESS = r"""
#include <cstdio>
#include <initializer_list>
#include "hist_bucket.hpp"
static double serial(double cnt, double c, double runs) { return c / 2 + (cnt / c < 1 ? 0 : cnt / c / runs / 2); }
int main() {
  for (uint32_t rank : {0u, he::kFinalSolo - 1, he::kFinalSolo, 255u})
    for (uint32_t chunk : {1u, 8u, 16u, 100u, 256u, 1u << 20})
      for (uint64_t cnt = 0; cnt < (1ull << 32); cnt += 1 + cnt / 7) {
        const uint64_t c = he::item_chunk((uint32_t)cnt, rank, chunk);
        const double runs = rank < he::kFinalSolo ? 8 : 2;
        double best = 1e300;
        for (uint64_t x = chunk; x < (1ull << 33); x *= 2) best = best < serial(cnt, x, runs) ? best : serial(cnt, x, runs);
        const bool same = cnt > 4 * chunk || c == chunk;
        if (c < chunk || !same || serial(cnt, c, runs) > 1.6 * best) {
          printf("cnt %llu rank %u chunk %u: %llu\n", (unsigned long long)cnt, rank, chunk, (unsigned long long)c);
          return 1;
        }
      }
}
"""


def test_rule(tmp_path):
    (tmp_path / "h.cpp").write_text(HARNESS)
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover=all",
                        "-I", os.path.join(ROOT, "paper_2504_03909_amd", "csrc"), "-o", str(tmp_path / "h"),
                        str(tmp_path / "h.cpp")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(tmp_path / "h")], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
