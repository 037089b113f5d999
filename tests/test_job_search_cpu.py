"""The search for the job of an entry of a batch's flat arrays, against a scan."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HARNESS = r"""
#include <cstdio>
#include <random>
#include <vector>
#include "hist_bucket.hpp"
struct Job { uint64_t a; uint32_t b; };
int main() {
  std::mt19937 rng(5);
  for (uint32_t n : {1u, 2u, 3u, 5u, 8u, 64u, 1000u}) {
    for (int empties = 0; empties < 3; ++empties) {
      std::vector<Job> jobs(n);  // no element past the end
      uint64_t at = 0;
      for (uint32_t j = 0; j < n; ++j) {
        jobs[j] = {at, (uint32_t)at};
        if (empties == 0 || rng() % 3 >= (uint32_t)empties) at += 1 + rng() % 4;
      }
      for (uint64_t x = 0; x < at + 2; ++x) {
        uint32_t want = 0;
        while (want + 1 < n && jobs[want + 1].a <= x) ++want;
        if (he::find_job(jobs.data(), n, &Job::a, x) != want || he::find_job(jobs.data(), n, &Job::b, x) != want) {
          printf("n %u x %llu\n", n, (unsigned long long)x);
          return 1;
        }
      }
    }
  }
}
"""


def test_search_equals_scan(tmp_path):
    (tmp_path / "h.cpp").write_text(HARNESS)
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                        "-I", os.path.join(ROOT, "paper_2504_03909_amd", "csrc"), "-o", str(tmp_path / "h"),
                        str(tmp_path / "h.cpp")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(tmp_path / "h")], capture_output=True, text=True,
                       env={**os.environ, "ASAN_OPTIONS": "detect_leaks=0"})
    assert r.returncode == 0, r.stdout + r.stderr
