"""The schedule of two powers that share their squarings, run on the host
against pow(): random exponents, and those whose buckets are empty or few
(one bit, one window, all ones), of equal and unequal lengths."""
import os
import random
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HARNESS = r"""
#include <cstdio>
#include <string>
#include "keysetup.hpp"
using namespace hebn;
static Limbs parse(const char *hex) {
  Limbs r; std::string s(hex); size_t n = s.size();
  for (size_t end = n; end > 0;) { size_t beg = end >= 8 ? end - 8 : 0;
    r.push_back((uint32_t)std::stoul(s.substr(beg, end - beg), nullptr, 16)); end = beg; }
  norm(r); return r;
}
static void out(const Limbs &x) {
  for (size_t i = x.size(); i-- > 0;) printf("%08x", x[i]);
  printf(x.empty() ? "0\n" : "\n");
}
int main(int argc, char **argv) {
  const Limbs N = parse(argv[1]), x = parse(argv[2]);
  for (int a = 3; a + 1 < argc; a += 2) {
    Limbs slot[2 * he29::kJointBuckets], state = mod(x, N);
    bool set[2 * he29::kJointBuckets] = {};
    for (uint32_t op : hekey::joint_schedule(parse(argv[a]), parse(argv[a + 1]))) {
      const uint32_t e = op & 0xFFu, what = (op >> 8) & 3u;
      for (uint32_t s = op >> 10; s > 0; --s) state = mulmod(state, state, N);
      if (e >= 2 * he29::kJointBuckets || (what != he29::kJointPut && !set[e])) return 1;
      if (what == he29::kJointPut) slot[e] = state;
      else if (what == he29::kJointLoad) state = slot[e];
      else if (what == he29::kJointTake) state = mulmod(state, slot[e], N);
      else slot[e] = mulmod(slot[e], state, N);
      set[e] = true;
    }
    out(slot[0]);
    out(state);
  }
}
"""


@pytest.fixture(scope="module")
def harness(tmp_path_factory):
    d = tmp_path_factory.mktemp("joint")
    (d / "h.cpp").write_text(HARNESS)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2504_03909_amd", "csrc"),
                    "-I", os.path.join(ROOT, "include"), "-o", str(d / "h"), str(d / "h.cpp")], check=True)
    return str(d / "h")


@pytest.mark.parametrize("bits", [64, 512, 1024])
def test_both_powers(harness, bits):
    rng = random.Random(bits)
    n = rng.getrandbits(256) | (1 << 255) | 1
    x = rng.getrandbits(256)
    pairs = [(rng.getrandbits(bits) | 1 << (bits - 1), rng.getrandbits(bits) | 1) for _ in range(4)]
    pairs += [(1, 1), (2, 1 << (bits - 1)), (31, 32), (3, (1 << bits) - 1), ((1 << bits) - 1, 1 << 5),
              (rng.getrandbits(bits) | 1, 7), (62, rng.getrandbits(bits) | 1), ((1 << bits) - 2, 30)]
    args = [f"{v:x}" for v in (n, x)] + [f"{v:x}" for fe in pairs for v in fe]
    got = [int(t, 16) for t in subprocess.run([harness] + args, capture_output=True, text=True,
                                              check=True).stdout.split()]
    assert got == [pow(x, v, n) for fe in pairs for v in fe]
