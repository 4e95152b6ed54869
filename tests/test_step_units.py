"""Host-side check of step_units (csrc/cf_run.h): the step of a duration inside a binade, in
units of the binade's spacing.

Where it returns D > 0, adding the duration to a point of the binade's grid adds exactly D to
the significand, for every start whose result stays in the binade: seeded random starts, both
parities, and the binade's first and last significands.  Where it returns 0 the duration is
not below the binade, is subnormal, ties (an odd multiple of half the spacing) or rounds to
no step.  The header is compiled with g++ (-O2 -ffp-contract=off).
"""
import os
import subprocess
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HDR = os.path.join(ROOT, "paper_2512_14098_amd", "csrc", "cf_run.h")

DRIVER = r"""
#include <cmath>
#include <cstdio>
#include "cf_run.h"

static uint64_t sm = 0x9E3779B97F4A7C15ull;
static uint64_t next64() {  // splitmix64
  uint64_t z = (sm += 0x9E3779B97F4A7C15ull);
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}
static const uint64_t kM = (1ull << 52) - 1;
static double from(int ex, uint64_t m) { return __builtin_bit_cast(double, ((uint64_t)ex << 52) | m); }

int main() {
  long bad = 0, ties = 0, last = 0, same = 0, s53 = 0, tiny = 0, subn = 0;
  for (int i = 0; i < 400000; i++) {
    const int ex = 1 + (int)(next64() % 2045);  // biased exponent of the binade
    const int kind = i % 8;
    int s = kind == 0 ? 53 : kind == 1 ? (int)(next64() % 4) - 2 : kind == 2 ? 54 + (int)(next64() % 20)
                                                                           : 1 + (int)(next64() % 53);
    int ed = ex - s;
    if (ed < 0) ed = 0;
    if (ed > 2046) ed = 2046;
    s = ex - ed;
    uint64_t md = next64() & kM;
    if (kind == 3 || (kind == 0 && i % 3 == 0)) {  // d/u an odd multiple of 1/2
      if (s >= 1 && s <= 53) md = ((md | (1ull << 52)) & ~((2ull << (s - 1)) - 1) & kM) | ((1ull << (s - 1)) & kM);
    }
    if (kind == 4) md &= ~0xFFFFFFFull;          // few bits
    if (kind == 5) ed = 0;                       // subnormal
    const double d = from(ed, md);
    const uint64_t D = cf::step_units(d, ex);
    // the same by exact integer arithmetic: d/u = (2^52 + md) / 2^s
    const unsigned __int128 full = (unsigned __int128)(md | (1ull << 52));
    const int sh = ex - ed;
    const bool low = ed > 0 && sh > 0;
    const bool tie = low && sh <= 53 && (full * 2) % ((unsigned __int128)1 << sh) == 0 &&
                     (((full * 2) >> sh) & 1);
    const uint64_t want = !low || sh > 53 || tie ? 0
                                                 : (uint64_t)((full + ((unsigned __int128)1 << (sh - 1))) >> sh);
    if (D != want) {
      if (bad++ < 10) std::printf("UNITS d=%a ex=%d: %llu, want %llu\n", d, ex, (unsigned long long)D, (unsigned long long)want);
      continue;
    }
    ties += tie; same += ed > 0 && sh <= 0; s53 += low && sh == 53 && !tie; tiny += low && sh > 53; subn += ed == 0;
    if (D == 0 || D > kM) continue;
    for (int j = 0; j < 6; j++) {
      uint64_t m = next64() % (kM - D + 1);  // m + D <= kM
      if (j == 0) m = 0;
      if (j == 1) { m = kM - D; last++; }    // ends on the binade's last significand
      if (j == 2) m |= 1;
      if (m + D > kM) continue;
      volatile double e = from(ex, m);
      const double r = e + d;
      if (r != from(ex, m + D)) {
        if (bad++ < 10) std::printf("STEP e=%a d=%a: %a, want %a\n", (double)e, d, r, from(ex, m + D));
      }
    }
  }
  std::printf("ties %ld last %ld same %ld s53 %ld tiny %ld subnormal %ld bad %ld\n", ties, last, same, s53, tiny, subn, bad);
  return bad != 0;
}
"""


def test_step_units_is_the_step_of_every_grid_point():
    with tempfile.TemporaryDirectory() as d:
        src, exe = os.path.join(d, "units.cpp"), os.path.join(d, "units")
        with open(src, "w") as f:
            f.write(DRIVER)
        subprocess.check_call(["g++", "-O2", "-std=c++20", "-ffp-contract=off", "-I", os.path.dirname(HDR), src, "-o", exe])
        p = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    print(p.stdout)
    assert p.returncode == 0, p.stdout
    w = p.stdout.strip().splitlines()[-1].split()
    stats = dict(zip(w[0::2], map(int, w[1::2])))
    # the generator reached the cases the function treats specially
    assert stats["bad"] == 0 and min(stats[k] for k in ("ties", "last", "same", "s53", "tiny", "subnormal")) > 1000, stats
