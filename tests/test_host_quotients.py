"""The short correctly rounded quotients of the FP64 pair terms, compiled for the
host from the kernels' own source with a seed within 2^-23 of 1/sqrt(x) in place
of the hardware's: sqrt, 1/sqrt and a / x against the compiler's, for random
operands and for quotients next to a rounding boundary. (The 256 significands
next to all ones, where the quotients depend on the hardware's seeds, are tested
on the GPU.)"""
import re
import shutil
import subprocess

import pytest

from paper_1004_1932_amd import build

PROGRAM = r"""
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>
#define __device__
#define __forceinline__ inline
template <class T, class U> static T bit_cast_(const U& u) { T t; std::memcpy(&t, &u, sizeof t); return t; }
#define __builtin_bit_cast(T, v) bit_cast_<T>(v)
static unsigned max(unsigned a, unsigned b) { return a > b ? a : b; }
static unsigned min(unsigned a, unsigned b) { return a < b ? a : b; }
static uint64_t state = 88172645463325252ull;
static uint64_t rnd() { state ^= state << 13; state ^= state >> 7; return state ^= state << 17; }
static double uniform() { return (rnd() >> 11) * 0x1p-53; }
static double seed(double x) { return (1.0 / std::sqrt(x)) * (1.0 + (2.0 * uniform() - 1.0) * 0x1p-23); }
#define __builtin_amdgcn_rsq seed
@SOURCE@
int main() {
  long wrong[3] = {0, 0, 0}, tried = 0, left = 0;
  for (long n = 0; n < 300000; ++n) {
    uint64_t X; /* the significand */
    const int kind = n % 4;
    if (kind == 0) X = (1ull << 52) | (rnd() >> 12);
    else if (kind == 1) X = (1ull << 53) - 1 - rnd() % 1024;
    else if (kind == 2) X = (1ull << 53) - 1 - rnd() % (1ull << (10 + rnd() % 40));
    else X = (1ull << 52) + rnd() % 4096;
    uint64_t inv = X | 1; /* inverse of an odd X modulo 2^64 */
    for (int i = 0; i < 6; ++i) inv *= 2 - (X | 1) * inv;
    for (int parity = 0; parity < 2; ++parity) {
      const double x = std::ldexp((double)X, -52 + parity);
      Range64 rg;
      double s, ir, y;
      rcp_sqrt_exact(x, s, ir, y, rg.ones);
      rg.r2(x);
      if (!rg.ok()) { ++left; continue; }
      wrong[0] += s != std::sqrt(x);
      wrong[1] += ir != 1.0 / s;
      double a[14];
      int na = 0;
      if (X >= (1ull << 53) - 512) { ++left; continue; }
      a[na++] = 1.0 + uniform();
      a[na++] = ir;
      if (X & 1) /* a / x = m + tiny, m an odd 54-bit integer: a 2^54 = m X - c */
        for (int c = -11; c <= 11; c += 2) {
          const uint64_t m = (inv * (uint64_t)(int64_t)c) & ((1ull << 54) - 1);
          if (m < (1ull << 53) || !(m & 1)) continue;
          __int128 A = (__int128)((unsigned __int128)m * X) - c;
          A >>= 54;
          if (A > 0 && A < ((__int128)1 << 53)) a[na++] = (double)(uint64_t)A;
        }
      for (int i = 0; i < na; ++i, ++tried) wrong[2] += div_exact(a[i], x, y) != a[i] / x;
    }
  }
  std::printf("%ld %ld %ld %ld %ld\n", wrong[0], wrong[1], wrong[2], tried, left);
}
"""


def _source():
    text = (build.CSRC / "ad_kernels.hip").read_text()
    start = text.index("__device__ __forceinline__ unsigned lo_word(double x)")
    end = re.search(r"double div_exact\(double a, double x, double y\) \{.*?\n\}\n", text, re.S).end()
    return text[start:end].replace("__builtin_fma(", "std::fma(").replace("static __device__", "static")


def test_quotients_are_the_rounded_ones_where_the_rule_takes_them(tmp_path):
    cxx = shutil.which("g++")
    if not cxx:
        pytest.skip("needs g++")
    (tmp_path / "q.cpp").write_text(PROGRAM.replace("@SOURCE@", _source()))
    subprocess.run([cxx, "-O2", "-std=c++17", "-ffp-contract=off", str(tmp_path / "q.cpp"), "-o", str(tmp_path / "q")],
                   check=True, capture_output=True)
    out = subprocess.run([str(tmp_path / "q")], check=True, capture_output=True, text=True).stdout
    root, inverse, quotient, tried, left = map(int, out.split())
    assert (root, inverse, quotient) == (0, 0, 0) and tried > 1_000_000
    assert left < 200_000  # the operands put there to be left out
