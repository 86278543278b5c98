"""The parts of the Jacobi that are plain functions of numbers (csrc/jacobi_scalar.h), compiled for the host.

LDS ranges of the column scales.  Between the last barrier of a sweep's last boundary round and the next one,
group k (1 <= k < ng) reads upper(k - 1) and group m writes the end entries of its slots, while groups in other
waves may be at either point: no entry written by one group may be one that another still reads, nor may either lie
outside the room that the kernel checks its buffer for.

Rotation arithmetic, with the hardware's estimates replaced by ones that are off by up to 2^-24 of their value (u =
2^-53 below).  t = s / (|dd| + sqrt(dd^2 + g2^2)): the sum of squares is within 2 u, its root within 2 u (half of
that and its own rounding), the denominator within 3 u, the quotient within 4 u; what the refinements leave out is of
the order of 2^-68.
1 / sqrt(a): rounded once, so within 2^-54, which is 2^-53 / sqrt(2) of the smallest value, 1 / sqrt(2).
"""
import os
import subprocess

import pytest

HEAD = """
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <random>
#include <algorithm>
using std::fabs; using std::fma; using std::fmin;
#define __device__
#define __forceinline__ inline
static double off(long double v) {  // an estimate of v, off by up to 2^-24 of it
  double d = (double)v; uint64_t b; std::memcpy(&b, &d, 8);
  b ^= b >> 33; b *= 0xff51afd7ed558ccdULL; b ^= b >> 33; b *= 0xc4ceb9fe1a85ec53ULL; b ^= b >> 33;
  return (double)(v * (1 + ((double)(b >> 11) / 4503599627370496.0 - 1) * std::ldexp(1.0L, -24)));
}
static double __builtin_amdgcn_rsq(double x) {
  const long double v = 1 / std::sqrt((long double)x);
  if (x == 1.0) return 1.0;                                            // as the hardware has it
  if (v < 1 && v > 1 - std::ldexp(1.0L, -28)) return 1 - std::ldexp(1.0, -53);
  return off(v);
}
static double __builtin_amdgcn_rcp(double x) { return off(1 / (long double)x); }
#include "jacobi_scalar.h"
"""
CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2503_20566_amd", "csrc")


def host_program(tmp_path, source):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(source)
    subprocess.run(["g++", "-Wno-unknown-pragmas", "-std=c++17", "-O2", "-ffp-contract=off", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    return subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split("\n")


@pytest.mark.parametrize("maxn,nc", [(16, 2), (32, 2), (48, 2), (72, 2), (128, 2), (128, 4)])
def test_scales_of_a_sweep_share_no_lds_entry(tmp_path, maxn, nc):
    lines = host_program(tmp_path, HEAD + """
int main() {
  for (int n = 2; n <= %(maxn)d; ++n) {
    const int ng = (n + %(nc)d - 1) / %(nc)d;
    const gipeps::JacobiScales s{ng};
    printf("%%d %%d", n, gipeps::JacobiScales::room(%(maxn)d, %(nc)d));
    for (int k = 0; k < ng; ++k) printf(" %%d %%d", s.lower(k), s.upper(k));
    for (int p = 0; p < ng * %(nc)d / 2; ++p) printf(" %%d", s.end(p));
    printf("\\n");
  }
}
""" % {"maxn": maxn, "nc": nc})
    for line in filter(None, lines):
        n, room, *at = map(int, line.split())
        ng = (n + nc - 1) // nc
        lower, upper, end = at[0:2 * ng:2], at[1:2 * ng:2], at[2 * ng:]
        assert len(set(lower)) == len(set(upper)) == ng and len(set(end)) == ng * nc // 2
        for k in range(1, ng):
            for m in range(ng):
                mine = end[m * nc // 2:(m + 1) * nc // 2]
                assert m == k or upper[k - 1] not in mine, (n, "group %d reads what group %d writes" % (k, m))
        assert not set(lower) & set(upper)
        # the J rows read the entries of every slot, used or not
        assert max(lower + upper) < room and end[0] + maxn // 2 <= room


@pytest.mark.parametrize("seed", [1, 2])
def test_rotation_tangent(tmp_path, seed):
    worst = float(host_program(tmp_path, HEAD + """
int main() {
  std::mt19937_64 r(%d);
  std::normal_distribution<double> n;
  std::uniform_real_distribution<double> u;
  long double worst = 0;
  for (int i = 0; i < 1000000; ++i) {
    // angles from pi / 4 (dd = 0) down to those of the last sweep
    const double dd = i %% 100 ? n(r) * std::pow(10, -12 * u(r)) : 0.0, g2 = n(r) * std::pow(10, -14 * u(r));
    const long double x = std::sqrt((long double)dd * dd + (long double)g2 * g2);
    const long double t = (dd < 0 ? -1 : 1) * (long double)g2 / (std::fabs((long double)dd) + x);
    worst = std::max(worst, std::fabs((gipeps::rotation_tangent(dd, g2) - t) / t));
  }
  printf("%%.6Lf", worst * std::ldexp(1.0L, 53));
}
""" % seed)[0])
    assert worst <= 4.01, "%.2f units of 2^-53" % worst


def test_inverse_root_is_rounded_once(tmp_path):
    worst = float(host_program(tmp_path, HEAD + """
int main() {
  std::mt19937_64 r(3);
  std::uniform_real_distribution<double> u;
  long double worst = 0;
  for (int i = 0; i < 400000; ++i) {
    const double t = i & 1 ? u(r) : std::pow(10, -3 - 5 * u(r)), a = fma(t, t, 1.0);  // any angle; a small one
    const long double c = 1 / std::sqrt((long double)a);
    worst = std::max(worst, std::fabs((gipeps::rsqrt_1to2(a) - c) / c));
  }
  printf("%.6Lf", worst * std::ldexp(1.0L, 53));
}
""")[0])
    assert worst <= 0.5 ** 0.5 * 1.0001, "%.3f units of 2^-53" % worst
