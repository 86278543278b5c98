"""The parts of the Jacobi that are plain functions of numbers (csrc/jacobi_scalar.h), compiled for the host.

LDS ranges of the column scales.  Between the last barrier of a sweep's last boundary round and the next one,
group k (1 <= k < ng) reads upper(k - 1) and group m writes the end entries of its slots, while groups in other
waves may be at either point: no entry written by one group may be one that another still reads, nor may either lie
outside the room that the kernel checks its buffer for.
"""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2503_20566_amd", "csrc")


def host_program(tmp_path, source):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(source)
    subprocess.run(["g++", "-std=c++17", "-O2", "-ffp-contract=off", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    return subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split("\n")


@pytest.mark.parametrize("maxn,nc", [(16, 2), (32, 2), (48, 2), (72, 2), (128, 2), (128, 4)])
def test_scales_of_a_sweep_share_no_lds_entry(tmp_path, maxn, nc):
    lines = host_program(tmp_path, """
#include <cstdio>
#include "jacobi_scalar.h"
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
