"""The workspace of a batch over short keys holds what every pass writes, at every
row count of a growing store (host arithmetic of csrc/short_groups.h, compiled
by the host compiler; no GPU needed).

A pass of ng <= g queries writes ng * n scores, or ng * groups maxima and behind
those (from the offset of g queries) the keys of k groups' rows.  Neither the way
a pass goes nor the number of groups is monotone in the row count (262144 rows
are 16384 groups of 16, 262145 are 8193 of 32)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "short_groups.h"
using namespace sense;
static size_t need(int64_t n, int ng, int g, int k) {
    if (!short_by_groups(n, ng, k)) return (size_t)ng * n * 4;
    const int64_t groups = short_groups(n);
    const int64_t hits = k < groups ? k : groups;
    return short_keys_offset(groups, g) + (size_t)ng * hits * short_group_rows(n) * 8;
}
int main() {
    long bad = 0;
    const int64_t lines[] = {40, 32768, 65536, 131072, 262144, 524288, 786432, 1048576, 3000000};
    const int ks[] = {1, 31, 32, 128, 129, 1024}, gs[] = {2, 3, 16, 33, 63, 64};
    for (int64_t line : lines)
        for (int64_t off = -40; off <= 40; off += 1)
            for (int k : ks)
                for (int g : gs) {
                    const int64_t capacity = line + off;
                    if (capacity < 1) continue;
                    for (int ng = 1; ng <= g; ng += (g > 4 ? g - 1 : 1))
                        if (need(capacity, ng, g, k) > short_area_bytes(capacity, g, k)) ++bad;
                    if (off % 8) continue;
                    const size_t area = short_area_most(capacity, g, k);
                    for (int64_t n = capacity; n >= 1; n -= 1 + n / 64)
                        for (int ng = 1; ng <= g; ng += (g > 4 ? g - 1 : 1))
                            if (need(n, ng, g, k) > area || short_groups(n) > short_groups_most(capacity))
                                if (bad++ < 3)
                                    printf("capacity %lld n %lld k %d g %d ng %d\n",
                                           (long long)capacity, (long long)n, k, g, ng);
                    for (int64_t at : lines)
                        for (int64_t n = at - 2; n <= at + 2; ++n)
                            if (n >= 1 && n <= capacity && need(n, g, g, k) > area) ++bad;
                }
    // A group is at most one wave's rescore, and a million rows one block's selection.
    for (int64_t n = 1; n < 5000000; n += 997)
        if (short_group_rows(n) % 16 || short_group_rows(n) > kMaxGroupRows ||
            (n <= 64 * kSelectGroups && short_groups(n) > kSelectGroups) ||
            short_groups(n) * short_group_rows(n) < n)
            ++bad;
    printf("%ld\n", bad);
    return bad != 0;
}
"""


def test_area_holds_every_pass(tmp_path):
    (tmp_path / "check.cpp").write_text(PROGRAM)
    exe = str(tmp_path / "check")
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-I",
                           os.path.join(ROOT, "paper_2606_00021_amd", "csrc"),
                           str(tmp_path / "check.cpp"), "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout
