"""The candidate lists of a filtered batch pass hold what the pass writes, at
every row count of a growing store (host arithmetic of
csrc/filter_lists.h, compiled by the host compiler; no GPU needed).

A workspace is sized once, from the capacity; the pass over the current n rows
writes filter_slots(n) slots and up to n overflow entries per query.  The
number of workgroups, and with it the slots, falls where a block more makes
every workgroup's run longer (768 -> 769 blocks on 256 compute units: 256 ->
193 workgroups), so a smaller n can need more entries than the capacity's own
pass."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "filter_lists.h"
using namespace sense;
int main(int argc, char** argv) {
    const int64_t cus = atoll(argv[1]);
    long bad = 0;
    // Around every step of the grid up to 12 blocks a workgroup, and over a
    // coarse walk: each capacity against row counts just below it and below the
    // last steps before it.
    for (int64_t run = 1; run <= 12; ++run) {
        for (int64_t off = -2; off <= 2; ++off) {
            const int64_t blocks = run * cus + off;
            if (blocks < 1) continue;
            for (int64_t tail = -255; tail <= 0; tail += 51) {
                const int64_t capacity = blocks * kFilterRows + tail;
                const int64_t entries = filter_list_entries(capacity, capacity, cus);
                for (int64_t n = capacity; n >= 1; n -= (capacity - n < 2000 ? 1 : 997)) {
                    const int64_t need = filter_slots(n, cus) + n;
                    if (need > entries && bad++ < 3)
                        printf("capacity %lld n %lld: %lld entries, %lld needed\n",
                               (long long)capacity, (long long)n, (long long)entries,
                               (long long)need);
                }
            }
        }
    }
    // A fixed store's list is its own pass's.
    for (int64_t n = 1; n < 4 * cus * kFilterRows; n += 613)
        if (filter_list_entries(n, 0, cus) != filter_slots(n, cus) + n ||
            filter_groups(n, cus) > cus)
            ++bad;
    printf("%ld\n", bad);
    return bad != 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("filter_lists")
    (d / "check.cpp").write_text(PROGRAM)
    exe = str(d / "check")
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-I",
                           os.path.join(ROOT, "paper_2606_00021_amd", "csrc"),
                           str(d / "check.cpp"), "-o", exe])
    return exe


@pytest.mark.parametrize("cus", [256, 304, 64, 1])
def test_lists_hold_every_row_count_up_to_the_capacity(program, cus):
    r = subprocess.run([program, str(cus)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout
