"""How the search divides a tensor over workgroups (csrc/search_split.h, compiled here for the host): every element in one
part, and no part so large that a moment word, which packs a count and a sum, can overflow when a whole part falls into
one interval."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2408_06995_amd", "csrc")

PROGRAM = r"""
#include <stdio.h>
#include <stdlib.h>
#include "search_split.h"
using namespace fpq;
// argv: number of elements, elements per load (4: the last n % 4 go to part 0, 1: unaligned tensor)
int main(int, char** argv)
{
    const size_t n = strtoull(argv[1], 0, 0), v = strtoull(argv[2], 0, 0), units = n / v;
    const int parts = search_parts(n);
    size_t next = 0, most = 0;
    for (int p = 0; p < parts; ++p) {
        const SearchRange r = search_range(units, p, parts);
        if (r.lo != next || r.hi < r.lo) { printf("gap\n"); return 1; }
        next = r.hi;
        const size_t here = (r.hi - r.lo) * v + (p == 0 ? n % v : 0);
        if (here > most) most = here;
    }
    if (next != units) { printf("rest\n"); return 1; }
    const uint32_t low = (1u << kSearchLowBits) - 1;
    const uint64_t word = most * search_moment(low);          // the sum of `most` equal moments, as 64-bit adds leave it
    printf("%d %zu %llu %llu %llu\n", parts, most, (unsigned long long)search_moment_count(word),
           (unsigned long long)search_moment_sum(word), (unsigned long long)kSearchMaxBinned);
    return 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("split")
    src, out = str(d / "split.cpp"), str(d / "split")
    with open(src, "w") as f:
        f.write(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-I", CSRC, src, "-o", out])
    return out


@pytest.mark.parametrize("v", [4, 1])
@pytest.mark.parametrize("n", [131072, 400000, 400003, 3 * 2 ** 20 + 1, 2 ** 30 - 1, 2 ** 30, 2 ** 30 + 5, 2 ** 31 - 257,
                               2 ** 31 - 255, 2 ** 31 - 1, 2 ** 31])
def test_a_part_in_one_interval_is_counted_whole(program, n, v):
    parts, most, count, total, limit = (int(t) for t in subprocess.check_output([program, str(n), str(v)]).split())
    assert n <= limit and parts % 8 == 0 and most * parts >= n
    assert count == most
    assert total == most * (2 ** 14 - 1)
    assert parts <= 64 or n > 2 ** 30
