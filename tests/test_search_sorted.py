"""The sorted form of the search: how it divides a tensor (host code, compiled here), and its errors against the two forms that a
smaller workspace selects (interval tables, where those ask for less, then direct evaluation) where stretches change hands: few and many equal values, parts
that do not fit a counter, ragged and unaligned tensors, more cuts of a group than lie in LDS at a time."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2408_06995_amd", "csrc")
PROGRAM = r"""
#include <stdio.h>
#include <initializer_list>
#include "search_split.h"
using namespace fpq;
int main()
{
    const size_t full = 256 * kSearchSortElems, third = full / 3;
    const size_t sizes[] = {131072, 480000, 480003, 4194303, 2 * third - 1, 2 * third, 2 * third + 1, 2 * third + 4, 4 * third + 3, full - 1,
                            full, full + 1, 2 * full + 3, kSearchMaxSorted - 1, kSearchMaxSorted};
    static_assert(kSearchSortElems + 3 <= 65535, "positions of a part in 16 bits");
    for (size_t n : sizes)
        for (size_t v : {(size_t)1, (size_t)4}) {
            const int parts = search_sort_parts(n), width = search_sort_width(n);
            size_t next = 0;
            if (parts % 8 || parts > 65535) return printf("parts %zu\n", n), 1;
            if (width != kSearchSortMost && width != kSearchSortMost * 2 / 3) return printf("width %zu\n", n), 1;
            if (search_count_from(n) < 4096 || search_count_from(n) > 65535) return printf("line %zu\n", n), 1;
            for (int p = 0; p < parts; ++p) {
                const SearchRange r = search_range(n / v, p, parts);
                if (r.lo != next || (r.hi - r.lo) * v > (size_t)width * 1024) return printf("share %zu\n", n), 1;
                next = r.hi;
            }
            if (next != n / v) return printf("rest %zu\n", n), 1;
        }
    // the line between the tables and the sorted form
    if (search_sorted_pays(1572863, 444) || !search_sorted_pays(1572864, 444) || search_sorted_pays(kSearchMaxSorted, 191) ||
        !search_sorted_pays(3145728, 222) || !search_sorted_pays(kSearchMaxSorted, 192) || search_sorted_pays(kSearchMaxSorted + 1, 444))
        return printf("rule\n"), 1;
    return 0;
}
"""
FP8 = [(2, 5), (3, 4), (4, 3), (5, 2)]


def test_every_part_fits_the_registers_of_a_workgroup(tmp_path):
    src, out = str(tmp_path / "split.cpp"), str(tmp_path / "split")
    with open(src, "w") as f:
        f.write(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-I", CSRC, src, "-o", out])
    subprocess.check_call([out])


def _tensor(kind, n):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    x = torch.randn(n, generator=g, device="cuda")
    if kind == "saturated":                               # many times one value at the top, zeros at the bottom
        return torch.clamp(x * 4, 0, 6)
    if kind == "two":                                     # one interval holds everything: tasks of one part each
        return torch.where(x > 0, 0.37, 0.370001)
    if kind == "levels":
        return torch.round(x * 4) * 0.01
    if kind == "wide":                                    # coarse intervals, and elements below all of them
        return x * torch.exp2(-40 * torch.rand(n, generator=g, device="cuda"))
    return x


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["normal", "saturated", "two", "levels", "wide"])
@pytest.mark.parametrize("n,offset,encodings,J", [(690001, 1, FP8 * 2, 128), (5000001, 1, FP8, 111), ((1 << 20) + 3, 0, FP8 * 2, 128),
                                                  ((1 << 20) + 3, 0, [(1, 2), (2, 1)], 128), (256 * 40960 + 5, 0, FP8, 111),
                                                  (256 * 40960 - 2, 1, FP8, 111), (256 * 40960, 0, FP8, 48), (256 * 61440 + 5, 0, FP8, 111),
                                                  (256 * 61440 - 2, 1, FP8, 111), (33000001, 0, [(4, 3), (3, 4)], 111)])
def test_the_three_forms_agree(kind, n, offset, encodings, J):
    import torch
    from paper_2408_06995_amd import binding as B
    if n * len(encodings) * J < 1572864 * 444:
        encodings = encodings * 4                         # the forms meet at this many evaluations
    x = _tensor(kind, n + offset)[offset:]
    size = B.fpq_search_workspace_size(n, len(encodings), J)
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")

    def search(bytes_of_workspace):
        mse = torch.empty(len(encodings) * J, device="cuda")
        res = torch.zeros(40, dtype=torch.uint8, device="cuda")
        B.fpq_search_format(x, encodings, J, mse, res, ws[:bytes_of_workspace])
        return mse.double(), bytes(res.cpu().numpy())

    got, chosen = search(size)
    again, chosen_again = search(size)
    assert torch.equal(got, again) and chosen == chosen_again
    table, _ = search(size - 256)
    # both in double from exact sums, reported as floats: an ulp each, and what the doubles keep where errors nearly vanish
    assert bool(((got - table).abs() <= 2.5e-7 * table + 1e-14 * table.max()).all())
    if n < 1 << 22:
        direct, _ = search(4096 + 256 + 1024 * len(encodings) * J * 4)
        assert bool(((got - direct).abs() <= 1e-4 * direct + 1e-30).all())
