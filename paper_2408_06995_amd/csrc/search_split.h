// How the search divides a tensor over workgroups and packs what it counts: plain arithmetic, for host and device.
#pragma once
#include <stddef.h>
#include <stdint.h>

namespace fpq {

// A moment word holds the count of an interval above, the sum of its low bits (at most 14 each) below.  Neither overflows while
// fewer than 2^25 elements are counted into one word.
constexpr int kSearchLowBits = 14;
constexpr int kSearchCountShift = 39;
constexpr uint64_t search_moment(uint32_t low) { return ((uint64_t)1 << kSearchCountShift) | low; }
constexpr uint64_t search_moment_count(uint64_t word) { return word >> kSearchCountShift; }
constexpr uint64_t search_moment_sum(uint64_t word) { return word & (((uint64_t)1 << kSearchCountShift) - 1); }

// Units [lo, hi) of part `part` of `parts`.
struct SearchRange {
    size_t lo, hi;
};
constexpr SearchRange search_range(size_t units, size_t part, size_t parts)
{
    const size_t per = (units + parts - 1) / parts;
    const size_t lo = part * per < units ? part * per : units;
    return SearchRange{lo, lo + per < units ? lo + per : units};
}

// Copies of the interval table, one per part of the tensor: a multiple of 8 (one per XCD), 64 when that leaves a part 49152
// elements (fewer do not pay for a table), and as many more as keep a part near 2^24 elements, below what a moment word counts.
constexpr int search_parts(size_t n)
{
    const size_t p = n / 49152 / 8 * 8, least = (n / ((size_t)1 << 24) + 7) / 8 * 8;
    const size_t q = p < 8 ? 8 : (p > 64 ? 64 : p);
    return (int)(q < least ? least : q);
}
// Parts of the sorted form, a multiple of 8 (one per XCD) of at most kSearchSortElems elements (and three, the rest of an aligned
// tensor): one for each compute unit, fewer while a part has less than 16384 elements (longer runs), and multiples of
// 256 beyond.  A part's positions are counted in 16 bits, which 60 elements per thread and the rest are just below, and with the
// counters of the stretches take 136 of the 160 KB of LDS.
constexpr int kSearchSortMost = 60;
constexpr size_t kSearchSortElems = (size_t)kSearchSortMost * 1024;
constexpr size_t kSearchMaxSorted = (size_t)1 << 26;
constexpr int search_sort_parts(size_t n)
{
    const size_t small = (n + 16383) / 16384, p = (small + 7) / 8 * 8, most = 256 * kSearchSortElems;
    return (int)(n > most ? (n + most - 1) / most * 256 : p < 8 ? 8 : p > 256 ? 256 : p);
}
// Elements per thread that a part is sorted with: all of them, or two thirds where those hold a part, which asks for fewer registers and
// less LDS (10.5 M elements 120.8 and 123.9 us; with two thirds alone twice as many parts from there on, 10.6 M 143 and 124 us).
constexpr int search_sort_width(size_t n)
{
    const size_t parts = (size_t)search_sort_parts(n), one = (n + parts - 1) / parts, four = (n / 4 + parts - 1) / parts * 4;
    return (one > four ? one : four) <= kSearchSortElems * 2 / 3 ? kSearchSortMost * 2 / 3 : kSearchSortMost;
}
// Where the sorted form is used among the tensors that are large enough for either.  It saves the interval tables' time per element and
// candidate and costs more per element, most for tensors whose values crowd in few intervals.  Ratios tables / sorted for normal values
// with outliers, rectified, SiLU and GELU outputs, 444 candidates: 0.5 M elements 1.06, 1.20, 0.73, 0.80; 1 M 1.03, 1.19, 0.86,
// 0.86; 2 M 1.14, 1.25, 0.90, 0.97; 4.2 M 1.16, 1.29, 1.01, 1.06; 222 candidates, 2 M 1.05, 1.19, 0.80, 0.89; 4.2 M 1.04, 1.14,
// 0.90, 0.96; 8.4 M 1.24, 1.30, 1.19, 1.18.  Few candidates gain nothing that heavy-tailed tensors do not lose: 111, 33 M elements, normal
// values 1.09, attention probabilities 0.89, quotients of normal values 0.88.
constexpr size_t kSearchSortedWork = (size_t)3 * 524288 * 444;   // elements x candidates
constexpr bool search_sorted_pays(size_t n, int nc) { return n <= kSearchMaxSorted && nc >= 192 && n * (size_t)nc >= kSearchSortedWork; }
// Elements from which a stretch is counted by position: a task takes about 12 us of a compute unit whatever it holds, element by element
// 1 us per 1024.  As many as a stretch has on average where that is more, or heavy-tailed tensors fill most stretches just above the line
// (33 M attention probabilities x 444 candidates: 579 us from 4096 on, 534 us from 8192 on).
constexpr uint32_t search_count_from(size_t n) { return n / 4096 > 4096 ? (uint32_t)(n / 4096) : 4096u; }
// Largest tensor of the binned form.
constexpr size_t kSearchMaxBinned = (size_t)1 << 31;

}  // namespace fpq
