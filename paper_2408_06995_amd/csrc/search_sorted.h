// The sorted form of the search (part of search.hip; its intervals, candidates and sums are explained there).
//
// A cut needs the elements of one interval, and the tensor has them anywhere: walking the tensor, every element looked its interval
// up, read the list of its cuts and added each term to another candidate's sum, a cache line and an integer atomic per element and
// cut (102 of 182 us for 10.5 M elements x 444 candidates).  Here the elements come to the cuts:
//   1. search_sort_kernel     one workgroup takes a part of at most 61440 elements into registers, counts them per stretch of 2^16
//                             float values in LDS, and writes their positions inside the stretches (16 bits each) in the order of the
//                             stretches, with the stretches' offsets: x is read once, everything written goes out in whole lines;
//   2. search_lists_kernel    the cuts of 64 neighbouring intervals (4 or 16 stretches), from the candidates alone, and the work for 3;
//   3. search_counts_kernel   stretches of many elements: a workgroup counts every one of the 2^16 positions in LDS; the intervals'
//                             moments and, from prefix sums, max(0, t - l) summed for each cut take no work per element and cut;
//   4. search_terms_kernel    stretches of few elements, 64 neighbouring intervals in an eighth of the parts: element by element, with
//                             lists, moments and sums in LDS;
//   5. search_closed_kernel   per candidate and 64 intervals: the closed form over ranges of equal quantized value, found by
//                             bisection, from prefix sums of the moments; plus what the cuts add, in a fixed order.
// All sums of 3 and 4 are integers, so the order of their additions does not matter.
// Measured, 10.5 M elements x 444 candidates, us: maximum 10, sort 22, lists 12.5, counts 34, terms 24, closed forms 10.5, sums and choice
// 12: 121, against 182 by the interval tables (moments 37, closed forms 25, cuts 102).
#pragma once

constexpr int kSortGroups = kBins / 64;                       // 64 neighbouring intervals each
constexpr int kStretches = (int)(kSpan >> 16);
constexpr int sort_stride(int width) { return width * 1024 + 8; }   // 16-bit positions of a part, whole 16 bytes
constexpr int kOffStride = kStretches + 8;                    // 16-bit offsets of a part
constexpr int sort_lds_bytes(int width) { return kStretches * 4 + sort_stride(width) * 2; }
constexpr uint32_t kCountMost = 65535;                        // elements of a task (16-bit counters)
constexpr int kCountLds = 65536 * 2 + 2 * 1024 * 4;
constexpr int kTaskSlices = 8;
constexpr int kWindowCuts = 1024;                             // cuts of a group that lie in LDS at a time
constexpr int kFineGroups = kFineBins / 64, kFineStretches = 64 >> (16 - kFineShift), kCoarseStretches = 64 >> (16 - kCoarseShift);
static_assert(kStretches == 4 * 1024 && kSearchSortElems + 8 < 65536, "sort buffer");
static_assert(kFineGroups * kFineStretches + (kSortGroups - kFineGroups) * kCoarseStretches == kStretches, "stretches of the groups");

struct SortGroup {
    uint32_t base, count;                                     // its cuts
};
struct SortMoments {
    unsigned long long n, s1, s2;
};
// `count` elements of a stretch in the parts [from, to).
struct CountTask {
    uint16_t stretch, from, to, count;
};
// Tasks: a stretch of up to kCountMost elements is one, others one for each slice of the parts, or several; two in a row that do not
// fit into one have more than kCountMost elements together.
inline size_t most_tasks(size_t n)
{
    return n / search_count_from(n) + n / kCountMost * (kTaskSlices + 2) + 64;
}
struct SortedLayout {
    size_t sorted, offsets, flags, cursor, totals, tasks, groups, bases, cuts, cutsums, moments, sums, total;
    int parts, width, chunks;                                 // chunks: workgroups of search_terms_kernel per group
    int sub;                                                  // workgroups per part for the elements outside all intervals
};
inline SortedLayout sorted_layout(size_t n, int nc)
{
    SortedLayout l;
    size_t at = 0;
    auto take = [&](size_t bytes) { const size_t was = at; at += up256(bytes); return was; };
    l.parts = search_sort_parts(n);
    l.width = search_sort_width(n);
    // a workgroup of search_terms_kernel wants 32 parts at least (2 M elements: 76 us with four, 88 with eight)
    l.chunks = l.parts < 64 ? 2 : l.parts < 256 ? 4 : 8;
    l.sub = l.parts <= 256 ? 4 : 2;
    l.sorted = take((size_t)l.parts * sort_stride(l.width) * 2);
    l.offsets = take((size_t)l.parts * kOffStride * 2);
    l.flags = take((size_t)l.parts * 4);
    l.cursor = take(256);
    l.totals = take((size_t)kStretches * 4);
    l.tasks = take(most_tasks(n) * sizeof(CountTask));
    l.groups = take((size_t)kSortGroups * sizeof(SortGroup));
    l.bases = take((size_t)kSortGroups * nc * 4);
    l.cuts = take(kMaxCuts * 4);
    const size_t copies = 1 + (size_t)l.chunks;               // search_counts_kernel's, search_terms_kernel's
    l.cutsums = take(kMaxCuts * 8 * copies);
    l.moments = take((size_t)kBins * copies * sizeof(SortMoments));
    l.sums = take((size_t)(kSortGroups + l.parts * l.sub) * nc * 8);
    l.total = at;
    return l;
}

// Elements [lo, hi) of a part and, in part 0 of an aligned tensor, the last n % 4.
struct SortShare {
    size_t lo, hi, tail_lo;
    int tail;
};
__device__ __forceinline__ SortShare sort_share(const float* x, size_t n, int part, int parts)
{
    const size_t v = (reinterpret_cast<uintptr_t>(x) & 15) == 0 ? 4 : 1;
    const SearchRange r = search_range(n / v, part, parts);
    return SortShare{r.lo * v, r.hi * v, n / v * v, part == 0 ? (int)(n % v) : 0};
}

// 22 us for 42 MB (counters: LDS busy 0.35 of the cycles, 0.22 with conflicts of the counters' atomics, vector instructions 0.35).  Bound by
// its phases in a row (load, count, scan, place, write out), one workgroup per compute unit: two of 40960 elements do not fit into
// LDS, and smaller parts make shorter runs for the kernel that reads them.
template <int E>   // elements per thread
__global__ __launch_bounds__(1024) void search_sort_kernel(const float* __restrict__ x, size_t n,
                                                           const float* __restrict__ absmax_parts_, int nparts, int parts,
                                                           uint16_t* __restrict__ sorted, uint16_t* __restrict__ offsets,
                                                           uint32_t* __restrict__ flags, uint32_t* __restrict__ cursor)
{
    extern __shared__ __attribute__((aligned(16))) uint32_t sort_lds[];          // counters; positions
    __shared__ uint32_t wave_sum[16];
    uint32_t* counters = sort_lds;
    uint16_t* place = reinterpret_cast<uint16_t*>(sort_lds + kStretches);
    const int tid = threadIdx.x, part = blockIdx.x;
    const SortShare share = sort_share(x, n, part, parts);
    uint32_t b[E + 1];
    if ((reinterpret_cast<uintptr_t>(x) & 15) == 0) {
        const uint4* x4 = reinterpret_cast<const uint4*>(x);
#pragma unroll
        for (int u = 0; u < E / 4; ++u) {
            const size_t i = share.lo / 4 + (size_t)u * 1024 + tid;
            const uint4 v = i < share.hi / 4 ? x4[i] : make_uint4(0u, 0u, 0u, 0u);
            b[4 * u] = v.x;
            b[4 * u + 1] = v.y;
            b[4 * u + 2] = v.z;
            b[4 * u + 3] = v.w;
        }
    } else {
#pragma unroll
        for (int u = 0; u < E; ++u) {
            const size_t i = share.lo + (size_t)u * 1024 + tid;
            b[u] = i < share.hi ? __float_as_uint(x[i]) : 0u;
        }
    }
    b[E] = tid < share.tail ? __float_as_uint(x[share.tail_lo + tid]) : 0u;
    reinterpret_cast<uint4*>(counters)[tid] = make_uint4(0u, 0u, 0u, 0u);
    if (part == 0 && tid < 2) cursor[tid] = 0;                                   // cuts and tasks, for search_lists_kernel
    const uint32_t top = top_bits(fold_absmax(absmax_parts_, nparts, 16));       // its barrier also closes the clearing
    int outside = 0;
#pragma unroll
    for (int u = 0; u <= E; ++u) {
        b[u] &= 0x7fffffffu;
        const uint32_t rel = top - b[u];
        const bool in = rel < kSpan && b[u] >= 0x00800000u;
        if (in) atomicAdd(&counters[rel >> 16], 1u);
        outside |= !in && b[u];
    }
    outside = __syncthreads_or(outside);
    if (tid == 0) flags[part] = outside ? 1u : 0u;
    // exclusive sums: a thread takes four stretches in a row
    uint4 w = reinterpret_cast<uint4*>(counters)[tid];
    const uint32_t own = (w.x + w.y) + (w.z + w.w);
    uint32_t incl = own;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t t = __shfl_up(incl, off, 64);
        if ((tid & 63) >= off) incl += t;
    }
    if ((tid & 63) == 63) wave_sum[tid >> 6] = incl;
    __syncthreads();
    uint32_t before = incl - own, total = 0;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        if (i < (tid >> 6)) before += wave_sum[i];
        total += wave_sum[i];
    }
    w = make_uint4(before, before + w.x, before + w.x + w.y, before + w.x + w.y + w.z);
    reinterpret_cast<uint4*>(counters)[tid] = w;
    uint16_t* off_out = offsets + (size_t)part * kOffStride;
    reinterpret_cast<uint2*>(off_out)[tid] = make_uint2(w.x | (w.y << 16), w.z | (w.w << 16));
    if (tid == 0) off_out[kStretches] = (uint16_t)total;
    __syncthreads();
#pragma unroll
    for (int u = 0; u <= E; ++u) {
        const uint32_t rel = top - b[u];
        if (rel < kSpan && b[u] >= 0x00800000u) place[atomicAdd(&counters[rel >> 16], 1u)] = (uint16_t)rel;
    }
    __syncthreads();
    uint4* out = reinterpret_cast<uint4*>(sorted + (size_t)part * sort_stride(E));
    const uint4* in = reinterpret_cast<const uint4*>(place);
    for (uint32_t i = tid; i < (total + 7) / 8; i += 1024) out[i] = in[i];
}

// Interval i of group g: bits of its upper end, and its width in units of the low bits.
struct GroupBits {
    uint32_t end, width;
    __device__ __forceinline__ GroupBits(uint32_t top, int g)
    {
        const int bin0 = g * 64;
        width = bin0 < kFineBins ? 1u << kFineShift : 1u << kCoarseShift;
        end = top - (bin0 < kFineBins ? (uint32_t)bin0 << kFineShift : kFineSpan + ((uint32_t)(bin0 - kFineBins) << kCoarseShift));
    }
    __device__ __forceinline__ uint32_t upper(int i) const { return end - (uint32_t)i * width; }
    __device__ __forceinline__ uint32_t lower(int i) const { return upper(i) - (width - 1); }
    // a group lies in one binade; below the normal numbers (where `end` may have wrapped around) it has no elements
    __device__ __forceinline__ bool normal(uint32_t top) const { return end <= top && end >= 0x00800000u; }
};

// Walks the 64 intervals of a group downwards for one candidate: stretch(from, to, q) for the intervals [from, to) whose quantized
// value (of a cut interval: that of its lower end) is q, then cut(i, q2, q1) for an interval that a boundary divides.
template <typename S, typename C>
__device__ __forceinline__ void walk_group(const Cand& k, const GroupBits& b, S stretch, C cut)
{
    auto q_at = [&](uint32_t bits) { return grid_value(__uint_as_float(bits), k.r, k.c0, k.m, k.b0); };
    const float last = q_at(b.lower(63));
    float q = q_at(b.upper(0));
    int from = 0;
    for (int step = 0; step < 128 && q != last; ++step) {     // a candidate has at most 127 boundaries
        int lo = from, hi = 63;
        while (lo < hi) {                                     // the first interval whose lower end has another value
            const int mid = (lo + hi) >> 1;
            if (q_at(b.lower(mid)) != q) hi = mid;
            else lo = mid + 1;
        }
        stretch(from, lo, q);
        from = lo;
        const float qh = q_at(b.upper(lo));
        if (qh == q) {
            const float ql = q_at(b.lower(lo));
            cut(lo, qh, ql);
            q = ql;
        } else {
            q = qh;                                           // the boundary lies between two intervals
        }
    }
    stretch(from, 64, q);
}

// Elements per stretch, and the tasks of search_counts_kernel; 64 stretches per workgroup.
__device__ void make_tasks(int block, const uint16_t* __restrict__ offsets, int parts, uint32_t most, uint32_t* __restrict__ totals,
                           CountTask* __restrict__ tasks, uint32_t* __restrict__ cursor, uint32_t count_from)
{
    __shared__ uint32_t slices[kTaskSlices][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, s = block * 64 + lane;
    const int per = (parts + kTaskSlices - 1) / kTaskSlices;
    auto end_of = [&](int slice) { return min((slice + 1) * per, parts); };
    uint32_t sum = 0;
#pragma unroll 8
    for (int p = wave * per; p < end_of(wave); ++p) {
        const uint16_t* o = offsets + (size_t)p * kOffStride + s;
        sum += (uint32_t)o[1] - (uint32_t)o[0];
    }
    slices[wave][lane] = sum;
    __syncthreads();
    uint32_t total = 0;
    for (int i = 0; i < kTaskSlices; ++i) total += slices[i][lane];
    if (wave == 0) totals[s] = total;
    if (total < count_from) return;
    auto add = [&](int from, int to, uint32_t count) {
        const uint32_t at = atomicAdd(cursor, 1u);
        if (at < most) tasks[at] = CountTask{(uint16_t)s, (uint16_t)from, (uint16_t)to, (uint16_t)count};
    };
    if (total <= kCountMost) {
        if (wave == 0) add(0, parts, total);
        return;
    }
    if (!sum) return;
    if (sum <= kCountMost) {
        add(wave * per, end_of(wave), sum);
        return;
    }
    int from = wave * per;
    uint32_t held = 0;
    for (int p = from; p < end_of(wave); p += 8) {            // parts in a row, as many as a task takes
        uint32_t c[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const uint16_t* o = offsets + (size_t)min(p + u, parts - 1) * kOffStride + s;
            c[u] = p + u < end_of(wave) ? (uint32_t)o[1] - (uint32_t)o[0] : 0u;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            if (held + c[u] > kCountMost) {
                add(from, p + u, held);
                from = p + u;
                held = 0;
            }
            held += c[u];
        }
    }
    if (held) add(from, end_of(wave), held);
}

// Workgroups [0, kSortGroups): the cuts of a group, t in 1/256 units | interval << 22, those of a candidate in a row from
// bases[group][candidate]; and the copies of sums that search_counts_kernel adds to, cleared.  The rest: make_tasks.
__global__ __launch_bounds__(512) void search_lists_kernel(const float* __restrict__ absmax_parts_, int nparts, SearchArgs a,
                                                           const uint16_t* __restrict__ offsets, int parts, uint32_t task_room,
                                                           uint32_t count_from, uint32_t* __restrict__ totals, CountTask* __restrict__ tasks,
                                                           uint32_t* __restrict__ cursor, SortGroup* __restrict__ groups,
                                                           uint32_t* __restrict__ bases, uint32_t* __restrict__ cuts,
                                                           unsigned long long* __restrict__ cutsums, SortMoments* __restrict__ moments)
{
    __shared__ uint32_t wave_sum[8], start;
    const int tid = threadIdx.x, g = blockIdx.x;
    if (g >= kSortGroups) {
        make_tasks(g - kSortGroups, offsets, parts, task_room, totals, tasks, cursor + 1, count_from);
        return;
    }
    const int NC = a.n_enc * a.J;
    if (tid < 64) moments[g * 64 + tid] = SortMoments{0, 0, 0};
    const float am = fold_absmax(absmax_parts_, nparts, 8);
    const GroupBits bits(top_bits(am), g);
    if (!bits.normal(top_bits(am))) {
        if (tid == 0) groups[g] = SortGroup{0u, 0u};
        return;
    }
    constexpr int H = kSearchMaxCandidates / 512;
    uint32_t own = 0;
    unsigned long long cut_mask[H];
#pragma unroll
    for (int h = 0; h < H; ++h) {                             // candidates in pairs: a thread's cuts are in a row
        cut_mask[h] = 0;
        if (tid * H + h < NC)
            walk_group(candidate(a, am, tid * H + h), bits, [](int, int, float) {},
                       [&](int i, float, float) { cut_mask[h] |= 1ull << i; });
        own += __popcll(cut_mask[h]);
    }
    uint32_t incl = own;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t t = __shfl_up(incl, off, 64);
        if ((tid & 63) >= off) incl += t;
    }
    if ((tid & 63) == 63) wave_sum[tid >> 6] = incl;
    __syncthreads();
    uint32_t at = incl - own, total = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        if (i < (tid >> 6)) at += wave_sum[i];
        total += wave_sum[i];
    }
    if (tid == 0) {
        start = atomicAdd(cursor, total);
        if ((size_t)start + total > kMaxCuts) start = 0;      // more than any formats of eight bits have
        groups[g] = SortGroup{start, total};
    }
    __syncthreads();
    at += start;
#pragma unroll
    for (int h = 0; h < H; ++h) {
        const int c = tid * H + h;
        if (c >= NC) continue;
        bases[(size_t)g * NC + c] = at;
        if (!cut_mask[h]) continue;
        const Cand k = candidate(a, am, c);
        for (unsigned long long mask = cut_mask[h]; mask; mask &= mask - 1) {
            const int i = __ffsll(mask) - 1;
            const float xh = __uint_as_float(bits.upper(i)), xl = __uint_as_float(bits.lower(i));
            const double q2 = (double)grid_value(xh, k.r, k.c0, k.m, k.b0) * (double)k.sc;
            const double q1 = (double)grid_value(xl, k.r, k.c0, k.m, k.b0) * (double)k.sc;
            const double inv_u = ldexp(1.0, 150 - (int)(bits.upper(i) >> 23));
            double t = rint(((double)xh - 0.5 * (q1 + q2)) * inv_u * 256.0);
            t = t < 0.0 ? 0.0 : (t > 4194303.0 ? 4194303.0 : t);
            if (at < kMaxCuts) {
                cuts[at] = (uint32_t)t | ((uint32_t)i << 22);
                cutsums[at] = 0;
            }
            ++at;
        }
    }
}

// First stretch of a group, and its stretches.
struct GroupStretches {
    int first, count, shift;
    __device__ __forceinline__ explicit GroupStretches(int g)
    {
        const bool fine = g < kFineGroups;
        count = fine ? kFineStretches : kCoarseStretches;
        first = fine ? g * kFineStretches : kFineGroups * kFineStretches + (g - kFineGroups) * kCoarseStretches;
        shift = fine ? kFineShift : kCoarseShift;
    }
};

typedef unsigned short Half2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t dot2(uint32_t a, uint32_t b, uint32_t c)
{
    return __builtin_amdgcn_udot2(__builtin_bit_cast(Half2, a), __builtin_bit_cast(Half2, b), c, false);
}

// A stretch's elements per position, 16 bits each.  A thread then owns 64 positions, a wavefront 4096: a fine interval, or a quarter of
// a coarse one.  Bound by its phases in a row (clear, count, scan, cuts), one workgroup per compute unit: the counters take 128 KB
// (10.5 M elements, 34 us: vector instructions 0.46 of the cycles, LDS 0.19).
template <int WIDTH>
__global__ __launch_bounds__(1024) void search_counts_kernel(const uint16_t* __restrict__ sorted, const uint16_t* __restrict__ offsets,
                                                             uint32_t task_room, const CountTask* __restrict__ tasks,
                                                             const uint32_t* __restrict__ cursor, const SortGroup* __restrict__ groups,
                                                             const uint32_t* __restrict__ cuts,
                                                             unsigned long long* __restrict__ cutsums, SortMoments* __restrict__ moments)
{
    extern __shared__ __attribute__((aligned(16))) uint32_t counts[];            // two positions per word
    __shared__ uint32_t wave_n[16], wave_s[16];
    uint32_t* before_n = counts + 32768;                                         // of a thread's positions, in its wavefront
    uint32_t* before_s = before_n + 1024;
    uint4* counts4 = reinterpret_cast<uint4*>(counts);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t ntasks = min(cursor[1], task_room);
    for (uint32_t it = blockIdx.x; it < ntasks; it += gridDim.x) {
        const CountTask task = tasks[it];
        const int s = (int)task.stretch;
        const int fine_stretches = kFineGroups * kFineStretches;
        const int g = s < fine_stretches ? s / kFineStretches : kFineGroups + (s - fine_stretches) / kCoarseStretches;
        const GroupStretches gs(g);
        const SortGroup grp = groups[g];
        const uint32_t mask = (1u << gs.shift) - 1u;
        auto count = [&](uint32_t two, uint32_t at, uint32_t lo, uint32_t hi) {
            if (at >= lo && at < hi) atomicAdd(&counts[(two & 0xffffu) >> 1], (two & 1u) ? 0x10000u : 1u);
            if (at + 1 >= lo && at + 1 < hi) atomicAdd(&counts[two >> 17], ((two >> 16) & 1u) ? 0x10000u : 1u);
        };
        // the same for runs that may hold one value many times (saturated and constant tensors), whose additions would go one by one
        auto count_alike = [&](uint32_t two, uint32_t at, uint32_t lo, uint32_t hi) {
            if (!__all(two == (uint32_t)__builtin_amdgcn_readfirstlane((int)two) && two >> 16 == (two & 0xffffu) && at >= lo && at + 1 < hi))
                return count(two, at, lo, hi);
            const unsigned long long lanes = __ballot(1);
            const uint32_t twice = 2u * (uint32_t)__popcll(lanes);
            if (lane == __ffsll(lanes) - 1) atomicAdd(&counts[two >> 17], (two & 1u) ? twice << 16 : twice);
        };
        auto clear = [&]() {
#pragma unroll
            for (int j = 0; j < 8; ++j) counts4[j * 1024 + tid] = make_uint4(0u, 0u, 0u, 0u);
        };
        const int np = task.to - task.from;
        if (np < 16 || task.count >= 512 * np) {                                 // long runs, of fewer parts several wavefronts share one
            clear();
            __syncthreads();
            const int slots = min(np, 16), sharing = 16 / slots, share = wave / slots;
            for (int p = task.from + wave % slots; p < task.to && share < sharing; p += slots) {
                const uint16_t* o = offsets + (size_t)p * kOffStride + s;
                const uint32_t* run = reinterpret_cast<const uint32_t*>(sorted + (size_t)p * sort_stride(WIDTH));
                const uint32_t lo = o[0], hi = o[1], step = 64u * (uint32_t)sharing;
                for (uint32_t word = (lo >> 1) + 64u * (uint32_t)share + lane; 2 * word < hi; word += 8 * step) {
                    uint32_t two[8];
#pragma unroll
                    for (uint32_t u = 0; u < 8; ++u) two[u] = 2 * (word + u * step) < hi ? run[word + u * step] : 0u;
#pragma unroll
                    for (uint32_t u = 0; u < 8; ++u) count_alike(two[u], 2 * (word + u * step), lo, hi);
                }
            }
        } else {
            bool cleared = false;
            for (int pb = task.from; pb < task.to; pb += 1024) {
                const int own = pb + wave + 16 * lane;                               // lane l has the offsets of the wavefront's part l
                uint32_t o0 = 0, o1 = 0;
                if (own < task.to) {
                    o0 = offsets[(size_t)own * kOffStride + s];
                    o1 = offsets[(size_t)own * kOffStride + s + 1];
                }
                if (!cleared) clear();
                for (int j = 0; j < 64 && (j == 0 || pb + wave + 16 * j < task.to); j += 16)
                    for (uint32_t from = 0;; from += 64) {                           // 64 words of each of sixteen runs, loads first
                        uint32_t two[16];
    #pragma unroll
                        for (int u = 0; u < 16; ++u) {
                            const uint32_t lo = __builtin_amdgcn_readlane(o0, j + u), hi = __builtin_amdgcn_readlane(o1, j + u);
                            const uint32_t word = (lo >> 1) + from + lane;
                            const uint32_t* run = reinterpret_cast<const uint32_t*>(sorted + (size_t)(pb + wave + 16 * (j + u)) * sort_stride(WIDTH));
                            two[u] = lo < hi && 2 * word < hi ? run[word] : 0u;
                        }
                        if (!cleared) {
                            __syncthreads();
                            cleared = true;
                        }
                        bool more = false;
    #pragma unroll
                        for (int u = 0; u < 16; ++u) {
                            const uint32_t lo = __builtin_amdgcn_readlane(o0, j + u), hi = __builtin_amdgcn_readlane(o1, j + u);
                            if (lo < hi) count(two[u], 2 * ((lo >> 1) + from + lane), lo, hi);
                            more |= lo < hi && 2 * ((lo >> 1) + from + 64) < hi;
                        }
                        if (!more) break;
                    }
            }
        }
        __syncthreads();
        // fewer than 2^16 elements: sums of positions below 2^14 fit 32 bits
        uint32_t n = 0, s1 = 0, s2 = 0;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const uint32_t c = (uint32_t)(j + lane) & 7u;                        // neighbouring lanes on different banks
            const uint4 v = counts4[8 * tid + c];
            const uint32_t w[4] = {v.x, v.y, v.z, v.w};
            uint32_t cn = 0, c1 = 0, c2 = 0;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const uint32_t p0 = 2 * k, p1 = 2 * k + 1;
                cn = dot2(w[k], 0x10001u, cn);
                c1 = dot2(w[k], p0 | (p1 << 16), c1);
                c2 = dot2(w[k], (p0 * p0) | ((p1 * p1) << 16), c2);
            }
            n += cn;
            s1 += c1 + 8 * c * cn;
            s2 += c2 + 16 * c * c1 + 64 * c * c * cn;
        }
        const uint32_t at = (uint32_t)(64 * tid) & mask;
        unsigned long long sq = s2 + (unsigned long long)at * (2ull * s1 + (unsigned long long)at * n);
        s1 += at * n;
        uint32_t in_n = n, in_s = s1;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t tn = __shfl_up(in_n, off, 64), ts = __shfl_up(in_s, off, 64);
            if (lane >= off) {
                in_n += tn;
                in_s += ts;
            }
            sq += __shfl_xor(sq, off, 64);
        }
        before_n[tid] = in_n - n;
        before_s[tid] = in_s - s1;
        if (lane == 63) {
            wave_n[wave] = in_n;
            wave_s[wave] = in_s;
            if (in_n) {
                SortMoments* m = moments + g * 64 + (((s - gs.first) << 16 | wave << 12) >> gs.shift);
                atomicAdd(&m->n, (unsigned long long)in_n);
                atomicAdd(&m->s1, (unsigned long long)in_s);
                atomicAdd(&m->s2, sq);
            }
        }
        __syncthreads();
        for (uint32_t i = tid; i < grp.count; i += 1024) {
            const uint32_t cut = cuts[grp.base + i], t = cut & 0x3fffffu;
            const uint32_t end = min((t + 255) >> 8, mask + 1);                  // positions below `end` count
            const uint32_t pos = (cut >> 22) << gs.shift;                        // in the group
            if ((int)(pos >> 16) != s - gs.first || end == 0) continue;
            const uint32_t last = (pos & 0xffffu) + end - 1, thread = last >> 6, room = (last & 63u) + 1;
            uint32_t cn = before_n[thread], cs = before_s[thread];
            for (uint32_t w = (pos & 0xffffu) >> 12; w < thread >> 6; ++w) {     // the interval's earlier wavefronts
                cn += wave_n[w];
                cs += wave_s[w];
            }
            uint32_t bn = 0, bs = 0;
            for (uint32_t q = 0; 8 * q < room; ++q) {
                const uint4 v = counts4[8 * thread + q];
                const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                for (uint32_t k = 0; k < 4; ++k) {
                    const uint32_t p = 8 * q + 2 * k, c = p + 1 < room ? w[k] : p < room ? w[k] & 0xffffu : 0u;
                    bn = dot2(c, 0x10001u, bn);
                    bs = dot2(c, p | ((p + 1) << 16), bs);
                }
            }
            cn += bn;
            cs += bs + ((64 * thread) & mask) * bn;
            if (cn)
                atomicAdd(&cutsums[grp.base + i], (unsigned long long)t * cn - 256ull * cs);
        }
        __syncthreads();                                                         // before the next task clears the counters
    }
}

// Element by element, 24 us where it has one tenth of 10.5 M elements (all of them: 75; vector instructions 0.56 of the cycles, LDS
// 0.25).  Bound by vector instructions, of the set-up of its 4352 workgroups and of the loop over an element's cuts (1.8 on average with four encodings of eight bits x
// 111 biases; a wavefront goes round as often as the element with the most).
template <int WIDTH>
__global__ __launch_bounds__(512) void search_terms_kernel(const uint16_t* __restrict__ sorted, const uint16_t* __restrict__ offsets,
                                                           int parts, int chunks, uint32_t count_from, const uint32_t* __restrict__ totals,
                                                           const SortGroup* __restrict__ groups, const uint32_t* __restrict__ cuts,
                                                           unsigned long long* __restrict__ cutsums, SortMoments* __restrict__ moments)
{
    __shared__ unsigned long long acc[kWindowCuts], packed[64], squares[64];
    __shared__ uint32_t t_of[kWindowCuts], slot[kWindowCuts];
    __shared__ uint32_t lists[64], cursor[64];               // first cut << 16 | cuts
    __shared__ uint16_t offs[64][kCoarseStretches + 1];
    const int tid = threadIdx.x, lane = tid & 63;
    const int chunk = blockIdx.x % chunks, g = blockIdx.x / chunks;
    const GroupStretches gs(g);
    const int stretches = gs.count, shift = gs.shift;
    const uint32_t mask = (1u << shift) - 1u;
    const uint32_t mine = lane < stretches ? totals[gs.first + lane] : 0u;
    const uint32_t light = (uint32_t)__ballot(mine > 0 && mine < count_from);    // the other stretches are search_counts_kernel's
    const SortGroup grp = groups[g];
    unsigned long long* sums = cutsums + (size_t)(1 + chunk) * kMaxCuts;
    SortMoments* bins = moments + (size_t)(1 + chunk) * kBins + g * 64;
    if (!light) {
        for (uint32_t i = tid; i < grp.count; i += 512) sums[grp.base + i] = 0;
        if (tid < 64) bins[tid] = SortMoments{0, 0, 0};
        return;
    }
    uint32_t window = 0;
    do {
        const uint32_t here = min(grp.count - window, (uint32_t)kWindowCuts);
        __syncthreads();                                      // the window before has written its sums
        for (int i = tid; i < kWindowCuts; i += 512) acc[i] = 0;
        if (tid < 64) {
            cursor[tid] = 0;
            if (window == 0) packed[tid] = squares[tid] = 0;
        }
        __syncthreads();
        for (uint32_t i = tid; i < here; i += 512) atomicAdd(&cursor[cuts[grp.base + window + i] >> 22], 1u);
        __syncthreads();
        if (tid < 64) {
            const uint32_t own = cursor[tid];
            uint32_t incl = own;
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const uint32_t v = __shfl_up(incl, off, 64);
                if (tid >= off) incl += v;
            }
            lists[tid] = ((incl - own) << 16) | own;
            cursor[tid] = incl - own;
        }
        __syncthreads();
        for (uint32_t i = tid; i < here; i += 512) {
            const uint32_t c = cuts[grp.base + window + i], at = atomicAdd(&cursor[c >> 22], 1u);
            t_of[at] = c & 0x3fffffu;
            slot[at] = grp.base + window + i;
        }
        __syncthreads();
        // sixteen lanes walk a part's run: 32 elements at a time, four parts per wavefront side by side
        for (int p0 = chunk; p0 < parts; p0 += 64 * chunks) {
            for (int i = tid; i < 64 * (stretches + 1); i += 512) {
                const int j = i / (stretches + 1), k = i - j * (stretches + 1), p = p0 + j * chunks;
                offs[j][k] = p < parts ? offsets[(size_t)p * kOffStride + gs.first + k] : (uint16_t)0;
            }
            __syncthreads();
            for (int j = tid >> 4; j < 64; j += 32) {
                const uint32_t lo = offs[j][0], hi = offs[j][stretches];
                const uint32_t* run = reinterpret_cast<const uint32_t*>(sorted + (size_t)(p0 + j * chunks) * sort_stride(WIDTH));
                for (uint32_t word = (lo >> 1) + (lane & 15); lo < hi && 2 * word < hi; word += 16) {
                    const uint32_t two = run[word];
                    uint32_t pos[2] = {two & 0xffffu, two >> 16}, list[2], at[2], most = 0;
                    for (int k = 1; k < stretches; ++k) {
                        const uint32_t from = offs[j][k];
                        pos[0] += 2 * word >= from ? 0x10000u : 0u;
                        pos[1] += 2 * word + 1 >= from ? 0x10000u : 0u;
                    }
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        const bool have = 2 * word + e >= lo && 2 * word + e < hi && ((light >> (pos[e] >> 16)) & 1u);
                        if (window == 0 && have) {
                            const uint32_t low = pos[e] & mask;
                            atomicAdd(&packed[pos[e] >> shift], (unsigned long long)search_moment(low));
                            atomicAdd(&squares[pos[e] >> shift], (unsigned long long)low * low);
                        }
                        list[e] = have ? lists[pos[e] >> shift] : 0u;
                        at[e] = (pos[e] & mask) << 8;
                        most = max(most, list[e] & 0xffffu);
                    }
                    for (uint32_t k = 0; k < most; ++k)
#pragma unroll
                        for (int e = 0; e < 2; ++e) {
                            if (k >= (list[e] & 0xffffu)) continue;
                            const uint32_t c = (list[e] >> 16) + k, t = t_of[c];
                            if (t > at[e]) atomicAdd(&acc[c], (unsigned long long)(t - at[e]));
                        }
                }
            }
            __syncthreads();
        }
        __syncthreads();
        for (uint32_t i = tid; i < here; i += 512) sums[slot[i]] = acc[i];
        window += kWindowCuts;
    } while (window < grp.count);
    if (tid < 64) bins[tid] = SortMoments{search_moment_count(packed[tid]), search_moment_sum(packed[tid]), squares[tid]};
}

// Workgroups [0, kSortGroups): a group's closed forms and cuts; the rest: elements outside all intervals, `sub` workgroups for
// each part that has any.
template <int COPIES>
__global__ __launch_bounds__(512) void search_closed_kernel(const float* __restrict__ x, size_t n,
                                                            const float* __restrict__ absmax_parts_, int nparts, SearchArgs a,
                                                            int parts, int sub, const uint32_t* __restrict__ flags,
                                                            const SortMoments* __restrict__ moments,
                                                            const uint32_t* __restrict__ bases,
                                                            const unsigned long long* __restrict__ cutsums,
                                                            double* __restrict__ sums)
{
        __shared__ unsigned long long one[64][3], upto[65][3];    // moments of an interval; of the group's first i, from its upper end
    const int tid = threadIdx.x;
    const int NC = a.n_enc * a.J;
    constexpr int H = kSearchMaxCandidates / 512;
    if (blockIdx.x >= kSortGroups) {
        const int part = (blockIdx.x - kSortGroups) / sub, at = (blockIdx.x - kSortGroups) % sub;
        if (!flags[part]) return;
        const float am = fold_absmax(absmax_parts_, nparts, 8);
        const SortShare share = sort_share(x, n, part, parts);
        const size_t per = (share.hi - share.lo + sub - 1) / sub;
        const size_t lo = min(share.lo + at * per, share.hi), hi = min(lo + per, share.hi);
        double sum[H] = {};
        add_outside(x, lo, hi - lo, share.tail_lo, at == 0 ? share.tail : 0, top_bits(am), am, a, NC, sum);
#pragma unroll
        for (int h = 0; h < H; ++h)
            if (tid + 512 * h < NC) sums[(size_t)blockIdx.x * NC + tid + 512 * h] = sum[h];
        return;
    }
    const int g = blockIdx.x;
    const float am = fold_absmax(absmax_parts_, nparts, 8);
    const GroupBits bits(top_bits(am), g);
    if (tid < 64) {
        unsigned long long v[3] = {0, 0, 0};
#pragma unroll
        for (int p = 0; p < COPIES; ++p) {
            const SortMoments m = moments[(size_t)p * kBins + g * 64 + tid];
            v[0] += m.n;
            v[1] += m.s1;
            v[2] += m.s2;
        }
        for (int j = 0; j < 3; ++j) one[tid][j] = v[j];
        const unsigned long long d = (unsigned long long)tid * bits.width;
        v[2] += d * (2 * v[1] + v[0] * d);
        v[1] += v[0] * d;
        for (int j = 0; j < 3; ++j) {
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const unsigned long long t = __shfl_up(v[j], off, 64);
                if (tid >= off) v[j] += t;
            }
            upto[tid + 1][j] = v[j];
            if (tid == 0) upto[0][j] = 0;
        }
    }
    __syncthreads();
    // squares of positions below 2^20 (64 coarse intervals): fewer than 2^23 elements of a group leave room in 64 bits, with more
    // the sums are taken interval by interval
    const bool many = upto[64][0] >= (1ull << 23);
    const bool none = upto[64][0] == 0;                       // (a group below the normal numbers among them)
    const double u = ldexp(1.0, (int)(bits.end >> 23) - 150);                    // one unit of the low bits
    // elements at upper - l u against the value q: n (d - mean)^2 and, exact as integers, their spread; d = upper - q
    auto errors = [&](unsigned long long cn, unsigned long long c1, unsigned long long c2, uint32_t upper, double q) -> double {
        if (!cn) return 0.0;
        const double nn = (double)cn, off = (double)__uint_as_float(upper) - q - u * ((double)c1 / nn);
        const double spread = (double)((unsigned __int128)c2 * cn - (unsigned __int128)c1 * c1) / nn;
        return fma(nn * off, off, u * u * spread);
    };
#pragma unroll
    for (int h = 0; h < H; ++h) {
        const int c = tid + 512 * h;
        if (c >= NC) continue;
        double sum = 0.0;
        if (!none) {
            const Cand k = candidate(a, am, c);
            uint32_t at = bases[(size_t)g * NC + c];
            walk_group(
                k, bits,
                [&](int from, int to, float q) {
                    const double v = (double)q * (double)k.sc;
                    if (!many) {
                        sum += errors(upto[to][0] - upto[from][0], upto[to][1] - upto[from][1], upto[to][2] - upto[from][2],
                                      bits.end, v);
                    } else {
                        for (int i = from; i < to; ++i) sum += errors(one[i][0], one[i][1], one[i][2], bits.upper(i), v);
                    }
                },
                [&](int, float qh, float ql) {
                    unsigned long long s = 0;
#pragma unroll
                    for (int p = 0; p < COPIES; ++p) s += cutsums[(size_t)p * kMaxCuts + at];
                    ++at;
                    sum -= 2.0 * (double)(qh - ql) * (double)k.sc * u * 0.00390625 * (double)s;
                });
        }
        sums[(size_t)g * NC + c] = sum;
    }
}

// Mean squared errors: the rows of the groups, and those of the parts with elements outside all intervals.
__global__ __launch_bounds__(1024) void search_sorted_sums_kernel(const double* __restrict__ sums, int parts, int sub,
                                                                  const uint32_t* __restrict__ flags, size_t n, int NC,
                                                                  double* __restrict__ mse)
{
    __shared__ double red[64][16];
    const int col = threadIdx.x & 15, c = blockIdx.x * 16 + col, row = threadIdx.x >> 4;
    double s = 0.0;
    if (c < NC) {
        for (int r = row; r < kSortGroups; r += 64) s += sums[(size_t)r * NC + c];
        for (int r = row; r < parts * sub; r += 64)
            if (flags[r / sub]) s += sums[(size_t)(kSortGroups + r) * NC + c];
    }
    s = fold_rows(s, red);
    if (threadIdx.x < 16 && c < NC) mse[c] = s / (double)n;
}
