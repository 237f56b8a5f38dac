// Encoding and bias search of Section V-A (Algorithm 1).
//
// A candidate is an encoding (e, m) with the max value c_j = absmax * (j + 1) / J; its real-valued bias (Eq. (7) solved
// for b) is carried as the integer bias b0 = 2^(e-1) plus the scale c_j / c0, c0 = Eq. (7) at b0, so a candidate is
// exactly what fpq_quantize computes for the format (e, m, b0) and that scale.  Every candidate's sum of squared errors is
// wanted.  Three forms, chosen by elements times candidates (kSearchBinnedWork):
//
// Direct: a lane holds eight elements in registers and walks a share of the candidates over them (quantize with the
// encoder's magic-add rounding, dequantize, square): about 11 vector instructions per element and candidate.  The
// candidates are split over blockIdx.y so that a small tensor still fills the chip.
//
// Binned: a quantizer is a step function, so over an interval of magnitudes that no rounding boundary of a candidate
// cuts, the interval's count, sum and sum of squares give the candidate's error in closed form.  The magnitudes are
// sorted into intervals of 2^-11 of their binade (12 binades below the maximum; 2^-9 for 20 more): no format has two
// boundaries closer than 2^-7, so an interval is cut at most once per candidate and only by few of them.
//   1. search_bins_kernel       moments per interval as exact integers in LDS (the position inside an interval is the low
//                               bits of the float), one copy per part of the tensor;
//   2. search_intervals_kernel  adds the copies; every candidate's closed form over every interval in double, cut
//                               intervals counted as if they lay below the boundary; a list of the cuts per interval;
//   3. search_cuts_kernel       every element adds, for each candidate that cuts its interval, what the upper side changes:
//                               (x - q2)^2 - (x - q1)^2 = -2 g (x - mid), g = q2 - q1, if x > mid, else nothing (the error is
//                               continuous at the boundary, so which side a tie takes does not matter).
// The terms of step 3 arrive in any order, so they are added as integers, in units of at most 2^-60 of the candidate's sum of step
// 2 (search_base_kernel).  No element's term is larger than its own share of that sum, so nothing overflows, and together they
// are a small part of it (at most 2^-9 in tensors drawn or made to lie in cut intervals), so nothing is lost.  Every call gives the same bits, and candidates that quantize the tensor alike
// have equal errors, which the choice of the first minimum rests on.
// About five such terms per element instead of 444 evaluations.  A workgroup of step 3 that meets elements more than 32 binades
// below the maximum, or subnormal ones, reads its share again and evaluates those directly (add_outside); with such elements
// only, that costs what the direct form costs.
// Sorted (search_sorted.h): the same intervals and closed forms with the elements sorted into stretches of float values first, so that
// neither moments nor cuts cost a cache line or an atomic per element and candidate.  From kSearchSortedWork elements x candidates to
// kSearchMaxSorted elements; other tensors, and callers with less workspace than the stated size, take the interval tables, or the
// direct form where those do not fit either.  Its workspace is mostly the sorted positions, two bytes per place of a part; 444 candidates
// (the tables' in brackets): 23 MB at 1.6 M elements (25), 47 at 10.5 M (42), 58 at 10.6 M, 197 at 67 M (42).
// Measured, 444 candidates, sorted / tables / direct, us: 10.5 M elements 121 / 186 / 1758; 67 M 498 / 848; 2 M 77 / 86; 480 K - / 75 /
// 78; all of 10.5 M equal 162 / 337.  20 K elements: 17 us direct.
#include "fpq_dev.h"
#include "fpq_host.h"
#include "search_split.h"

namespace fpq {

namespace {

constexpr int kSearchElems = 8;   // elements per lane and round of the direct form

// Interval of a magnitude with bits b when the maximum lies in binade `top` (top = largest float of that binade, as bits):
// rel = top - b counts down from there.
constexpr uint32_t kFineSpan = 12u << 23, kSpan = 32u << 23;
constexpr int kFineShift = 12, kCoarseShift = 14;
constexpr int kFineBins = (int)(kFineSpan >> kFineShift);
constexpr int kBins = kFineBins + (int)((kSpan - kFineSpan) >> kCoarseShift);
constexpr int kBinGroups = 4;                       // LDS holds a quarter of the intervals: 64 in a row per group, in turn
constexpr int kGroupBins = kBins / kBinGroups;
constexpr int kBinBlocks = kBins / 64;              // workgroups of the interval kernel, 64 neighbouring intervals each
static_assert(kBins % (64 * kBinGroups) == 0 && kGroupBins * 16 <= 160 * 1024, "interval table");
static_assert(kFineShift <= kSearchLowBits && kCoarseShift <= kSearchLowBits, "moment word");

// A boundary inside an interval: an element l units below the upper end adds slope * (l - t) to its candidate's error if
// l < t.  `where` = t in 1/256 units << 10 | candidate (an element at the boundary adds nothing, so t may be rounded).
// Slopes are in units of 4^e, e the exponent of the maximum's binade: errors are squares, and those of a tensor of values around
// 10^-17 or 10^20 would leave a float's range (in these units they span 2^-103 to 2^-8).
struct Cut {
    float slope;
    uint32_t where;
};
// Number of cuts: a candidate has at most 2^(e+m) - 1 <= 127 boundaries.
constexpr size_t kMaxCuts = (size_t)kSearchMaxCandidates * 127;

struct BinnedLayout {
    size_t table, cursors, starts, cuts, sums_i, sums_c, base, shifts, total;
};
__host__ __device__ inline size_t up256(size_t v) { return (v + 255) / 256 * 256; }
constexpr int kCutBlocks = 1024;
inline BinnedLayout binned_layout(size_t n, int nc)
{
    BinnedLayout l;
    size_t at = 0;
    auto take = [&](size_t bytes) { const size_t was = at; at += up256(bytes); return was; };
    l.table = take((size_t)search_parts(n) * kBins * 16);
    l.cursors = take(256);
    l.starts = take((size_t)kBins * 4);
    l.cuts = take((kMaxCuts + 1) * sizeof(Cut));
    l.sums_i = take((size_t)kBinBlocks * nc * 8);
    l.sums_c = take((size_t)kCutBlocks * nc * 8);
    l.base = take((size_t)nc * 8);
    l.shifts = take((size_t)nc * 4);
    l.total = at;
    return l;
}

// max |x| from the per-block maxima (all threads of the workgroup call this; `waves` wavefronts), 1 for an all-zero tensor.
__device__ __forceinline__ float fold_absmax(const float* __restrict__ parts, int nparts, int waves)
{
    __shared__ float part[16];
    float v = 0.0f;
    for (int i = threadIdx.x; i < nparts; i += waves * 64) v = fmaxf(v, parts[i]);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = fmaxf(v, __shfl_xor(v, off, 64));
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = v;
    __syncthreads();
    v = part[0];
    for (int w = 1; w < waves; ++w) v = fmaxf(v, part[w]);
    return v > 0.0f ? v : 1.0f;
}

struct Cand {
    float r, sc, c0;
    int m, b0;
};
__device__ __forceinline__ float cand_max(float am, int j, int J) { return (float)((double)am * (double)(j + 1) / (double)J); }
__device__ __forceinline__ Cand candidate(const SearchArgs& a, float am, int c)
{
    const int i = c / a.J, j = c - i * a.J;
    Cand k;
    k.sc = (float)((double)cand_max(am, j, a.J) / (double)a.enc[i].c0);
    k.r = __fdiv_rn(1.0f, k.sc);
    k.c0 = a.enc[i].c0;
    k.m = a.enc[i].m;
    k.b0 = a.enc[i].b0;
    return k;
}

// Eq. (6), (9), (8) on a magnitude, as a value of the format's grid (to be multiplied by the scale).
__device__ __forceinline__ float grid_value(float ax, float r, float c0, int m, int b0)
{
    const float aa = fminf(__fmul_rn(ax, r), c0);                            // Eq. (6)
    const int P = max((int)(__float_as_uint(aa) >> 23) - 127 + b0, 1);       // Eq. (9): s = 2^(P-b-m)
    const float C = __uint_as_float((uint32_t)(P - b0 - m + 150) << 23);     // 2^23 s
    return __fsub_rn(__fadd_rn(aa, C), C);                                   // Eq. (8): rne(aa / s) s
}

// ---------------------------------------------------------------------------------- direct form

// Sum over the wavefront, valid in lane 63: row shifts, then row broadcasts, one vector instruction each.
__device__ __forceinline__ float wave_sum_last(float v)
{
#define FPQ_DPP_ADD(ctrl, rows) \
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), ctrl, rows, 0xF, true))
    FPQ_DPP_ADD(0x111, 0xF);
    FPQ_DPP_ADD(0x112, 0xF);
    FPQ_DPP_ADD(0x114, 0xF);
    FPQ_DPP_ADD(0x118, 0xF);
    FPQ_DPP_ADD(0x142, 0xA);
    FPQ_DPP_ADD(0x143, 0xC);
#undef FPQ_DPP_ADD
    return v;
}

// partial[block x][candidate]: sums of squared errors of the candidates of share blockIdx.y.
__global__ __launch_bounds__(256) void search_direct_kernel(const float* __restrict__ x, size_t n,
                                                            const float* __restrict__ absmax_parts_, int nparts, SearchArgs a,
                                                            float* __restrict__ partial)
{
    __shared__ float tab_r[kSearchMaxCandidates], tab_s[kSearchMaxCandidates];
    __shared__ float wacc[4][kSearchMaxCandidates];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int NC = a.n_enc * a.J;
    const float am = fold_absmax(absmax_parts_, nparts, 4);
    const int share = (NC + gridDim.y - 1) / gridDim.y;
    const int c_lo = blockIdx.y * share, c_hi = min(c_lo + share, NC);
    for (int c = c_lo + tid; c < c_hi; c += 256) {
        const Cand k = candidate(a, am, c);
        tab_s[c] = k.sc;
        tab_r[c] = k.r;
        wacc[0][c] = wacc[1][c] = wacc[2][c] = wacc[3][c] = 0.0f;
    }
    __syncthreads();
    const size_t chunk = (size_t)256 * kSearchElems;
    const bool aligned = (reinterpret_cast<uintptr_t>(x) & 15) == 0;
    for (size_t base = (size_t)blockIdx.x * chunk; base < n; base += (size_t)gridDim.x * chunk) {
        const size_t i0 = base + (size_t)tid * kSearchElems;
        float ax[kSearchElems];
        if (aligned && i0 + kSearchElems <= n) {
            const float4 v0 = *reinterpret_cast<const float4*>(x + i0);
            const float4 v1 = *reinterpret_cast<const float4*>(x + i0 + 4);
            ax[0] = fabsf(v0.x); ax[1] = fabsf(v0.y); ax[2] = fabsf(v0.z); ax[3] = fabsf(v0.w);
            ax[4] = fabsf(v1.x); ax[5] = fabsf(v1.y); ax[6] = fabsf(v1.z); ax[7] = fabsf(v1.w);
        } else {
#pragma unroll
            for (int k = 0; k < kSearchElems; ++k) ax[k] = (i0 + k < n) ? fabsf(x[i0 + k]) : 0.0f;   // 0 adds no error
        }
        for (int i = 0; i < a.n_enc; ++i) {
            const int m = a.enc[i].m, b0 = a.enc[i].b0;
            const float c0 = a.enc[i].c0;
            const int from = max(i * a.J, c_lo), to = min((i + 1) * a.J, c_hi);
            for (int c = from; c < to; ++c) {
                const float r = tab_r[c], sc = tab_s[c];
                float sum = 0.0f;
#pragma unroll
                for (int k = 0; k < kSearchElems; ++k) {
                    const float d = __fmaf_rn(-grid_value(ax[k], r, c0, m, b0), sc, ax[k]);
                    sum = __fmaf_rn(d, d, sum);
                }
                sum = wave_sum_last(sum);
                if (lane == 63) wacc[wave][c] += sum;
            }
        }
    }
    __syncthreads();
    for (int c = c_lo + tid; c < c_hi; c += 256)
        partial[(size_t)blockIdx.x * NC + c] = (wacc[0][c] + wacc[1][c]) + (wacc[2][c] + wacc[3][c]);
}

// ---------------------------------------------------------------------------------- binned form

__device__ __forceinline__ uint32_t top_bits(float am) { return (__float_as_uint(am) | 0x7fffffu) & 0x7fffffffu; }
__device__ __forceinline__ int top_exponent(uint32_t top) { return (int)(top >> 23) - 127; }

// Interval and position below its upper end of a magnitude; false for one outside all intervals (or NaN).
__device__ __forceinline__ bool locate(uint32_t b, uint32_t top, int& bin, uint32_t& low)
{
    const uint32_t rel = top - b;
    if (rel < kFineSpan) {
        bin = (int)(rel >> kFineShift);
        low = rel & ((1u << kFineShift) - 1u);
    } else {
        bin = kFineBins + (int)((rel - kFineSpan) >> kCoarseShift);
        low = (rel - kFineSpan) & ((1u << kCoarseShift) - 1u);
    }
    return rel < kSpan && b >= 0x00800000u;
}

// Calls f4 with the bits of the magnitudes of part `part` of `parts`, four at a time (0: no element, or a zero, which has no
// error with any candidate); 16-byte loads where alignment allows.
template <int THREADS, typename F>
__device__ __forceinline__ void for_elements(const float* __restrict__ x, size_t n, int part, int parts, F f4)
{
    if ((reinterpret_cast<uintptr_t>(x) & 15) == 0) {
        const size_t n4 = n >> 2;
        const auto [lo, hi] = search_range(n4, part, parts);
        const uint4* x4 = reinterpret_cast<const uint4*>(x);
        for (size_t i = lo + threadIdx.x; i < hi; i += 4 * THREADS) {
            uint4 v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = i + u * THREADS < hi ? x4[i + u * THREADS] : make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
            for (int u = 0; u < 4; ++u)
                f4(make_uint4(v[u].x & 0x7fffffffu, v[u].y & 0x7fffffffu, v[u].z & 0x7fffffffu, v[u].w & 0x7fffffffu));
        }
        if (part == 0 && threadIdx.x < (n & 3))
            f4(make_uint4(__float_as_uint(x[(n4 << 2) + threadIdx.x]) & 0x7fffffffu, 0u, 0u, 0u));
    } else {
        const auto [lo, hi] = search_range(n, part, parts);
        for (size_t i = lo + threadIdx.x; i < hi; i += 4 * THREADS) {
            uint32_t v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = i + u * THREADS < hi ? __float_as_uint(x[i + u * THREADS]) & 0x7fffffffu : 0u;
            f4(make_uint4(v[0], v[1], v[2], v[3]));
        }
    }
}

// Moments of the intervals of one group over one part of the tensor: {search_moment of all, sum of low^2}.  A part is
// read by one workgroup per group, all on the same XCD (workgroup ids go round-robin over the eight).
__global__ __launch_bounds__(1024) void search_bins_kernel(const float* __restrict__ x, size_t n,
                                                           const float* __restrict__ absmax_parts_, int nparts, int parts,
                                                           ulonglong2* __restrict__ table, uint32_t* __restrict__ cursors)
{
    extern __shared__ __attribute__((aligned(16))) unsigned long long bins[];   // [kGroupBins] packed, [kGroupBins] squares
    unsigned long long* packed = bins;
    unsigned long long* squares = bins + kGroupBins;
    const int group = (blockIdx.x >> 3) & (kBinGroups - 1);
    const int part = (blockIdx.x >> 5) * 8 + (blockIdx.x & 7);
    for (int i = threadIdx.x; i < 2 * kGroupBins; i += 1024) bins[i] = 0;
    if (blockIdx.x == 0 && threadIdx.x == 0) cursors[0] = 0;                     // cuts, for the next kernel
    const uint32_t top = top_bits(fold_absmax(absmax_parts_, nparts, 16));       // its barrier also closes the clearing
    auto count = [&](uint32_t b) {
        int bin;
        uint32_t low;
        if (locate(b, top, bin, low) && ((bin >> 6) & (kBinGroups - 1)) == group) {
            const int at = ((bin >> 8) << 6) | (bin & 63);
            atomicAdd(&packed[at], (unsigned long long)search_moment(low));
            atomicAdd(&squares[at], (unsigned long long)low * low);
        }
    };
    for_elements<1024>(x, n, part, parts, [&](uint4 b) {
        count(b.x);
        count(b.y);
        count(b.z);
        count(b.w);
    });
    __syncthreads();
    ulonglong2* out = table + ((size_t)group * parts + part) * kGroupBins;
    for (int i = threadIdx.x; i < kGroupBins; i += 1024) out[i] = make_ulonglong2(packed[i], squares[i]);
}

// 64 neighbouring intervals per workgroup, a candidate (or two) per thread.
__global__ __launch_bounds__(512) void search_intervals_kernel(const ulonglong2* __restrict__ table, int parts,
                                                               const float* __restrict__ absmax_parts_, int nparts, SearchArgs a,
                                                               uint32_t* __restrict__ cursors, uint32_t* __restrict__ starts,
                                                               Cut* __restrict__ cuts, double* __restrict__ sums)
{
    __shared__ unsigned long long red[8][64][3];
    __shared__ double cnt[64], lin[64], sqr[64];
    __shared__ int ncuts[64], at[64];
    const int tid = threadIdx.x;
    const int group = blockIdx.x / (kGroupBins / 64), lb = blockIdx.x - group * (kGroupBins / 64);
    const int bin0 = (lb * kBinGroups + group) * 64;
    const float am = fold_absmax(absmax_parts_, nparts, 8);
    const uint32_t top = top_bits(am);
    const uint32_t width = bin0 < kFineBins ? 1u << kFineShift : 1u << kCoarseShift;
    const uint32_t rel0 = bin0 < kFineBins ? (uint32_t)bin0 << kFineShift : kFineSpan + ((uint32_t)(bin0 - kFineBins) << kCoarseShift);
    {
        const int i = tid & 63, p = tid >> 6;
        unsigned long long n = 0, s1 = 0, s2 = 0;
        const ulonglong2* t = table + (size_t)group * parts * kGroupBins + lb * 64 + i;
        for (int q = p; q < parts; q += 8) {
            const ulonglong2 v = t[(size_t)q * kGroupBins];
            n += search_moment_count(v.x);
            s1 += search_moment_sum(v.x);
            s2 += v.y;
        }
        red[p][i][0] = n; red[p][i][1] = s1; red[p][i][2] = s2;
    }
    __syncthreads();
    auto upper = [&](int i) -> uint32_t { return top - rel0 - (uint32_t)i * width; };   // bits of the interval's upper end
    if (tid < 64) {
        unsigned long long n = 0, s1 = 0, s2 = 0;
        for (int p = 0; p < 8; ++p) { n += red[p][tid][0]; s1 += red[p][tid][1]; s2 += red[p][tid][2]; }
        const double u = n ? ldexp(1.0, (int)(upper(tid) >> 23) - 150) : 0.0;           // one unit of the low bits
        cnt[tid] = (double)n;
        lin[tid] = 2.0 * u * (double)s1;
        sqr[tid] = u * u * (double)s2;
        ncuts[tid] = 0;
    }
    __syncthreads();
    const int NC = a.n_enc * a.J;
    unsigned long long cut_mask[kSearchMaxCandidates / 512];
#pragma unroll
    for (int h = 0; h < kSearchMaxCandidates / 512; ++h) {
        cut_mask[h] = 0;
        const int c = tid + 512 * h;
        if (c >= NC) continue;
        const Cand k = candidate(a, am, c);
        double sum = 0.0;
        for (int i = 0; i < 64; ++i) {
            const double ni = cnt[i];
            if (ni == 0.0) continue;
            const float xh = __uint_as_float(upper(i)), xl = __uint_as_float(upper(i) - (width - 1));
            const float qh = grid_value(xh, k.r, k.c0, k.m, k.b0), ql = grid_value(xl, k.r, k.c0, k.m, k.b0);
            const double d = fma(-(double)ql, (double)k.sc, (double)xh);                // x - q = d - low u
            sum += fma(d, fma(ni, d, -lin[i]), sqr[i]);
            if (qh != ql) {
                cut_mask[h] |= 1ull << i;
                atomicAdd(&ncuts[i], 1);
            }
        }
        sums[(size_t)blockIdx.x * NC + c] = sum;
    }
    __syncthreads();
    if (tid < 64) {
        const int own = ncuts[tid];
        int incl = own;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int t = __shfl_up(incl, off, 64);
            if (tid >= off) incl += t;
        }
        uint32_t base = 0;
        if (tid == 63) base = atomicAdd(&cursors[0], (uint32_t)incl);
        base = __shfl(base, 63, 64);
        at[tid] = (int)base + incl - own;
        starts[bin0 + tid] = ((base + incl - own) << 11) | (uint32_t)own;               // at most 1024 cuts per interval
    }
    __syncthreads();
#pragma unroll
    for (int h = 0; h < kSearchMaxCandidates / 512; ++h) {
        unsigned long long mask = cut_mask[h];
        if (!mask) continue;
        const int c = tid + 512 * h;
        const Cand k = candidate(a, am, c);
        while (mask) {
            const int i = __ffsll(mask) - 1;
            mask &= mask - 1;
            const float xh = __uint_as_float(upper(i)), xl = __uint_as_float(upper(i) - (width - 1));
            const double q2 = (double)grid_value(xh, k.r, k.c0, k.m, k.b0) * (double)k.sc;
            const double q1 = (double)grid_value(xl, k.r, k.c0, k.m, k.b0) * (double)k.sc;
            const double inv_u = ldexp(1.0, 150 - (int)(upper(i) >> 23));
            double t = rint(((double)xh - 0.5 * (q1 + q2)) * inv_u * 256.0);
            t = t < 0.0 ? 0.0 : (t > 4194303.0 ? 4194303.0 : t);
            Cut e;
            e.slope = (float)ldexp(2.0 * (q2 - q1), (int)(upper(i) >> 23) - 150 - 2 * top_exponent(top));
            e.where = ((uint32_t)t << 10) | (uint32_t)c;
            const int p = atomicAdd(&at[i], 1);
            if ((size_t)p < kMaxCuts) cuts[p] = e;
        }
    }
}

constexpr int kOutsideRound = 4;                     // elements per thread and round of add_outside

// Squared errors of the elements of this workgroup's share (`inside` from `lo` on, then `tail` from `tail_lo` on) that lie outside all
// intervals, of candidate threadIdx.x + 512 h in sum[h] (all 512 threads call this): the elements of a round are gathered in LDS, in
// the order of the tensor, and every thread walks them with its candidates.
__device__ void add_outside(const float* __restrict__ x, size_t lo, size_t inside, size_t tail_lo, size_t tail, uint32_t top, float am,
                            const SearchArgs& a, int NC, double (&sum)[kSearchMaxCandidates / 512])
{
    __shared__ float found[512 * kOutsideRound];
    __shared__ int counts[kOutsideRound * 8];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const size_t total = inside + tail;
    // magnitudes here are below 2^(e + 1 - 32), e the exponent of the maximum's binade: scaled to below 2^60, the squares of
    // values up to 120 binades smaller stay normal numbers
    const int shift = 60 + 31 - top_exponent(top);
    Cand k[kSearchMaxCandidates / 512];
#pragma unroll
    for (int h = 0; h < kSearchMaxCandidates / 512; ++h) k[h] = candidate(a, am, min(tid + 512 * h, NC - 1));
    for (size_t base = 0; base < total; base += 512 * kOutsideRound) {
        float value[kOutsideRound];
        unsigned long long mask[kOutsideRound];
#pragma unroll
        for (int u = 0; u < kOutsideRound; ++u) {
            const size_t j = base + (size_t)u * 512 + tid;
            const size_t i = j < inside ? lo + j : tail_lo + (j - inside);
            const uint32_t b = j < total ? __float_as_uint(x[i]) & 0x7fffffffu : 0u;
            int bin;
            uint32_t low;
            const bool take = b && !locate(b, top, bin, low);
            mask[u] = __ballot(take);
            value[u] = take ? __uint_as_float(b) : -1.0f;
            if (lane == 0) counts[u * 8 + wave] = __popcll(mask[u]);
        }
        __syncthreads();
        int at[kOutsideRound], count = 0;
#pragma unroll
        for (int u = 0; u < kOutsideRound; ++u)
            for (int w = 0; w < 8; ++w) {
                if (w == wave) at[u] = count;
                count += counts[u * 8 + w];
            }
#pragma unroll
        for (int u = 0; u < kOutsideRound; ++u)
            if ((mask[u] >> lane) & 1) found[at[u] + __popcll(mask[u] & ((1ull << lane) - 1))] = value[u];
        __syncthreads();
        for (int i = 0; i < count; i += 4) {
#pragma unroll
            for (int h = 0; h < kSearchMaxCandidates / 512; ++h) {
                if (512 * h >= NC) continue;
                float four = 0.0f;
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    if (i + u >= count) continue;
                    const float e = found[i + u];
                    const float d = ldexpf(__fmaf_rn(-grid_value(e, k[h].r, k[h].c0, k[h].m, k[h].b0), k[h].sc, e), shift);
                    four = __fmaf_rn(d, d, four);
                }
                sum[h] += (double)four;
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int h = 0; h < kSearchMaxCandidates / 512; ++h) sum[h] = ldexp(sum[h], -2 * shift);
}

// Sum over the 64 rows of a workgroup of 16 x 64 threads, always in the same order, valid in the first 16 threads.
__device__ __forceinline__ double fold_rows(double s, double (&red)[64][16])
{
    const int col = threadIdx.x & 15, row = threadIdx.x >> 4;
    red[row][col] = s;
    __syncthreads();
    for (int off = 32; off > 0; off >>= 1) {
        if (row < off) red[row][col] += red[row + off][col];
        __syncthreads();
    }
    return red[0][col];
}

// Sum of a column of `rows` sums per candidate, candidate blockIdx.x * 16 + threadIdx.x % 16 of NC: 64 rows at a time, always in
// the same order.  Valid in the first 16 of the 1024 threads; all of them call this.
template <typename T>
__device__ __forceinline__ double column_sum(const T* __restrict__ sums, int rows, int NC, double (&red)[64][16])
{
    const int col = threadIdx.x & 15, c = blockIdx.x * 16 + col, row = threadIdx.x >> 4;
    double s = 0.0;
    if (c < NC)
        for (int r = row; r < rows; r += 64) s += (double)sums[(size_t)r * NC + c];
    return fold_rows(s, red);
}

// Closed forms of all intervals per candidate, and the unit of the terms that the cuts add to it: 2^-shift of the slopes' unit,
// the power of two that makes the sum less than 2^61.
__global__ __launch_bounds__(1024) void search_base_kernel(const double* __restrict__ sums, int rows,
                                                           const float* __restrict__ absmax_parts_, int nparts, int NC,
                                                           double* __restrict__ base, int* __restrict__ shifts)
{
    __shared__ double red[64][16];
    const double s = column_sum(sums, rows, NC, red);
    const int e = top_exponent(top_bits(fold_absmax(absmax_parts_, nparts, 16)));
    const int c = blockIdx.x * 16 + threadIdx.x;
    if (threadIdx.x < 16 && c < NC) {
        base[c] = s;
        // no sum, no elements in cut intervals; an infinite one or NaN keeps whatever is added
        shifts[c] = s > 0.0 && s < __builtin_huge_val() ? 60 - ilogb(s) + 2 * e : 0;
    }
}

// What the upper sides of the cut intervals change, per candidate, and the errors of the elements outside all intervals.
__global__ __launch_bounds__(512) void search_cuts_kernel(const float* __restrict__ x, size_t n,
                                                          const float* __restrict__ absmax_parts_, int nparts, SearchArgs a,
                                                          const uint32_t* __restrict__ starts, const Cut* __restrict__ cuts,
                                                          const int* __restrict__ shifts, double* __restrict__ sums)
{
    __shared__ unsigned long long acc[kSearchMaxCandidates];     // two's complement, in units of 2^-shift of the slopes' unit
    __shared__ int shift[kSearchMaxCandidates];
    const int NC = a.n_enc * a.J;
    for (int c = threadIdx.x; c < NC; c += 512) {
        acc[c] = 0;
        shift[c] = shifts[c];
    }
    const float am = fold_absmax(absmax_parts_, nparts, 8);                              // its barrier also closes the clearing
    const uint32_t top = top_bits(am);
    int outside = 0;
    // four elements side by side: the loads of a step (first the lists' places, then their next entries) are independent
    for_elements<512>(x, n, blockIdx.x, gridDim.x, [&](uint4 b4) {
        const uint32_t b[4] = {b4.x, b4.y, b4.z, b4.w};
        uint32_t left[4], at[4], most = 0;
        float l[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            int bin;
            uint32_t low;
            const bool in = locate(b[k], top, bin, low);
            const uint32_t s = in ? starts[bin] : 0u;
            at[k] = s >> 11;
            left[k] = s & 2047u;
            l[k] = (float)low;
            most = max(most, left[k]);
            outside |= !in && b[k];
        }
        auto add = [&](uint32_t slope, uint32_t where, float low) {
            const float v = __uint_as_float(slope) * (low - (float)(where >> 10) * 0.00390625f);
            if (v < 0.0f) atomicAdd(&acc[where & 1023u], (unsigned long long)(long long)ldexpf(v, shift[where & 1023u]));
        };
        for (uint32_t i = 0; i < most; i += 2) {
            uint4 e[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                e[k] = make_uint4(0u, 0u, 0u, 0u);
                if (i < left[k]) __builtin_memcpy(&e[k], cuts + at[k] + i, 16);      // two entries; the list's end has slack
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                add(e[k].x, e[k].y, l[k]);
                add(i + 1 < left[k] ? e[k].z : 0u, e[k].w, l[k]);
            }
        }
    });
    double sum[kSearchMaxCandidates / 512] = {};
    if (__syncthreads_or(outside)) {
        // the elements that for_elements gives this part: a range, and the last n % 4 in part 0
        const size_t v = (reinterpret_cast<uintptr_t>(x) & 15) == 0 ? 4 : 1;
        const SearchRange range = search_range(n / v, blockIdx.x, gridDim.x);
        add_outside(x, range.lo * v, (range.hi - range.lo) * v, n / v * v, blockIdx.x == 0 ? n % v : 0, top, am, a, NC, sum);
    }
#pragma unroll
    for (int h = 0; h < kSearchMaxCandidates / 512; ++h) {
        const int c = threadIdx.x + 512 * h;
        if (c < NC) sums[(size_t)blockIdx.x * NC + c] = ldexp((double)(long long)acc[c], 2 * top_exponent(top) - shift[c]) + sum[h];
    }
}

// ---------------------------------------------------------------------------------- sorted form

#include "search_sorted.h"

// ---------------------------------------------------------------------------------- sums over workgroups, the choice

// Mean squared errors from the rows of partial sums of either form (base: NULL, or what they are added to).
template <typename T>
__global__ __launch_bounds__(1024) void search_reduce_kernel(const T* __restrict__ sums, int rows, const double* __restrict__ base,
                                                             size_t n, int NC, double* __restrict__ mse)
{
    __shared__ double red[64][16];
    const double s = column_sum(sums, rows, NC, red);
    const int c = blockIdx.x * 16 + threadIdx.x;
    if (threadIdx.x < 16 && c < NC) mse[c] = (base ? base[c] + s : s) / (double)n;
}

// Every candidate's mean squared error (from `mse`, or summed here over the rows of the direct form) and the choice: the
// first minimum in the order of Algorithm 1 (encodings outer, biases inner).
__global__ __launch_bounds__(1024) void search_select_kernel(const double* __restrict__ mse_in, const float* __restrict__ partial,
                                                             int rows, size_t n, const float* __restrict__ absmax_parts_,
                                                             int nparts, SearchArgs a, float* __restrict__ mse_out,
                                                             fpq_search_result* __restrict__ result)
{
    __shared__ double best_v[16];
    __shared__ int best_i[16];
    const int NC = a.n_enc * a.J, c = threadIdx.x;
    const float am = fold_absmax(absmax_parts_, nparts, 16);
    double v = 0.0;
    int at = kSearchMaxCandidates;
    if (c < NC) {
        if (mse_in) {
            v = mse_in[c];
        } else {
            double s = 0.0;
            int r = 0;
            for (; r + 8 <= rows; r += 8) {
                float t[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) t[k] = partial[(size_t)(r + k) * NC + c];
#pragma unroll
                for (int k = 0; k < 8; ++k) s += (double)t[k];
            }
            for (; r < rows; ++r) s += (double)partial[(size_t)r * NC + c];
            v = n ? s / (double)n : 0.0;
        }
        if (mse_out) mse_out[c] = (float)v;
        at = c;
    }
    const double own = v;
    if (!(v == v)) v = __builtin_huge_val();         // an error that is no number is as bad as an infinite one: never less than another
    auto take = [&](double ov, int oi) {
        if (oi < kSearchMaxCandidates && (at == kSearchMaxCandidates || ov < v || (ov == v && oi < at))) {
            v = ov;
            at = oi;
        }
    };
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const double ov = __shfl_xor(v, off, 64);
        const int oi = __shfl_xor(at, off, 64);
        take(ov, oi);
    }
    if ((c & 63) == 0) { best_v[c >> 6] = v; best_i[c >> 6] = at; }
    __syncthreads();
    if (c == 0) {
        for (int w = 1; w < 16; ++w) take(best_v[w], best_i[w]);
        const int i = at / a.J, j = at - i * a.J;
        const float cj = cand_max(am, j, a.J);
        const int e = a.enc[i].e, m = a.enc[i].m;
        result->encoding = i;
        result->bias_index = j;
        result->ebits = e;
        result->mbits = m;
        result->int_bias = a.enc[i].b0;
        result->maxval = cj;
        result->scale = (float)((double)cj / (double)a.enc[i].c0);
        result->mse = (float)(at == 0 ? own : v);    // thread 0's own candidate is the first one
        // Eq. (7) solved for the bias: c = (2 - 2^-m) 2^(2^e - b - 1)
        result->real_bias = (float)((double)((1 << e) - 1) - log2((double)cj / (2.0 - exp2((double)-m))));
    }
}

// The interval tables have a cost of their own (about 73 us: launches, the candidates' walks, the tables written and read once, whatever
// n is); the direct form takes 0.13 us per 1024 elements at 444 candidates, in steps of a full chip.  450000 elements: 78 us direct, 73
// tables; 500000: 78 and 75.
constexpr size_t kSearchBinnedWork = (size_t)480000 * 444;   // elements x candidates
bool binned_pays(size_t n, int nc) { return n * (size_t)nc >= kSearchBinnedWork && n >= 131072 && n <= kSearchMaxBinned; }

}  // namespace

size_t search_binned_bytes(size_t n, int nc)
{
    return !binned_pays(n, nc) ? 0 : search_sorted_pays(n, nc) ? sorted_layout(n, nc).total : binned_layout(n, nc).total;
}

int launch_search(const float* x, size_t n, const SearchArgs& a, const float* maxparts, float* partial, size_t partial_bytes,
                  float* mse_out, fpq_search_result* result, hipStream_t st)
{
    const int NC = a.n_enc * a.J;
    const int nparts = absmax_parts(n);
    const double* mse = nullptr;
    int rows = search_blocks(n);
    if (binned_pays(n, NC) && search_sorted_pays(n, NC) && partial_bytes >= sorted_layout(n, NC).total + up256((size_t)NC * 8)) {
        const SortedLayout l = sorted_layout(n, NC);
        uint8_t* ws = reinterpret_cast<uint8_t*>(partial);
        uint16_t* sorted = reinterpret_cast<uint16_t*>(ws + l.sorted);
        uint16_t* offsets = reinterpret_cast<uint16_t*>(ws + l.offsets);
        uint32_t* flags = reinterpret_cast<uint32_t*>(ws + l.flags);
        uint32_t* cursor = reinterpret_cast<uint32_t*>(ws + l.cursor);
        uint32_t* totals = reinterpret_cast<uint32_t*>(ws + l.totals);
        CountTask* tasks = reinterpret_cast<CountTask*>(ws + l.tasks);
        SortGroup* groups = reinterpret_cast<SortGroup*>(ws + l.groups);
        uint32_t* bases = reinterpret_cast<uint32_t*>(ws + l.bases);
        uint32_t* cuts = reinterpret_cast<uint32_t*>(ws + l.cuts);
        unsigned long long* cutsums = reinterpret_cast<unsigned long long*>(ws + l.cutsums);
        SortMoments* moments = reinterpret_cast<SortMoments*>(ws + l.moments);
        double* sums = reinterpret_cast<double*>(ws + l.sums);
        double* mse_w = reinterpret_cast<double*>(ws + l.total);
        constexpr int narrow = kSearchSortMost * 2 / 3;
        const bool two_thirds = l.width == narrow;
        auto sort = two_thirds ? search_sort_kernel<narrow> : search_sort_kernel<kSearchSortMost>;
        auto counts = two_thirds ? search_counts_kernel<narrow> : search_counts_kernel<kSearchSortMost>;
        auto terms = two_thirds ? search_terms_kernel<narrow> : search_terms_kernel<kSearchSortMost>;
        static std::atomic<uint64_t> allowed_sort[2]{}, allowed_counts[2]{};      // per instantiation
        if (!allow_dynamic_lds(reinterpret_cast<const void*>(sort), sort_lds_bytes(l.width), allowed_sort[two_thirds]) ||
            !allow_dynamic_lds(reinterpret_cast<const void*>(counts), kCountLds, allowed_counts[two_thirds]))
            return FPQ_ERR_LAUNCH;
        hipLaunchKernelGGL(sort, dim3(l.parts), dim3(1024), sort_lds_bytes(l.width), st, x, n, maxparts, nparts, l.parts, sorted, offsets,
                           flags, cursor);
        const uint32_t room = (uint32_t)most_tasks(n), from = search_count_from(n);
        hipLaunchKernelGGL(search_lists_kernel, dim3(kSortGroups + kStretches / 64), dim3(512), 0, st, maxparts, nparts, a, offsets, l.parts,
                           room, from, totals, tasks, cursor, groups, bases, cuts, cutsums, moments);
        hipLaunchKernelGGL(counts, dim3(256), dim3(1024), kCountLds, st, sorted, offsets, room, tasks, cursor, groups, cuts,
                           cutsums, moments);
        hipLaunchKernelGGL(terms, dim3(kSortGroups * l.chunks), dim3(512), 0, st, sorted, offsets, l.parts, l.chunks, from, totals, groups,
                           cuts, cutsums, moments);
        auto closed = l.chunks == 2 ? search_closed_kernel<3> : l.chunks == 4 ? search_closed_kernel<5> : search_closed_kernel<9>;
        hipLaunchKernelGGL(closed, dim3(kSortGroups + l.parts * l.sub), dim3(512), 0, st, x, n, maxparts, nparts, a, l.parts, l.sub, flags,
                           moments, bases, cutsums, sums);
        hipLaunchKernelGGL(search_sorted_sums_kernel, dim3((NC + 15) / 16), dim3(1024), 0, st, sums, l.parts, l.sub, flags, n, NC, mse_w);
        mse = mse_w;
    } else if (binned_pays(n, NC) && partial_bytes >= binned_layout(n, NC).total + up256((size_t)NC * 8)) {
        const BinnedLayout l = binned_layout(n, NC);
        uint8_t* ws = reinterpret_cast<uint8_t*>(partial);
        ulonglong2* table = reinterpret_cast<ulonglong2*>(ws + l.table);
        uint32_t* cursors = reinterpret_cast<uint32_t*>(ws + l.cursors);
        uint32_t* starts = reinterpret_cast<uint32_t*>(ws + l.starts);
        Cut* cuts = reinterpret_cast<Cut*>(ws + l.cuts);
        double* sums_i = reinterpret_cast<double*>(ws + l.sums_i);
        double* sums_c = reinterpret_cast<double*>(ws + l.sums_c);
        double* base = reinterpret_cast<double*>(ws + l.base);
        int* shifts = reinterpret_cast<int*>(ws + l.shifts);
        double* mse_w = reinterpret_cast<double*>(ws + l.total);
        const int parts = search_parts(n);
        constexpr int lds = kGroupBins * 16;
        static std::atomic<uint64_t> allowed{0};
        if (!allow_dynamic_lds(reinterpret_cast<const void*>(search_bins_kernel), lds, allowed)) return FPQ_ERR_LAUNCH;
        hipLaunchKernelGGL(search_bins_kernel, dim3(parts * kBinGroups), dim3(1024), lds, st, x, n, maxparts, nparts, parts, table,
                           cursors);
        hipLaunchKernelGGL(search_intervals_kernel, dim3(kBinBlocks), dim3(512), 0, st, table, parts, maxparts, nparts, a, cursors,
                           starts, cuts, sums_i);
        hipLaunchKernelGGL(search_base_kernel, dim3((NC + 15) / 16), dim3(1024), 0, st, sums_i, kBinBlocks, maxparts, nparts, NC, base,
                           shifts);
        const int cb = (int)(n / 4096 < kCutBlocks ? (n / 4096 > 0 ? n / 4096 : 1) : kCutBlocks);
        hipLaunchKernelGGL(search_cuts_kernel, dim3(cb), dim3(512), 0, st, x, n, maxparts, nparts, a, starts, cuts, shifts,
                           sums_c);
        hipLaunchKernelGGL(search_reduce_kernel<double>, dim3((NC + 15) / 16), dim3(1024), 0, st, sums_c, cb, base, n, NC, mse_w);
        mse = mse_w;
    } else if (rows > 0) {
        // few elements: split the candidates, at least 16 for a workgroup (the lane sums that end each candidate weigh more
        // than its eight elements otherwise), towards four workgroups per compute unit
        int shares = 1024 / rows;
        if (shares > (NC + 15) / 16) shares = (NC + 15) / 16;
        if (shares < 1) shares = 1;
        hipLaunchKernelGGL(search_direct_kernel, dim3(rows, shares), dim3(256), 0, st, x, n, maxparts, nparts, a, partial);
        const size_t used = up256((size_t)rows * NC * 4);
        if (rows > 48 && partial_bytes >= used + up256((size_t)NC * 8)) {   // more rows than one workgroup adds in the time of a launch
            double* mse_w = reinterpret_cast<double*>(reinterpret_cast<uint8_t*>(partial) + used);
            hipLaunchKernelGGL(search_reduce_kernel<float>, dim3((NC + 15) / 16), dim3(1024), 0, st, partial, rows, nullptr, n, NC, mse_w);
            mse = mse_w;
        }
    }
    hipLaunchKernelGGL(search_select_kernel, dim3(1), dim3(1024), 0, st, mse, partial, rows, n, maxparts, nparts, a, mse_out, result);
    return hipGetLastError() == hipSuccess ? FPQ_OK : FPQ_ERR_LAUNCH;
}

}  // namespace fpq
