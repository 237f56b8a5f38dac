// Host-side declarations shared by the libfpq translation units: buffer geometry, the packed
// weight header, and the kernel launchers that api.hip calls after validating arguments.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <atomic>
#include <type_traits>

#include "../../include/fpq.h"

namespace fpq {

struct QParams;
struct ScaleSrc;

// Channels of a channels-last code buffer: C rounded up to a whole 16-byte chunk.
static inline int64_t padded_channels(int64_t C) { return (C + 15) / 16 * 16; }

// A kernel that uses more than 64 KB of dynamic LDS must be told so once per device; `done` is the launcher's
// bit mask of the devices that have been (one static per kernel instantiation; setting it twice is harmless).
static inline bool allow_dynamic_lds(const void* kernel, int bytes, std::atomic<uint64_t>& done)
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return false;
    const uint64_t bit = dev < 64 ? (uint64_t)1 << dev : 0;
    if (bit && (done.load(std::memory_order_relaxed) & bit)) return true;
    if (hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes) != hipSuccess) return false;
    done.fetch_or(bit, std::memory_order_relaxed);
    return true;
}

// Length of a packed weight row: taps * Cp rounded up to the 128-code K step of the kernels.
static inline int64_t padded_k(int64_t Cin, int64_t taps) { return (taps * padded_channels(Cin) + 127) / 128 * 128; }

// Blocks of the first absmax pass (each folds >= 4096 elements; at most kAbsmaxParts partials).
constexpr int kAbsmaxParts = 1024;
static inline int absmax_parts(size_t n)
{
    size_t g = (n + 4095) / 4096;
    return (int)(g > kAbsmaxParts ? kAbsmaxParts : g);
}

// Header in front of the packed rows.  The rows start kPackedRowsOffset bytes into the buffer so that, for a
// 256-byte aligned buffer, every 128-byte K chunk of a row is one whole cache line (a chunk that straddles two
// lines halves the rate of the LDS loads).
struct PackedHeader {
    uint32_t magic;      // 'FPQW'
    uint32_t layout;     // 1
    int32_t ebits, mbits, bias;
    float maxval;
    int64_t N, Cin;
    int32_t kh, kw;
    int32_t Cp, Kpad;
    uint32_t reserved[2];
};
static_assert(sizeof(PackedHeader) == 64, "header is 64 bytes");
constexpr size_t kPackedRowsOffset = 256;
constexpr uint32_t kPackedMagic = 0x57515046u;

// How an operand's codes reach the matrix unit.
enum OperandKind : int {
    OPK_FP8 = 0,      // (4, 3, b): hardware E4M3 bit pattern, value * 2^(7 - b)
    OPK_BF8 = 1,      // (5, 2, b): hardware E5M2 bit pattern, value * 2^(15 - b)
    OPK_FP4 = 2,      // (2, 1, b): hardware E2M1 bit pattern, value * 2^(1 - b), two codes per byte
    OPK_GENERIC8 = 3, // any other format, one code per byte, decoded arithmetically
    OPK_GENERIC4 = 4, // any other format of <= 4 bits, two codes per byte, decoded arithmetically
    OPK_HALF8 = 5,    // a format with e <= 4, one code per byte, moved into the bits of a half: value * 2^(b - 15)
    OPK_HALF4 = 6     // the same with two codes per byte
};

// Division of 0 <= n < 2^31 by a positive d, for kernels: n / d = mulhi(2 n, mul) >> shift with shift = ceil(log2 d) and
// mul = ceil(2^(31 + shift) / d) < 2^32.  (n mul / 2^(31 + shift) exceeds n / d by n e / (d 2^(31 + shift)) with e < d <= 2^shift: by less
// than 1 / d.)
struct Divisor {
    uint32_t mul, shift;
};
static inline Divisor divisor(int64_t d)
{
    const uint32_t s = d > 1 ? 64u - (uint32_t)__builtin_clzll((uint64_t)d - 1) : 0u;
    return Divisor{(uint32_t)((((uint64_t)1 << (31 + s)) + (uint64_t)d - 1) / (uint64_t)d), s};
}

struct GemmArgs {
    const uint8_t* x;       // activation codes, channels-last [B, H, W, Cp] (linear: [M, K])
    const uint8_t* wrows;   // packed weight rows (after the header)
    const float* sw;        // [N]
    const float* bias;      // [N] or null
    const float* sx_dev;    // device scale or null
    float sx;               // host scale (used when sx_dev is null)
    float alpha;            // power of two that maps hardware-decoded values to format values
    float* y;
    int M, N;               // GEMM sizes (M = B * Ho * Wo)
    int Kpad;               // packed row length in codes
    int Kreal;              // taps * Cp: codes of x that exist
    int B, H, W, Cp;        // activation geometry (linear: B = M, H = W = 1)
    int Ho, Wo;
    int kh, kw, stride, pad;
    int conv_out;           // 1: y is NCHW [B, N, Ho, Wo]; 0: y is [M, N]
    int xkind, wkind;       // OperandKind
    int xe, xm, xb;         // activation format (for the generic decode)
    int we, wm, wb;         // weight format
    int acc_mode;
    uint32_t x_bytes;       // size of the activation code buffer (bound of the buffer loads)
    uint32_t w_bytes;       // size of the packed weight rows
    float* partial;         // split-K: splits x [M*N] partial results (null: no split)
    int splits;             // number of K slices (>= 1)
    int tile;               // GemmTile chosen by plan_gemm
    int accumulate;         // 1: add the result to y instead of storing it
    // Output as codes for the next quantized layer (not null): the fp32 result is quantized with Eq. (6)-(9)
    // (format below, per-tensor scale sy / sy_dev) and written one code per byte, row-major [M, ldq]
    // (a convolution's rows are its output pixels, i.e. channels-last); y is not written.
    uint8_t* yq;
    int ldq;                // codes per row: N rounded up to 16; columns N .. ldq - 1 receive code 0
    int ym, yb, yem;        // output format: mantissa bits, bias, e + m
    float yc;               // its max value
    int ykind;              // 1 / 2: the format is the hardware's E4M3 / E5M2 (conversion instruction); 0: any other
    float sy;               // host scale (used when sy_dev is null)
    const float* sy_dev;
    int act;                // 0, FPQ_ACT_SILU or FPQ_ACT_GEGLU: applied to the fp32 result before it is quantized
};
// (36 bytes more, for what follows, cost every sliced layer 0.2 us of 27 to 31, and its making 0.05 us of a call)
static_assert(sizeof(GemmArgs) <= 240, "the argument of every layer kernel");
// What the kernels with K over the wavefronts want besides in a convolution of at most 31 taps: worked out at their launch, so that no
// other layer pays for it.
struct ConvArgs : GemmArgs {
    Divisor by_hw, by_wo, by_cp, by_kw;   // Ho Wo, Wo, Cp, kw
    uint32_t tap_rows;      // bit r kw for every kernel row r
};
static inline ConvArgs conv_args(const GemmArgs& a)
{
    ConvArgs c{};
    static_cast<GemmArgs&>(c) = a;
    c.by_hw = divisor((int64_t)a.Ho * a.Wo);
    c.by_wo = divisor(a.Wo);
    c.by_cp = divisor(a.Cp);
    c.by_kw = divisor(a.kw);
    for (int r = 0; r < a.kh; ++r) c.tap_rows |= 1u << (r * a.kw);
    return c;
}
template <bool CONV>
static inline auto wave_args(const GemmArgs& a)
{
    if constexpr (CONV)
        return conv_args(a);
    else
        return a;
}
template <bool CONV>
using WaveArgs = std::conditional_t<CONV, ConvArgs, GemmArgs>;

// Grouped linear layers (fpq_gemm_grouped): up to kGroupMax independent problems per launch, each launch taking the
// problems' pointers and sizes as a kernel argument (no copy to the device, so the call can be captured into a graph).
constexpr int kGroupMax = 32;
constexpr int kGroupAbsmaxParts = 32;   // partial maxima per problem in the dynamic-scale form
struct GroupedProblem {
    const float* x32;       // fp32 activations [M, K] (dynamic-scale form) or null
    const uint8_t* xcodes;  // activation codes [M, K]: the caller's, or where the grouped quantizer writes them
    const uint8_t* wrows;   // packed weight rows (after the header)
    const float* sw;        // [N]
    const float* bias;      // [N] or null
    const float* sx_dev;    // device scale of the codes; dynamic-scale form: where [scale, absmax] are published
    float* y;               // [M, N]
    float* partials;        // dynamic-scale form: kGroupAbsmaxParts partial maxima
    int M, N, K, Kpad;      // K = codes per row of x (a multiple of 16), Kpad = packed row length in codes
    uint32_t w_bytes;       // size of the packed weight rows
};
struct GroupedArgs {
    GroupedProblem p[kGroupMax];
    int count;
    uint32_t over_waves;    // bit i: problem i has its K split over the wavefronts (launch_gemm_grouped)
    GemmArgs common;        // formats, operand kinds, alpha, accumulate mode; the per-problem fields are filled in the kernel
};
static_assert(sizeof(GroupedArgs) <= 4096, "kernel arguments are limited to 4 KB");

// Kernel family / tile for a problem, and how many K slices share an output tile.
enum GemmTile : int {
    TILE_GENERIC = 0,    // register-staged 128x128 / 64x64 kernels: any shape, any operand kinds
    TILE_256x160_S3 = 1, // LDS-DMA kernel, three stages: deep K
    TILE_128x160_S2 = 2, // LDS-DMA kernel, two stages, two workgroups per compute unit
    TILE_128x64 = 3,     // the same pipeline on smaller tiles, two workgroups per compute unit
    TILE_128x128 = 4,
    TILE_WAVE_K4 = 5,    // 64 x 64 tiles, K split over the wavefronts (gemm_wk_kernel.h): four stages, one workgroup per compute unit
    TILE_WAVE_K2 = 6,    // two stages, two workgroups
    TILE_WAVE_128x80 = 7, // K split over the wavefronts, blocks of 16 x 16, one workgroup per compute unit (gemm_wk16_kernel.h)
    TILE_WAVE_64x80 = 8
};
struct GemmPlan {
    int tile;
    int splits;
};

// Which tile, from sweeps of tile x slices over the U-Net's layers and 60 shapes of other widths.
//
// Widths that are multiples of 160 (every U-Net width, a multiple of 320, is): deep K with enough 256-row tiles to fill the
// compute units takes the 256 x 160 tile with three stages (one workgroup per compute unit), everything else the 128 x 160 tile
// with two stages, of which two workgroups fit on a compute unit.  When the tile grid alone would leave compute units idle and K
// is deep, K is cut into slices (each split costs a reduction launch and a round trip of the partial sums, which only a deep K
// pays back): 2 to 4 slices of the 256-row tile when that gives about one work item per compute unit with at least 32 K steps
// each, otherwise one work item per compute unit of the 128-row tile (two when each keeps 20 K steps), with at least 8 K steps
// each.  At most 256 MB of partial sums.  Exceptions:
//   - small outputs with a short K (M N <= 2 Mi, at most 20 steps of 128 codes), at most three columns of 160-wide tiles with a
//     grid of at most 512 64 x 64 tiles, and grids of less than 32 tiles of 128 x 160: plan_small (4096 x 2880 -> 320: 27 us
//     sliced, 19 us with K over the wavefronts; 40 x 5120 -> 1280: 18.9 and 9.8 us; 256 x 11520 -> 1280: 24.4 and 18.8 us);
//   - a grid of less than 192 tiles of 128 x 160 that is not sliced, K of at least 8 steps: 128 x 64 tiles
//     (2048 x 1280 -> 1280: 18.3 -> 13.7 us).
//
// Small problems and other widths, with K of at least 8 steps of 128 codes: grids of at most 256 tiles of 64 x 64 split K over the
// wavefronts of a workgroup with four stages, and K over workgroups too as far as that leaves every compute unit at most one and
// every slice 8 steps (slices need more than 20 steps to pay for their launch: 512 x 1280 -> 320 7.2 us whole, 8.6 us in two);
// grids of at most 512 do so with two stages while K has at most 40 steps (beyond that 128 x 64 tiles in slices are faster:
// 1024 x 9216 -> 1100 37.7 and 32.3 us).  A shorter K takes the register-staged kernel, which starts faster (616 x 768 -> 320:
// 6.1 us against 6.3 us).  Larger grids: plan_unsliced with a K of less than 32 steps, plan_tiled beyond.
enum PlanForm : int {
    PLAN_LINEAR = 0,        // hardware encodings, fp32 results
    PLAN_CONV = 1,
    PLAN_LINEAR_CODES = 2,  // results that leave as codes
    PLAN_CONV_CODES = 3,
    PLAN_HALF = 4           // operands moved into halves, fp32 results
};
// The register-staged 64 x 64 tile or one of the three larger tiles of the load-to-LDS pipeline, as a model of the time prefers:
// t[0] + w (t[1] + t[2] nk) us for launch, epilogue and steps of 128 codes, with w = tiles per compute unit (of the large tiles, of
// which few fit at once, half way between that and the next whole number, and 1.1 for at most one each).  The constants were fitted to
// 1060 shapes of random sizes x tiles; the tiles that the model chooses take 1.02 to 1.05 times the time of the best one in the geometric
// mean.  A choice by K steps times columns among the large tiles alone took 1.17 to 1.31 times, the register-staged kernel with
// 128 x 128 tiles from 512 of them on 1.14 to 1.27 times: its epilogue, an activation ahead of codes above all, runs on one or two
// workgroups per compute unit (1477 x 384 -> 3072, gated GELU, codes out: 14 us in 64 x 64 tiles, 30 us in 128 x 160).  A large tile has
// to be 5 % faster by the model: where the two are close, it errs for either.
static inline GemmPlan plan_unsliced(int64_t M, int64_t N, int64_t nk, PlanForm form)
{
    static const float us_of[5][4][3] = {
        {{3.72f, 0.37f, 0.34f}, {4.47f, 1.04f, 0.53f}, {4.06f, 2.10f, 0.87f}, {3.69f, 2.71f, 1.05f}},
        {{5.87f, 0.68f, 0.38f}, {5.17f, 2.24f, 0.58f}, {4.54f, 3.64f, 0.92f}, {3.82f, 4.32f, 1.14f}},
        {{4.37f, 0.79f, 0.36f}, {8.13f, 1.32f, 0.51f}, {9.92f, 2.34f, 0.86f}, {10.0f, 3.70f, 1.08f}},
        {{7.76f, 1.23f, 0.39f}, {8.20f, 2.10f, 0.58f}, {9.89f, 4.05f, 0.81f}, {10.0f, 5.07f, 1.08f}},
        {{4.98f, 0.19f, 0.68f}, {6.66f, 0.77f, 0.99f}, {6.72f, 1.61f, 1.33f}, {6.18f, 2.09f, 1.77f}},
    };
    const int bx[4] = {64, 128, 128, 128}, bw[4] = {64, 64, 128, 160};
    const int tile[4] = {TILE_GENERIC, TILE_128x64, TILE_128x128, TILE_128x160_S2};
    int best = 0;
    double least = 1e30;
    for (int i = 0; i < 4; ++i) {
        const int64_t tiles = ((M + bx[i] - 1) / bx[i]) * ((N + bw[i] - 1) / bw[i]);
        const double per = (double)tiles / 256.0;
        const double w = i == 0 ? (per > 1.0 ? per : 1.0) : tiles <= 256 ? 1.1 : 0.5 * ((double)((tiles + 255) / 256) + per);
        const float* t = us_of[form][i];
        const double us = (t[0] + w * (t[1] + t[2] * (double)nk)) * (i == 0 ? 0.95 : 1.0);
        if (us < least) { least = us; best = i; }
    }
    return GemmPlan{tile[best], 1};
}
// A deep K: the 128 x 64, 128 x 128 or 128 x 160 tile and the slices that a model of the time prefers: a step of 128 codes over 128 rows
// costs 6 ns per column of the tile (times 1.15 / 1 / 0.97 for the three) and per work item on the busiest compute unit, 1.4 times that
// where a compute unit has one work item only; slices cost 3 us and their partial sums at 5 TB/s (2048 x 11520 -> 1100: 79 us whole, 61 us
// in three).
static inline GemmPlan plan_tiled(int64_t M, int64_t N, int64_t nk)
{
    const int bw[3] = {64, 128, 160};
    const double per[3] = {1.15, 1.0, 0.97};
    const int tile[3] = {TILE_128x64, TILE_128x128, TILE_128x160_S2};
    GemmPlan best{TILE_128x64, 1};
    double least = 1e30;
    for (int i = 0; i < 3; ++i)
        for (int s = 1; s == 1 || (s <= 4 && nk >= 16 * s); ++s) {
            const int64_t items = ((M + 127) / 128) * ((N + bw[i] - 1) / bw[i]) * s;
            const double busiest = items <= 256 ? 1.4 : (double)((items + 255) / 256);
            double us = busiest * bw[i] * per[i] * 0.006 * (double)((nk + s - 1) / s);
            if (s > 1) us += 3.0 + (double)s * (double)M * (double)N * 8.0 / 5e6;
            if (us < least) { least = us; best = GemmPlan{tile[i], s}; }
        }
    return best;
}
static inline GemmPlan plan_small(int64_t M, int64_t N, int64_t nk, PlanForm form)
{
    const int64_t t64 = ((M + 63) / 64) * ((N + 63) / 64);
    if (t64 > 512 && nk < 32) return plan_unsliced(M, N, nk, form);
    if (t64 > 512 || (t64 > 256 && nk > 40)) return plan_tiled(M, N, nk);
    if (nk < 8) return GemmPlan{TILE_GENERIC, 1};
    if (t64 > 256) return GemmPlan{TILE_WAVE_K2, 1};
    int64_t s = 256 / t64;
    if (s > nk / 8) s = nk / 8;
    if (s > 32) s = 32;
    if (nk <= 20) s = 1;
    return GemmPlan{TILE_WAVE_K4, (int)s};
}
static inline bool takes_plan_small(int64_t M, int64_t N, int64_t nk)
{
    const int64_t t64 = ((M + 63) / 64) * ((N + 63) / 64), tiles = ((M + 127) / 128) * ((N + 159) / 160);
    return M <= 16 || N % 160 != 0 || (M * N <= ((int64_t)2 << 20) && nk <= 20) || (N <= 480 && t64 <= 512 && nk >= 8) ||
           (tiles < 32 && nk <= 128);
}
// Widths that are multiples of 160: the 256 x 160 and 128 x 160 tiles and their slices.
static inline GemmPlan plan_wide(int64_t M, int64_t N, int64_t nk)
{
    GemmPlan p{TILE_128x160_S2, 1};
    const int64_t tiles256 = ((M + 255) / 256) * (N / 160), tiles = ((M + 127) / 128) * (N / 160);
    int64_t s = 1;
    if (nk >= 16 && tiles256 >= 192) {
        p.tile = TILE_256x160_S3;
        return p;
    }
    if (tiles256 < 192 && tiles256 >= 48 && nk >= 32 * ((256 + tiles256 / 2) / tiles256)) {
        p.tile = TILE_256x160_S3;
        s = (256 + tiles256 / 2) / tiles256;
    } else if (tiles < 192 && nk >= 16) {
        s = (256 + tiles - 1) / tiles;              // one work item per compute unit ...
        if (nk / (2 * s) >= 20) s *= 2;             // ... two when each still has 20 K steps
        if (s > nk / 8) s = nk / 8;
        if (s > 32) s = 32;
    } else if (tiles <= 16 && nk >= 4) {
        s = nk / 2 < 8 ? nk / 2 : 8;                // a few tiles and a short K: bound by the length of the serial K loop
    }
    while (s > 1 && s * M * N * 4 > ((int64_t)256 << 20)) --s;
    p.splits = s < 1 ? 1 : (int)s;
    return p;
}
// A plan of plan_wide that leaves compute units idle and is not sliced.
static inline bool unsliced_part_grid(const GemmPlan& p, int64_t M, int64_t N, int64_t nk)
{
    return p.splits == 1 && p.tile == TILE_128x160_S2 && ((M + 127) / 128) * (N / 160) < 192 && nk >= 8;
}
// Operands with a hardware conversion or moved into halves.
static inline GemmPlan plan_gemm(int64_t M, int64_t N, int64_t Kpad, PlanForm form)
{
    GemmPlan p{TILE_GENERIC, 1};
    if (M < 1) return p;
    const int64_t nk = Kpad / 128;
    if (M <= 16) {           // (linear layers of at most 16 rows have a kernel of their own)
        p = plan_small(M, N, nk, form);
        p.splits = 1;
        return p;
    }
    if (takes_plan_small(M, N, nk)) {
        p = plan_small(M, N, nk, form);
        while (p.splits > 1 && p.splits * M * N * 4 > ((int64_t)256 << 20)) --p.splits;
        return p;
    }
    p = plan_wide(M, N, nk);
    if (unsliced_part_grid(p, M, N, nk)) p.tile = TILE_128x64;
    return p;
}
// The tiles of gemm_wk16_kernel.h (128 x 80 or 64 x 80, K split over the wavefronts, one workgroup per compute unit, one K slice)
// in the place of a plan of plan_gemm, where a model of the time finds the better of them at least 10 % faster: fp32 results in the
// exact mode, operands with a hardware conversion or moved into halves, kernels of at most 31 taps.  us = t[0] + rounds (t[1] + t[2]
// steps): rounds of 256 tiles, each with its start and its end (nothing overlaps them) and steps of 4 x 64 codes.  The other kernels as
// in plan_unsliced, sliced ones t[0] + w t[1] steps of 128 codes per slice + t[2] us per million partial sums, with w from their work
// items as there from the tiles.  In linear layers of the hardware's encodings the time here grows by up to a quarter as the codes outgrow the
// level-2 caches, 8 to 24 MB (measured over modelled 1.06 below 5 MB, 1.14 to 15, 1.19 to 40, 1.23 beyond; the other kernels 0.98 to 1.05).
// Constants fitted to 8960 layers of random sizes, that growth and the margins for several rounds to 371 linear ones.  1193 others that take
// these tiles need 0.76 of the other plans' time in the geometric mean; 23 of them are slower by more than 3 %, at most by 18 % (9 x 35 x 35 x 21 -> 26,
// 3 x 3, E2M1 weights: 7.2 -> 8.5 us; 1108 x 6928 -> 452 18.1 -> 20.9).  Of the U-Net's layers at batch 1 to 16, 660 by sizes and operands, 315 take these tiles, in 0.73 of the time,
// none of them slower by more than 3 %.
//   - 256-row tiles of images that are no multiple of four pixels, whose stores are single elements, lose throughout (102 layers: 0.41
//     to 0.85 of their time here).
//   - Few tiles with a deep K stay in slices: this kernel has 8 to 64 workgroups there, each with all of K (1 x 2560 x 8 x 8 -> 1280, 3 x 3:
//     31.8 us in 22 slices, 45.9 here; moved into halves 36 and 73).  Half a round and more leave them (8 x 1280 x 16 x 16 -> 1280, 3 x 3: 57 + 10 us
//     in four slices, 46 us here).
//   - Convolutions with K of at most 128, one or two steps of the others, keep their tiles (50 layers of 5 to 6 us: 0.95 to 1.12 times their time here,
//     1.03 in the mean; K of 129 to 256 0.89).
//   - Halves with K of at most 2560 keep their tiles where this kernel goes more than eight rounds (51 layers of 128 x 160 tiles: 0.88 to 1.3
//     times their time here; 49284 x 1504 -> 1280 294 and 373 us; 11080 x 2384 -> 9493 650 and 700), 128 x 160 tiles with K of at most 1280 from the second round on (218 layers,
//     0.77 to 1.9; 1024 x 1280 -> 3840 23.1 and 25.1 us): the rounds of the others overlap.
//   - Whole rounds of 256-row tiles have to be beaten by 20 %: several rounds in a row run here at the clock that the matrix unit's power
//     leaves (8 x 960 x 64 x 64 -> 320, 3 x 3: 145 and 155 us, where the model has 143 and 121; 8 x 1280 x 32 x 32 -> 1280 176 and 180).
//     Linear layers of more than one round and convolutions of more than two have to beat narrower tiles than 160 columns (convolutions: 128 x 160 too)
//     by 15 %: 2230 x 4208 -> 1651 40.5 and 44.6 us, 15 x 1198 x 38 x 16 -> 814, 3 x 3, 139 and 157.
//   - Linear layers with K of at most 1024, or with at most twelve 64 x 64 tiles, keep their kernels: their sums are those of the
//     grouped call, bit for bit.  What K4 cuts into slices keeps them: few tiles.
static inline GemmPlan plan_over_waves(const GemmPlan& p, int64_t M, int64_t N, int64_t Kreal, PlanForm form, bool ragged_images)
{
    static const float us_here[3][2][3] = {
        {{-0.4f, 6.3f, 0.777f}, {0.7f, 4.3f, 0.458f}}, {{0.8f, 6.2f, 0.704f}, {1.6f, 4.1f, 0.43f}}, {{0.85f, 6.3f, 1.18f}, {1.75f, 4.2f, 0.778f}}};
    static const float us_whole[3][7][3] = {
        {{4.2f, -0.03f, 0.413f}, {3.9f, 6.3f, 1.84f}, {2.0f, 3.0f, 1.09f}, {8.9f, -2.6f, 0.602f}, {4.0f, 2.2f, 0.924f}, {4.1f, 0.0f, 0.316f},
         {8.75f, -2.4f, 0.381f}},
        {{6.3f, 0.26f, 0.466f}, {3.0f, 7.0f, 1.95f}, {1.0f, 7.4f, 1.07f}, {6.0f, 0.84f, 0.64f}, {2.8f, 5.7f, 0.91f}, {4.9f, 0.0f, 0.295f},
         {9.4f, -2.3f, 0.339f}},
        {{5.1f, 0.68f, 0.864f}, {3.0f, 9.0f, 2.6f}, {-2.0f, 9.6f, 1.78f}, {21.0f, -6.5f, 0.985f}, {1.4f, 6.6f, 1.35f}, {5.0f, 0.0f, 0.417f},
         {13.2f, -5.0f, 0.493f}}};
    static const float us_sliced[3][4][3] = {{{1.2f, 1.84f, 2.84f}, {9.6f, 1.1f, 0.9f}, {2.5f, 0.57f, 2.54f}, {-1.9f, 1.01f, 1.79f}},
                                             {{27.0f, 1.88f, 0.58f}, {16.3f, 1.085f, 0.65f}, {6.7f, 0.57f, 2.47f}, {2.4f, 0.84f, 2.6f}},
                                             {{31.8f, 2.65f, 0.0f}, {12.8f, 1.88f, 1.29f}, {10.7f, 0.92f, 1.6f}, {-2.2f, 1.43f, 2.6f}}};
    static const int bx[7] = {64, 256, 128, 128, 128, 64, 64}, bw[7] = {64, 160, 160, 64, 128, 64, 64};
    const int f = form == PLAN_LINEAR ? 0 : form == PLAN_CONV ? 1 : form == PLAN_HALF ? 2 : -1;
    if (f < 0 || (f == 1 && Kreal <= 128) || p.tile > TILE_WAVE_K2 || (p.tile == TILE_WAVE_K4 && p.splits > 1)) return p;
    auto tiles = [&](int64_t x, int64_t w) { return ((M + x - 1) / x) * ((N + w - 1) / w); };
    const double steps = (double)((Kreal + 255) / 256), nk = (double)((Kreal + 127) / 128);
    const double mb = (double)M * (double)Kreal * 1e-6;
    const double far = f != 0 || mb < 8.0 ? 1.0 : mb < 24.0 ? 1.0 + 0.25 / 16.0 * (mb - 8.0) : 1.25;
    double us[2];
    for (int i = 0; i < 2; ++i) {
        const float* t = us_here[f][i];
        us[i] = far * (t[0] + (double)((tiles(i ? 64 : 128, 80) + 255) / 256) * (t[1] + t[2] * steps));
    }
    const GemmPlan here{us[0] < us[1] ? TILE_WAVE_128x80 : TILE_WAVE_64x80, 1};
    if (f == 1 && p.tile == TILE_256x160_S3 && p.splits == 1 && ragged_images) return here;
    if (f == 2 && Kreal <= 2560 && tiles(128, 80) > (Kreal <= 1280 && p.tile == TILE_128x160_S2 ? 256 : 8 * 256)) return p;
    const int64_t items = tiles(bx[p.tile], bw[p.tile]) * p.splits;
    const double per = (double)items / 256.0, up = (double)((items + 255) / 256);
    const double w = p.tile == TILE_GENERIC || p.tile >= TILE_WAVE_K4 ? (per > 1.0 ? per : 1.0)
                     : p.tile == TILE_256x160_S3                     ? up
                                                                     : (items <= 256 ? 1.1 : 0.5 * (up + per));
    const float* t = p.splits > 1 ? us_sliced[f][p.tile - 1] : us_whole[f][p.tile];
    const double other = p.splits > 1 ? t[0] + w * t[1] * nk / p.splits + t[2] * (double)p.splits * (double)M * (double)N * 1e-6
                                      : t[0] + w * (t[1] + t[2] * nk);
    const int64_t grid = tiles(us[0] < us[1] ? 128 : 64, 80);
    double margin = 0.9;
    if (f == 0 && grid > 256 && p.tile != TILE_256x160_S3 && p.tile != TILE_128x160_S2)
        margin = 0.85;
    else if (f == 1 && p.tile == TILE_256x160_S3 && p.splits == 1)
        margin = per >= 0.9 * up ? 0.8 : 0.9;
    else if (f == 1 && grid > 512)
        margin = 0.85;
    return (us[0] < us[1] ? us[0] : us[1]) < margin * other ? here : p;
}
// Operands decoded arithmetically (five exponent bits and more): the small tiles are not built for them, so widths that are
// multiples of 160 keep the 160-wide tiles and their slices (E5M2, 256 x 11520 -> 1280: 70 us, 209 us on the register-staged
// kernel; 40 x 5120 -> 1280: 60 and 92 us; 4096 x 2880 -> 320: 86 and 98 us).  The register-staged kernel serves small outputs with
// a short K, and grids of less than 192 tiles that are not sliced (2048 x 1280 -> 1280: 63 us, 69 us on 128 x 160 tiles).
static inline GemmPlan plan_arithmetic(int64_t M, int64_t N, int64_t Kpad)
{
    const int64_t nk = Kpad / 128;
    if (N % 160 != 0 || M <= 16 || (M * N <= ((int64_t)2 << 20) && nk <= 20)) return GemmPlan{TILE_GENERIC, 1};
    const GemmPlan p = plan_wide(M, N, nk);
    return unsliced_part_grid(p, M, N, nk) ? GemmPlan{TILE_GENERIC, 1} : p;
}

// Tile of the integer layer (igemm.hip): rows x columns, stages of 128 codes.
enum IntTile : int { INT_64x64_S2 = 0, INT_64x64_S3 = 1, INT_64x128 = 2, INT_128x128 = 3 };
// 128 x 128 tiles where they fill the compute units, cover few columns beyond N and have 10 G multiply-adds or more to do: their rate
// is the higher one and their start and last round the longer ones (time of 64 x 64 over theirs, 456 layers of random sizes:
// 0.7 to 0.9 below that, 1.0 there, 1.1 to 1.3 beyond; K of at most 128 0.7 to 0.95 throughout.  2048 x 1280 -> 10240 57 and 41 us,
// 5200 x 528 -> 1024 11.9 and 17.0).  64 x 64 tiles with a third stage where a deep K has to hide its loads with at most two
// workgroups per compute unit (2000 x 5120 -> 640: 45 us, 52 with two stages; 32815 x 2672 -> 28, 513 tiles: 21.5 and 17.8), which
// otherwise costs the room for five of them (30000 x 64 -> 1001: 56 and 47).
// 64 x 128 tiles between the two: more of them run together than of the large ones (three per compute unit, five with 4-bit weights,
// two of the others) and each reads half the weights of two small ones.  8 G multiply-adds and more in 600 to 1500 of them, not
// just over one round of 768 (4-bit weights: 700 to 1024), unless the large tiles make one well filled round: 0.88 of the others'
// time over the 44 layers of random sizes that these ends were found on, 0.89 over 61 others, at most 1.05 (2702 x 1216 -> 4352 27.9 -> 29.3 us; 8192 x 2560 -> 640 28.4 -> 24.8 us, 8192 x 1280 -> 1280 26.5 -> 23.6, 1472 x 1024
// -> 7040 32.5 -> 19.9; elsewhere: 7936 x 1472 -> 832, 868 tiles, 21.9 and 23.8; in a round of 384 to 512 large tiles up to
// 1.2 times their time, beyond 1500 1.0 to 1.3, K below 1000 0.9 to 1.1).
static inline IntTile int_tile(int64_t M, int64_t N, int64_t K, int64_t Kpad, int wbits)
{
    const int64_t tiles128 = ((M + 127) / 128) * ((N + 127) / 128), tiles64 = ((M + 63) / 64) * ((N + 63) / 64);
    const int64_t tiles64x128 = ((M + 63) / 64) * ((N + 127) / 128);
    const bool few_beyond = (N + 127) / 128 * 128 * 10 <= N * 11;
    const bool large = tiles128 >= 320 && few_beyond && K > 128 && M * N * K >= (int64_t)10000000000;
    const bool middle = few_beyond && K >= 1000 && M * N * K >= (int64_t)8000000000 && !(large && tiles128 >= 384 && tiles128 <= 512) &&
                        (wbits == 4 ? tiles64x128 >= 700 && tiles64x128 <= 1024
                                    : tiles64x128 >= 600 && tiles64x128 <= 1500 && (tiles64x128 <= 768 || tiles64x128 >= 900));
    const bool third = Kpad >= 2048 && tiles64 <= 512;
    return middle ? INT_64x128 : large ? INT_128x128 : third ? INT_64x64_S3 : INT_64x64_S2;
}

static inline size_t split_workspace_bytes(const GemmPlan& p, int64_t M, int64_t N)
{
    return p.splits > 1 ? (size_t)p.splits * (size_t)M * (size_t)N * sizeof(float) : 0;
}
// Partial sums that a layer of any operand kinds may want (slices do not depend on the form).
static inline size_t most_split_workspace_bytes(int64_t M, int64_t N, int64_t Kpad)
{
    const size_t a = split_workspace_bytes(plan_gemm(M, N, Kpad, PLAN_LINEAR), M, N);
    const size_t b = split_workspace_bytes(plan_arithmetic(M, N, Kpad), M, N);
    return a > b ? a : b;
}

// Encoding / bias search (Section V-A): at most 8 encodings x 128 bias candidates.
constexpr int kSearchMaxEncodings = 8;
constexpr int kSearchMaxCandidates = 1024;
struct SearchEnc {
    int32_t e, m, b0;   // b0 = 2^(e-1)
    float c0;           // Eq. (7) at b0
};
struct SearchArgs {
    int32_t n_enc, J;
    SearchEnc enc[kSearchMaxEncodings];
};
// Blocks of the search pass: 2048 elements per block and round, at most 1024 blocks.
static inline int search_blocks(size_t n)
{
    size_t g = (n + 2047) / 2048;
    return (int)(g > 1024 ? 1024 : g);
}
// maxparts: what launch_absmax_partials left; partial: workspace of partial_bytes (the binned form of large tensors wants
// search_binned_bytes plus one double per candidate; with less the direct form runs).
size_t search_binned_bytes(size_t n, int nc);
int launch_search(const float* x, size_t n, const SearchArgs& a, const float* maxparts, float* partial, size_t partial_bytes,
                  float* mse_out, fpq_search_result* result, hipStream_t st);

// Rounding learning (Section V-B): launchers of rounding.hip.
size_t rl_workspace_bytes(int64_t M, int64_t N, int64_t K);
int launch_rl_init(const float* w, const float* sw, int64_t N, int64_t K, const QParams& q, float* alpha, hipStream_t st);
int launch_rl_mask(const float* alpha, size_t n, uint8_t* mask, hipStream_t st);
int launch_rl_im2col(const float* x, int64_t B, int64_t C, int64_t H, int64_t W, int kh, int kw, int stride, int pad,
                     float* a, hipStream_t st);
int launch_rl_step(const float* w, const float* sw, int64_t N, int64_t K, const QParams& q, float* alpha, const float* a,
                   int64_t M, float lr, float reg_weight, float* loss_out, float* grad_out, void* workspace, hipStream_t st);

// Zero count (Section VI, "Sparsity"): blocks of the counting pass, each with a contiguous share of the bytes.
static inline int count_zeros_parts(size_t nbytes)
{
    const size_t p = (nbytes + 16383) / 16384;
    return p < 1 ? 1 : (p > 1024 ? 1024 : (int)p);
}
int launch_count_zeros(const void* x, int is_fp32, size_t n, int em, bool four_bit, unsigned long long* out,
                       unsigned long long* partial, hipStream_t st);
int launch_absmax(const float* x, size_t n, float maxval, float* absmax_out, float* scale_out, float* partial,
                  hipStream_t st);
int launch_absmax_partials(const float* x, size_t n, float* partial, hipStream_t st);
int launch_quantize_dynamic_small(const float* x, size_t n, const QParams& q, float maxval, float* publish, uint8_t* codes,
                                  hipStream_t st);
int launch_quantize(const float* x, size_t n, const QParams& q, bool four_bit, const ScaleSrc& ss, uint8_t* codes,
                    hipStream_t st);
int launch_quantize_nhwc(const float* x, int64_t B, int64_t C, int64_t H, int64_t W, const QParams& q,
                         const ScaleSrc& ss, uint8_t* codes, hipStream_t st);
int launch_dequantize(const uint8_t* codes, size_t n, int e, int m, int b, float scale, float* out, hipStream_t st);
int launch_pack_weights(const float* w, int64_t N, int64_t Cin, int taps, const QParams& q, bool four_bit,
                        const float* scale_in, const uint8_t* mask, uint8_t* packed_rows, float* scale_out,
                        uint8_t* codes_out, hipStream_t st);
int launch_gemm(const GemmArgs& a, hipStream_t st);
bool gemm_rows16_applicable(const GemmArgs& a);             // linear layers with at most 16 rows
// One launch for a dynamically scaled linear layer with at most 16 rows (x: the fp32 activations; a.x is not used;
// codes [M, K] and publish [scale, absmax] receive what the two-launch form leaves in the workspace).
int launch_gemm_skinny_dynamic(const GemmArgs& a, const float* x, const QParams& qx, float maxval, uint8_t* codes,
                               float* publish, hipStream_t st);
// Grouped forms (gemm.hip, quant.hip): one launch each over all problems of g.
int launch_gemm_grouped(const GroupedArgs& g, hipStream_t st);                 // small tiles, any shape
static inline bool grouped_wk_applicable(const GemmArgs& a)                    // operand kinds of that one
{
    if (a.acc_mode == FPQ_ACC_FP8_MFMA) return a.xkind == OPK_FP8 && (a.wkind == OPK_FP8 || a.wkind == OPK_FP4);
    return (a.xkind == OPK_FP8 && (a.wkind == OPK_FP8 || a.wkind == OPK_FP4)) || a.xkind == OPK_HALF8;
}
bool skinny_grouped_applicable(const GroupedArgs& g);                           // all problems: at most 16 rows, <= 16 Ki activations
int launch_gemm_skinny_dynamic_grouped(const GroupedArgs& g, const QParams& qx, float maxval, hipStream_t st);
int launch_quantize_dynamic_grouped(const GroupedArgs& g, const QParams& qx, float maxval, hipStream_t st);
// Structured-sparse weight operand (gemm_sparse.hip).
int launch_pack_weights_sparse(const float* w, int64_t N, int64_t Cin, int taps, const QParams& q, bool four_bit,
                               const float* scale_in, const uint8_t* mask, uint8_t* code_rows, uint32_t* pos_rows,
                               float* scale_out, uint8_t* codes_out, unsigned long long* altered, hipStream_t st);
int launch_gemm_sparse(const GemmArgs& a, const uint32_t* pos_rows, hipStream_t st);
// Uniform integer baseline of Eq. (4) (igemm.hip).
int launch_int_params(const float* x, size_t n, int bits, fpq_int_params* out, float* partial, hipStream_t st);
int launch_int_quantize(const float* x, size_t n, int bits, float scale, int zp, const fpq_int_params* params_dev, uint8_t* codes,
                        hipStream_t st);
int launch_int_pack_weights(const float* w, int64_t N, int64_t K, int bits, uint8_t* rows, float* scale_out, int32_t* zp_out,
                            int32_t* rowsum_out, uint8_t* codes_out, hipStream_t st);
int launch_int_gemm(const uint8_t* x, float sx, int zx, const fpq_int_params* px_dev, const uint8_t* wrows, const int32_t* wsum,
                    int wbits, const float* sw, const int32_t* zw, const float* bias, float* y, int64_t M, int64_t N, int64_t K,
                    hipStream_t st);
// Machine-ceiling probes (peaks.hip): kind 0 / 1 = register-only bf16 / 8-bit MFMA loop, 2 = device copy,
// 3 / 4 = bf16 MFMA with the conversions of a 64 x 160 / 32 x 160 wave tile, 5 = device fill.
int launch_probe(int kind, int iters, const void* src, void* dst, size_t bytes, int* grid_out, hipStream_t st);
bool gemm_dma_applicable(const GemmArgs& a);
int launch_gemm_dma(const GemmArgs& a, hipStream_t st);
int launch_gemm_dma_q(const GemmArgs& a, hipStream_t st);   // the same with the result as codes (a.yq)
int launch_gemm_dma_s(const GemmArgs& a, hipStream_t st);   // small tiles
int launch_gemm_dma_sq(const GemmArgs& a, hipStream_t st);
int launch_gemm_wk(const GemmArgs& a, hipStream_t st);      // K split over the wavefronts
int launch_gemm_wk_q(const GemmArgs& a, hipStream_t st);
int launch_gemm_wk16(const GemmArgs& a, hipStream_t st);    // the same in blocks of 16 x 16
int launch_gemm_wk16_h(const GemmArgs& a, hipStream_t st);
bool gemm_strip_applicable(const GemmArgs& a);              // weights in registers: a short K (gemm_strip_kernel.h)
int launch_gemm_strip(const GemmArgs& a, hipStream_t st);
int launch_gemm_strip_h(const GemmArgs& a, hipStream_t st);
int launch_gemm_strip_q(const GemmArgs& a, hipStream_t st);

}  // namespace fpq
