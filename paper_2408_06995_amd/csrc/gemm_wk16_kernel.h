// Quantized linear / convolution layer on ExMy codes for gfx950: tiles of 128 x 80 and 64 x 80 with K split over the wavefronts.
//
// A workgroup of four wavefronts owns a tile of 16 MI activation rows and 16 NI weight rows; the wavefronts take the steps of 64
// codes of K in turn, each computes the whole tile over its steps in blocks of 16 x 16 with an LDS ring of its own (no barrier in
// the loop, NST steps deep), and the four partial tiles are added through LDS.  What that buys:
//   - 13 fragments (9 in the small tile) are read and converted for 40 (20) MFMAs, and nothing twice: the 128 x 160 tiles convert 6 for 5
//     MFMAs of twice the size, every weight four times in a workgroup;
//   - a tile over all of K where 160-wide tiles leave compute units idle and have to be cut into K slices: no partial sums in memory
//     (42 MB out and back for 2048 x 11520 -> 1280 in four slices, 10 us), no second launch;
//   - tiles of 80 columns divide every width that is a multiple of 80, and 256 of them one image of 64 x 64 pixels x 320 channels.
// One workgroup fits on a compute unit (up to 160 KB of LDS, 390 registers), so grids of one round of 256 tiles are what it is for.
// Loads run NST steps ahead: with two stages of 64 codes, as in gemm_wk_kernel.h, a step took as long as a load (2000 cycles).  A step of
// the 128 x 80 tile is 1280 cycles of MFMAs, measured 1800 with masked loads: what bounds it is the issue of one wavefront's MFMAs,
// conversions and loads (80, 104 and 13 a step).  Outside the loop: 3000 cycles to the first load's issue and 11000 for sums and stores.
// us before -> here, 3 x 3: 8 x 1280 x 16 x 16 -> 1280, codes in, E4M3 68.8 -> 50.7; E2M1 weights, dynamic scale, 72.9 -> 54.8; E3M4 x E3M0,
// static scale, 96.5 -> 66.3; 8 x 640 x 32 x 32 -> 640, codes in, 67.8 -> 57.0; with a dynamic scale 1 x 320 x 64 x 64 -> 320 23.9 -> 17.2, and
// 3 x 200 x 75 x 53 -> 392, stride 2, 23.5 -> 19.0.  Tried without gain: operands from memory straight into registers (sixteen rows
// of 64 bytes a load are 61 cache accesses, 15 in the order that LDS allows: 79 us for the first of these), eight wavefronts with two
// steps each in flight (the small tile 18.3 us where four take 17.6).
// Error of four partial sums against one or the slices (root mean square of the difference to the sum in 64 bits, over the sum of the
// products' magnitudes, before -> here), 0.67 to 1.01 of it over 21 layers: 8 x 1280 x 16 x 16 -> 1280 1.484e-9 -> 1.476e-9, E2M1 weights 9.7e-10 -> 6.5e-10; 1 x 320 x 64 x 64 -> 320
// 2.05e-9 -> 2.07e-9; 3 x 200 x 75 x 53 -> 392 2.31e-9 -> 2.30e-9; 3000 x 3632 -> 641 2.53e-9 -> 1.92e-9.
#pragma once
#include "gemm_dma_kernel.h"

namespace fpq {

typedef unsigned v4u __attribute__((ext_vector_type(4)));
typedef float v4acc __attribute__((ext_vector_type(4)));

// Two codes of a fragment of eight: pair p of the codes in (lo, hi), in lo alone for 4-bit operands.
template <int KIND>
__device__ __forceinline__ uint32_t decode2(uint32_t lo, uint32_t hi, int p, const GenFmt& f)
{
    const uint32_t w = p < 2 ? lo : hi;
    if constexpr (KIND == OPK_FP8) {
        return p & 1 ? __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w, 1.0f, true))
                     : __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w, 1.0f, false));
    } else if constexpr (KIND == OPK_FP4) {
        return __builtin_bit_cast(uint32_t, p == 0   ? __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(lo, 1.0f, 0)
                                            : p == 1 ? __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(lo, 1.0f, 1)
                                            : p == 2 ? __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(lo, 1.0f, 2)
                                                     : __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(lo, 1.0f, 3));
    } else {
        static_assert(KIND == OPK_HALF8 || KIND == OPK_HALF4, "operand kinds of this kernel");
        union {
            v8bf v;
            uint32_t u[4];
        } o;
        o.v = decode8<KIND>(lo, hi, f);
        return o.u[p];
    }
}

template <int KIND>
__device__ __forceinline__ v4acc mfma16(const uint32_t (&p)[4], const uint32_t (&q)[4], v4acc c)
{
    const v4u pv = {p[0], p[1], p[2], p[3]}, qv = {q[0], q[1], q[2], q[3]};
    if constexpr (KIND == OPK_HALF8 || KIND == OPK_HALF4)
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(v8h, pv), __builtin_bit_cast(v8h, qv), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, pv), __builtin_bit_cast(v8bf, qv), c, 0, 0, 0);
}

// f(integral constant B), ..., f(integral constant E - 1)
template <int B, int E, class F>
__device__ __forceinline__ void static_for(F&& f)
{
    if constexpr (B < E) {
        f(std::integral_constant<int, B>{});
        static_for<B + 1, E>(f);
    }
}

constexpr int wk16_stage(int mi, int ni, bool w4) { return 1024 * (mi + (w4 ? (ni + 1) / 2 : ni)); }
// ring of one wavefront, later its partial tile
constexpr int wk16_wave_lds(int mi, int ni, int nst, bool w4)
{
    return nst * wk16_stage(mi, ni, w4) > mi * ni * 1024 ? nst * wk16_stage(mi, ni, w4) : mi * ni * 1024;
}

template <int MI, int NI, int NST, int XKIND, int WKIND, bool CONV>
__global__ __launch_bounds__(256, 1) void gemm_wk16_kernel(const WaveArgs<CONV> a)
{
    constexpr bool W4 = kind_is_4bit(WKIND);
    constexpr int BX = 16 * MI, BW = 16 * NI, XTILE = MI * 1024, STAGE = wk16_stage(MI, NI, W4), WAVE_LDS = wk16_wave_lds(MI, NI, NST, W4);
    constexpr int XLD = MI, WLD = W4 ? (NI + 1) / 2 : NI, LOADS = XLD + WLD;      // loads of 1 KB per wavefront and stage
    static_assert(MI % 4 == 0, "every wavefront finishes MI / 4 rows of blocks; fragment 0 of a step is in set 0");
    // P = operand along the accumulator registers (four neighbouring rows or pixels per lane), Q = operand along the lanes.  NCHW
    // results want four neighbouring pixels of a channel in a lane, row-major ones four neighbouring columns of a row.
    constexpr bool P_IS_W = !CONV;
    constexpr int WAIT_LDS = 15 | (7 << 4) | (0 << 8) | (3 << 14);                // s_waitcnt lgkmcnt(0) alone
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    const int lane = threadIdx.x & 63, r16 = lane & 15, q = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

    // Ids go round-robin over the 8 XCDs: each takes a contiguous run of bands of four tile rows, rows innermost, so that the workgroups
    // that run together on an XCD share activations as well as weights.
    const int tiles_w = (a.N + BW - 1) / BW, tiles_x = (a.M + BX - 1) / BX;
    int tile = blockIdx.x;
    {
        const int per = gridDim.x >> 3;
        if (tile < (per << 3)) tile = (tile & 7) * per + (tile >> 3);
    }
    const int band = tile / (4 * tiles_w), rows = tiles_x - 4 * band;
    const int at = tile - band * 4 * tiles_w;
    const int tw = rows >= 4 ? at >> 2 : at / rows, tx = 4 * band + at - tw * (rows >= 4 ? 4 : rows);
    const int m0 = tx * BX, n0 = tw * BW;

    // steps of 64 codes, dealt out to the wavefronts in turn: the halves of a 128-byte line are read by neighbours at the same time
    const int nk = ((a.Kreal + 63) / 64 - wave + 3) >> 2;              // not positive: none

    // ---- loads of 16 rows of 64 bytes (4-bit weights: 32 rows of 32 bytes): lane p holds row p / 4, LDS chunk p % 4, i.e. logical
    // chunk (p % 4) ^ swizzle(row)
    const v4i xrsrc = make_rsrc(a.x, a.x_bytes);
    const v4i wrsrc = make_rsrc(a.wrows, a.w_bytes);
    const unsigned lds0 = (unsigned)(size_t)((__attribute__((address_space(3))) void*)smem) + wave * WAVE_LDS;
    constexpr unsigned OOB = 0x80000000u;      // an offset with this bit delivers zeros = code 0
    const int xc = (lane & 3) ^ ((lane >> 4) & 3);
    unsigned xbase[XLD], xout[XLD], wbase[WLD];  // byte offset of a row's tap (0, 0), channel 0; bit t: tap t lies outside
    int x_k = wave * 64 + 16 * xc, x_ci = x_k, x_kh = 0, x_kw = 0, x_tap = 0;
    if constexpr (CONV) {
        // a lane works out one or two rows, and the rows change hands in LDS (in the wavefront's own ring, still empty)
        uint2* table = reinterpret_cast<uint2*>(smem + wave * WAVE_LDS);
#pragma unroll
        for (int r = 0; r < BX; r += 64) {
            const int m = m0 + r + lane;
            unsigned base, taps;
            conv_row(a, m, base, taps);
            table[r + lane] = make_uint2(base, m < a.M ? ~taps : ~0u);   // bit 31: beyond the end of K
        }
        asm volatile("" ::: "memory");
#pragma unroll
        for (int i = 0; i < XLD; ++i) {
            const uint2 v = table[16 * i + (lane >> 2)];
            xbase[i] = v.x;
            xout[i] = v.y;
        }
        __builtin_amdgcn_s_waitcnt(WAIT_LDS);
        asm volatile("" ::: "memory");
        x_tap = divide(x_k, a.by_cp);
        x_ci = x_k - x_tap * a.Cp;
        x_kh = divide(x_tap, a.by_kw);
        x_kw = x_tap - x_kh * a.kw;
    } else {
#pragma unroll
        for (int i = 0; i < XLD; ++i) {
            const int m = m0 + 16 * i + (lane >> 2);
            xbase[i] = (unsigned)m * (unsigned)a.Cp;
            xout[i] = m < a.M ? 0x80000000u : ~0u;
        }
    }
    // scales and biases of the columns that this lane finishes: fetched ahead of the loop, waited for behind it.  P = weights: columns
    // 4 q .. + 3 of every block; else channel r16
    constexpr int NS = P_IS_W ? 4 : 1;
    float sw[NI][NS], bv[NI][NS];
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
        for (int e = 0; e < NS; ++e) {
            const int n = min(n0 + 16 * j + (P_IS_W ? 4 * q + e : r16), a.N - 1);
            sw[j][e] = a.sw[n];
            bv[j][e] = a.bias ? a.bias[n] : 0.0f;
        }
    constexpr unsigned WSTEP = W4 ? 128 : 256;  // bytes of a weight row from a step to this wavefront's next
    {
        const unsigned wrow_bytes = W4 ? (unsigned)a.Kpad / 2 : (unsigned)a.Kpad;
#pragma unroll
        for (int i = 0; i < WLD; ++i) {
            const int row = W4 ? 32 * i + (lane >> 1) : 16 * i + (lane >> 2);
            const int chunk = W4 ? (lane & 1) ^ ((row >> 3) & 1) : xc;
            const int n = n0 + row;
            wbase[i] = row < BW && n < a.N ? (unsigned)n * wrow_bytes + (unsigned)wave * (WSTEP / 4) + 16 * chunk : OOB;
        }
    }
    // position of the step being loaded: offset from xbase, and 31 - the bit of xout that tells whether it exists
    unsigned x_delta = 0, x_shift = 0;
    // (a wavefront's next step is 256 codes on: whole taps and a rest, at most one carry from channels to taps and from columns to rows)
    int step_tap = 0, step_ci = 0, step_kh = 0, step_kw = 0;
    if constexpr (CONV) {
        step_tap = divide(256, a.by_cp);
        step_ci = 256 - step_tap * a.Cp;
        step_kh = divide(step_tap, a.by_kw);
        step_kw = step_tap - step_kh * a.kw;
    }
    auto place = [&]() {
        x_shift = x_k < a.Kreal ? 31u - (unsigned)x_tap : 0u;
        x_delta = CONV ? (unsigned)((x_kh * a.W + x_kw) * a.Cp + x_ci) : (unsigned)x_k;
        x_k += 256;
        if (CONV) {
            x_ci += step_ci;
            const int carry = x_ci >= a.Cp ? 1 : 0;
            x_ci -= carry ? a.Cp : 0;
            x_tap += step_tap + carry;
            x_kw += step_kw + carry;
            const int row = x_kw >= a.kw ? 1 : 0;
            x_kw -= row ? a.kw : 0;
            x_kh += step_kh + row;
        }
    };
    int live = -1;                             // what dma16_live wants
    auto load = [&](int idx, unsigned to, auto all_live) {
        if (idx < WLD) {
            if constexpr (decltype(all_live)::value)
                dma16(wrsrc, wbase[idx], to + XTILE + idx * 1024);
            else
                dma16_live(wrsrc, wbase[idx], to + XTILE + idx * 1024, live);
            wbase[idx] += WSTEP;               // (far from carrying OOB's bit out: a row has less than 2^29 bytes)
        } else {
            const int i = idx - WLD;
            const unsigned off = ((xout[i] << x_shift) & OOB) | (xbase[i] + x_delta);
            if constexpr (decltype(all_live)::value)
                dma16(xrsrc, off, to + i * 1024);
            else
                dma16_live(xrsrc, off, to + i * 1024, live);
        }
    };
    // (steps that do not exist load with one lane: the waits count on NST steps' loads)
#pragma unroll
    for (int s = 0; s < NST; ++s) {
        place();
        live = s < nk ? -1 : 1;
#pragma unroll
        for (int idx = 0; idx < LOADS; ++idx) load(idx, lds0 + s * STAGE, std::false_type{});
    }

    v4acc acc[MI][NI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) acc[i][j] = v4acc{0.0f, 0.0f, 0.0f, 0.0f};

    // ---- K loop.  A step of 64 codes is two MFMA steps of 32 (number ks: codes 8 ks .. + 7 of the 16 of every lane), each MI rows of
    // NI MFMAs; one slot per MFMA.  In a row's slots the fragment of the next row is converted, and, spread over the MFMA step, the weight
    // fragments of the next one.  The second MFMA step opens with the wait for the next step's loads and reads that step from LDS,
    // every block as soon as its registers are free; so a slot of the ring is empty when its step begins, and the first MFMA step
    // issues the loads of the step NST ahead into it.
    const GenFmt wfm{a.we, a.wm, a.wb}, xfm{a.xe, a.xm, a.xb};
    uint4 xr[MI], wr[NI];
    uint32_t xf[2][4], wf[2][NI][4];
    auto read_x = [&](int slot, int i) {
        xr[i] = *reinterpret_cast<const uint4*>(smem + wave * WAVE_LDS + slot * STAGE + lds_off<64>(16 * i + r16, q));
    };
    auto read_w = [&](int slot, int j) {
        const uint8_t* w = smem + wave * WAVE_LDS + slot * STAGE + XTILE;
        const int row = 16 * j + r16;
        if constexpr (W4) {
            const uint2 v = *reinterpret_cast<const uint2*>(w + row * 32 + (((q >> 1) ^ ((row >> 3) & 1)) << 4) + 8 * (q & 1));
            wr[j] = make_uint4(v.x, v.y, 0, 0);
        } else {
            wr[j] = *reinterpret_cast<const uint4*>(w + lds_off<64>(row, q));
        }
    };
    auto x_pair = [&](int ks, int i, int p, int to) {
        xf[to][p] = ks ? decode2<XKIND>(xr[i].z, xr[i].w, p, xfm) : decode2<XKIND>(xr[i].x, xr[i].y, p, xfm);
    };
    auto w_pair = [&](int ks, int j, int p, int to) {
        if constexpr (W4)
            wf[to][j][p] = decode2<WKIND>(ks ? wr[j].y : wr[j].x, 0u, p, wfm);
        else
            wf[to][j][p] = ks ? decode2<WKIND>(wr[j].z, wr[j].w, p, wfm) : decode2<WKIND>(wr[j].x, wr[j].y, p, wfm);
    };
    // the next step's loads have landed when at most those of the NST - 1 steps after it are outstanding
    auto wait_next = [&]() {
        __builtin_amdgcn_s_waitcnt(vmcnt_imm((NST - 1) * LOADS));
        asm volatile("" ::: "memory");
    };
    static_assert((NST - 1) * LOADS <= 63, "the counter's range");
    // L0: slot of the first MFMA step from which loads go out (its LDS reads are rows behind), W0: slot of the second from which weight
    // fragments are converted
    constexpr int SLOTS = MI * NI, WUNITS = 4 * NI, L0 = NI, W0 = 2 * NI;
    // (constants all the way: a slot's share of conversions and loads depends on its number)
    auto step = [&](auto st, auto all_live) __attribute__((always_inline)) {
        constexpr int next = st + 1 == NST ? 0 : st + 1;
        const unsigned to = lds0 + st * STAGE;
        static_for<0, 2 * SLOTS>([&](auto slot_at) {
            constexpr int ks = decltype(slot_at)::value / SLOTS, slot = decltype(slot_at)::value % SLOTS, i = slot / NI, j = slot % NI;
            constexpr int cur = i & 1;
            acc[i][j] = P_IS_W ? mfma16<XKIND>(wf[ks][j], xf[cur], acc[i][j]) : mfma16<XKIND>(xf[cur], wf[ks][j], acc[i][j]);
            if constexpr (ks == 0) {
                if constexpr (slot == 0) place();
                if constexpr (slot == L0) {
                    __builtin_amdgcn_s_waitcnt(WAIT_LDS);
                    asm volatile("" ::: "memory");
                }
                if constexpr (slot >= L0)
                    static_for<(slot - L0) * LOADS / (SLOTS - L0), (slot - L0 + 1) * LOADS / (SLOTS - L0)>(
                        [&](auto idx) { load(idx, to, all_live); });
            } else {
                if constexpr (slot == 0) wait_next();
                if constexpr (slot == 0) static_for<0, NI>([&](auto w) { read_w(next, w); });
                if constexpr (j == 0) read_x(next, i);     // its last codes were converted in the row before
            }
            static_for<(4 * j + NI - 1) / NI, (4 * (j + 1) + NI - 1) / NI>([&](auto p) {              // the next row's fragment
                if constexpr (i + 1 < MI)
                    x_pair(ks, i + 1, p, cur ^ 1);
                else
                    x_pair(ks ^ 1, 0, p, cur ^ 1);
            });
            if constexpr (ks == 0)
                static_for<slot * WUNITS / SLOTS, (slot + 1) * WUNITS / SLOTS>([&](auto u) { w_pair(1, u >> 2, u & 3, 1); });
            else if constexpr (slot >= W0)
                static_for<(slot - W0) * WUNITS / (SLOTS - W0), (slot - W0 + 1) * WUNITS / (SLOTS - W0)>(
                    [&](auto u) { w_pair(0, u >> 2, u & 3, 0); });
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    wait_next();                               // (the first step's)
#pragma unroll
    for (int j = 0; j < NI; ++j) read_w(0, j);
#pragma unroll
    for (int i = 0; i < MI; ++i) read_x(0, i);
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
        for (int p = 0; p < 4; ++p) w_pair(0, j, p, 0);
#pragma unroll
    for (int p = 0; p < 4; ++p) x_pair(0, 0, p, 0);
    // the sums stay in the same accumulation registers through both loops (the compiler would move half of them out and in at every step)
    auto pin = [&]() {
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NI; ++j) asm volatile("" : "+a"(acc[i][j]));
    };
    // whole rounds of the ring whose loads all exist, then the rest (masking lanes off costs three scalar instructions a load)
    int kt = 0;
    pin();
    for (; kt + 2 * NST <= nk; kt += NST)
        static_for<0, NST>([&](auto st) { step(st, std::true_type{}); });
    pin();
    for (; kt < nk; kt += NST)
        static_for<0, NST>([&](auto st) {
            if (kt + st < nk) {
                live = kt + st + NST < nk ? -1 : 1;
                step(st, std::false_type{});
            }
        });
    pin();
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));                      // no load may land in LDS from here on
    asm volatile("" ::: "memory");

    // ---- add the four partial tiles: every wavefront leaves its own in LDS (its own ring: [block][lane], four values each);
    // wavefront w finishes block rows w MI / 4 .. + MI / 4 - 1
    float4* part = reinterpret_cast<float4*>(smem) + lane;
    constexpr int WAVE_F4 = WAVE_LDS / 16;
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j)
            part[wave * WAVE_F4 + (i * NI + j) * 64] = make_float4(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]);
    const float sxa = (a.sx_dev ? a.sx_dev[0] : a.sx) * a.alpha;
    __syncthreads();
    const bool accum = a.accumulate;
    const int hw = a.Ho * a.Wo;
#pragma unroll
    for (int ii = 0; ii < MI / 4; ++ii) {
        const int i = wave * (MI / 4) + ii;
        const int mp = m0 + 16 * i + 4 * q;                        // NCHW: the lane's first pixel
        int bi = 0;
        if constexpr (CONV) bi = divide(mp, a.by_hw);
        const int pix = mp - bi * hw;
#pragma unroll
        for (int j = 0; j < NI; ++j) {
            float4 v[4];
#pragma unroll
            for (int w = 0; w < 4; ++w) v[w] = part[w * WAVE_F4 + (i * NI + j) * 64];
            float o[4] = {((v[0].x + v[1].x) + v[2].x) + v[3].x, ((v[0].y + v[1].y) + v[2].y) + v[3].y,
                          ((v[0].z + v[1].z) + v[2].z) + v[3].z, ((v[0].w + v[1].w) + v[2].w) + v[3].w};
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = o[e] * (sxa * sw[j][P_IS_W ? e : 0]) + bv[j][P_IS_W ? e : 0];
            if constexpr (P_IS_W) {
                const int m = m0 + 16 * i + r16, n = n0 + 16 * j + 4 * q;
                if (m >= a.M) continue;
                float* to = a.y + (size_t)m * a.N + n;
                if (n + 3 < a.N && !accum) {
                    *reinterpret_cast<v4f_any*>(to) = v4f{o[0], o[1], o[2], o[3]};
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (n + e < a.N) to[e] = accum ? o[e] + to[e] : o[e];
                }
            } else {
                const int n = n0 + 16 * j + r16;
                if (mp >= a.M || n >= a.N) continue;
                float* to = a.y + ((size_t)bi * a.N + n) * hw + pix;
                if (mp + 3 < a.M && pix + 3 < hw && !accum) {
                    *reinterpret_cast<v4f_any*>(to) = v4f{o[0], o[1], o[2], o[3]};
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        if (mp + e >= a.M) break;
                        // pixels beyond this image belong to the images after it
                        const int be = divide(mp + e, a.by_hw);
                        float* te = a.y + ((size_t)be * a.N + n) * hw + (mp + e - be * hw);
                        *te = accum ? o[e] + *te : o[e];
                    }
                }
            }
        }
    }
}

template <int MI, int NI, int NST, int XKIND, int WKIND, bool CONV>
static int launch_wk16_one(const GemmArgs& a, hipStream_t st)
{
    constexpr int smem = 4 * wk16_wave_lds(MI, NI, NST, kind_is_4bit(WKIND));
    static_assert(smem <= 160 * 1024, "LDS of a compute unit");
    const int items = ((a.M + 16 * MI - 1) / (16 * MI)) * ((a.N + 16 * NI - 1) / (16 * NI));
    auto kern = gemm_wk16_kernel<MI, NI, NST, XKIND, WKIND, CONV>;
    static std::atomic<uint64_t> allowed{0};   // per instantiation
    if (!allow_dynamic_lds(reinterpret_cast<const void*>(kern), smem, allowed)) return FPQ_ERR_LAUNCH;
    hipLaunchKernelGGL(kern, dim3(items), dim3(256), smem, st, wave_args<CONV>(a));
    return hipGetLastError() == hipSuccess ? FPQ_OK : FPQ_ERR_LAUNCH;
}

template <int XKIND, int WKIND>
static int launch_wk16_shape(const GemmArgs& a, hipStream_t st)
{
    constexpr int NST = kind_is_4bit(WKIND) ? 5 : 4;
    if (a.tile == TILE_WAVE_128x80)
        return a.conv_out ? launch_wk16_one<8, 5, 3, XKIND, WKIND, true>(a, st) : launch_wk16_one<8, 5, 3, XKIND, WKIND, false>(a, st);
    return a.conv_out ? launch_wk16_one<4, 5, NST, XKIND, WKIND, true>(a, st) : launch_wk16_one<4, 5, NST, XKIND, WKIND, false>(a, st);
}

}  // namespace fpq
