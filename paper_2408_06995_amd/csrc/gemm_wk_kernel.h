// Quantized linear / convolution layer on ExMy codes for gfx950: the kernel for problems of few or ragged tiles.
//
// A workgroup owns a 64 x 64 tile of the output and its four wavefronts split K: each computes the whole tile over its own
// quarter of the K range (2 x 2 blocks of 32 x 32) and the four partial tiles are added through LDS at the end.  What that
// buys over wavefronts that split the tile (32 x 32 each):
//   - a code is read from LDS and converted once per workgroup instead of twice: one conversion per MFMA, which fits behind it;
//   - four MFMAs between a fragment's LDS read and its use, where a 32 x 32 wavefront has one and waits for LDS every time;
//   - every wavefront loads what it reads itself (its own LDS ring), so the K loop has no barrier, and the serial chain of a
//     deep K is a quarter as long (a few tiles with K = 13000 would keep a few compute units busy for 100 steps each).
// Codes travel global memory -> LDS as in gemm_dma_kernel.h (buffer loads to LDS, out-of-range lanes deliver code 0), in steps
// of 64 codes: 16 rows of 64 bytes per load, NST stages per wavefront.  With four stages (128 KB) a compute unit holds one
// workgroup, with two it holds two: the launcher takes the first while every compute unit gets at most one tile anyway.
// Such problems are bound by latencies: start-up, the chain of K steps, the reduction.  Measured against 64 x 64 tiles split over the
// wavefronts and staged through registers: 40 x 5120 -> 1280 18 -> 9.8 us (with K slices), 1407 x 3312 -> 749 23.5 -> 19 us,
// 320 x 64 x 64 -> 320, 3 x 3: 27 -> 19 us, 1446 x 15 x 89 -> 469, 3 x 3: 74 -> 19 us.
#pragma once
#include "gemm_dma_kernel.h"

namespace fpq {

constexpr int wk_wave_lds(int nst, bool w4) { return nst * (64 * 64 + (w4 ? 64 * 32 : 64 * 64)) < 16384 ? 16384 : nst * (64 * 64 + (w4 ? 64 * 32 : 64 * 64)); }

template <int NST, int XKIND, int WKIND, int ACC, bool CONV, bool QOUT>
__device__ __forceinline__ void gemm_wk_tile(const WaveArgs<CONV>& a, int item, uint8_t* smem)
{
    constexpr bool W4 = kind_is_4bit(WKIND);
    constexpr int XTILE = 64 * 64, WTILE = W4 ? 64 * 32 : 64 * 64, STAGE = XTILE + WTILE;
    constexpr int XLD = 4, WLD = W4 ? 2 : 4, LOADS = XLD + WLD;
    constexpr int WAVE_LDS = wk_wave_lds(NST, W4);   // ring of one wavefront, later its partial tile
    // P = operand along the accumulator registers, Q = operand along the lanes.  NCHW results want lanes along the pixels.
    constexpr bool P_IS_W = CONV && !QOUT;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, g = lane >> 5;

    // Work items = (tile, K slice), tile-major.  Ids go round-robin over the 8 XCDs: each takes a contiguous run.
    const int tiles_w = (a.N + 63) / 64, tiles_x = (a.M + 63) / 64;
    const int nitems = tiles_w * tiles_x * a.splits;
    {
        const int per = nitems >> 3;
        if (item < (per << 3)) item = (item & 7) * per + (item >> 3);
    }
    const int tile = item / a.splits, sl = item - tile * a.splits;
    const int tx = tile / tiles_w, tw = tile - tx * tiles_w;
    const int m0 = tx * 64, n0 = tw * 64;

    // this wavefront's steps of 64 codes
    const int nks = (a.Kreal + 63) / 64;
    const int s_lo = nks * sl / a.splits, s_cnt = nks * (sl + 1) / a.splits - s_lo;   // (at most 2^25 steps, 32 slices)
    const int k_lo = s_lo + s_cnt * wave / 4, nk = s_lo + s_cnt * (wave + 1) / 4 - k_lo;

    // ---- loads: load i of the activations covers rows 16 i .. + 15; lane p holds row p / 4 of them, LDS chunk p % 4, i.e. logical
    // chunk (p % 4) ^ swizzle(row); weights of 8 bits likewise, of 4 bits rows of 32 bytes, 32 rows per load
    const v4i xrsrc = make_rsrc(a.x, a.x_bytes);
    const v4i wrsrc = make_rsrc(a.wrows, a.w_bytes);
    const unsigned lds0 = (unsigned)(size_t)((__attribute__((address_space(3))) void*)smem) + wave * WAVE_LDS;
    constexpr unsigned OOB = 0x80000000u;
    const int xc = (lane & 3) ^ ((lane >> 4) & 3);
    unsigned xbase[XLD], xmask[XLD], wbase[WLD];
    int x_k = k_lo * 64 + xc * 16, x_ci = x_k, x_kh = 0, x_kw = 0, x_tap = 0, x_sel = 31;
    unsigned x_delta = 0;
    {
#pragma unroll
        for (int i = 0; i < XLD; ++i) {
            const int m = m0 + 16 * i + (lane >> 2);
            if constexpr (CONV) {
                conv_row(a, m, xbase[i], xmask[i]);
                if (m >= a.M) xmask[i] = 0u;                       // no tap of this row lies inside
            } else {
                xbase[i] = (unsigned)m * (unsigned)a.Cp;
                xmask[i] = m < a.M ? 1u : 0u;
            }
        }
        if constexpr (CONV) {
            x_tap = divide(x_k, a.by_cp);
            x_ci = x_k - x_tap * a.Cp;
            x_kh = divide(x_tap, a.by_kw);
            x_kw = x_tap - x_kh * a.kw;
        }
        const unsigned wrow_bytes = W4 ? (unsigned)a.Kpad / 2 : (unsigned)a.Kpad;
#pragma unroll
        for (int i = 0; i < WLD; ++i) {
            const int row = W4 ? 32 * i + (lane >> 1) : 16 * i + (lane >> 2);
            const int chunk = W4 ? (lane & 1) ^ ((row >> 3) & 1) : xc;
            const int n = n0 + row;
            wbase[i] = n < a.N ? (unsigned)n * wrow_bytes + (unsigned)k_lo * (W4 ? 32u : 64u) + chunk * 16 : OOB;
        }
    }
    int todo = nk;                                                 // steps whose loads have not gone out
    int live = nk > 0 ? -1 : 1;                                       // what dma16_live wants
    // scale and bias of the column (NCHW: of channel l32 of the block) that this lane finishes: fetched ahead of the K loop
    const float sxa = (a.sx_dev ? a.sx_dev[0] : a.sx) * a.alpha;
    float my_scale = 0.0f, my_bias = 0.0f;
    {
        const int n = n0 + 32 * (P_IS_W ? wave >> 1 : wave & 1) + l32;
        if (n < a.N) {
            my_scale = a.sw[n];
            if (a.bias && sl == 0) my_bias = a.bias[n];
        }
    }
    auto x_refresh = [&]() {
        x_sel = x_k < a.Kreal ? x_tap : 31;
        x_delta = CONV ? (unsigned)((x_kh * a.W + x_kw) * a.Cp + x_ci) : (unsigned)x_k;
    };
    x_refresh();
    auto issue_one = [&](int idx, int slot) {
        const unsigned at = lds0 + slot * STAGE;
        if (idx < XLD) {
            const unsigned off = ((xmask[idx] >> x_sel) & 1u) ? xbase[idx] + x_delta : OOB;
            dma16_live(xrsrc, off, at + idx * 1024, live);
        } else {
            dma16_live(wrsrc, wbase[idx - XLD], at + XTILE + (idx - XLD) * 1024, live);
        }
    };
    auto issue_advance = [&]() {
        if (--todo <= 0) live = 1;
#pragma unroll
        for (int i = 0; i < WLD; ++i)
            if (wbase[i] != OOB) wbase[i] += W4 ? 32 : 64;
        x_k += 64;
        if (CONV) {
            x_ci += 64;
            while (x_ci >= a.Cp) {
                x_ci -= a.Cp;
                ++x_tap;
                if (++x_kw == a.kw) { x_kw = 0; ++x_kh; }
            }
        }
        x_refresh();
    };
#pragma unroll
    for (int s = 0; s < NST - 1; ++s) {
#pragma unroll
        for (int idx = 0; idx < LOADS; ++idx) issue_one(idx, s);
        issue_advance();
    }

    v16f acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

    // ---- K loop.  Fragments 0, 1 = operand P, 2, 3 = operand Q.
    const GenFmt wfm{a.we, a.wm, a.wb}, xfm{a.xe, a.xm, a.xb};
    const uint8_t* ring = smem + wave * WAVE_LDS;
    constexpr int PKIND = P_IS_W ? WKIND : XKIND, QKIND = P_IS_W ? XKIND : WKIND;
    constexpr int PFMT = mfma_fmt(PKIND), QFMT = mfma_fmt(QKIND);   // immediates of the MFMA
    auto is_w = [](int f) { return P_IS_W ? f < 2 : f >= 2; };
    auto w4_off = [](int row, int chunk) { return row * 32 + ((chunk ^ ((row >> 3) & 1)) << 4); };
    // the next slot's loads have landed when at most the NST - 2 younger groups are outstanding
    auto wait_next = [&]() {
        __builtin_amdgcn_s_waitcnt(vmcnt_imm((NST - 2) * LOADS));
        asm volatile("" ::: "memory");
    };
    wait_next();
    int slot = 0, to = NST - 1;
    if constexpr (ACC == FPQ_ACC_FP32) {
        // 64 codes = two rounds of LDS reads (lane half g: codes 32 j + 16 g .. + 15) x two MFMA steps; the slots as in
        // gemm_dma_kernel: after MFMA k of step st the LDS read of fragment k for the next round, its conversion for step st + 1
        uint4 raw[2][4];
        v8bf frag[2][4];
        auto lds_read = [&](int s, int j, int f) -> uint4 {
            const uint8_t* base = ring + s * STAGE;
            const int row = 32 * (f & 1) + l32;
            if (is_w(f)) {
                if (W4) {
                    const uint2 v = *reinterpret_cast<const uint2*>(base + XTILE + w4_off(row, j) + g * 8);
                    return make_uint4(v.x, v.y, 0, 0);
                }
                return *reinterpret_cast<const uint4*>(base + XTILE + lds_off<64>(row, 2 * j + g));
            }
            return *reinterpret_cast<const uint4*>(base + lds_off<64>(row, 2 * j + g));
        };
        auto dec = [&](int st, int f) -> v8bf {
            const uint4 r = raw[(st >> 1) & 1][f];
            const bool t = st & 1;
            if (is_w(f))
                return W4 ? decode8<WKIND>(t ? r.y : r.x, 0u, wfm) : decode8<WKIND>(t ? r.z : r.x, t ? r.w : r.y, wfm);
            return decode8<XKIND>(t ? r.z : r.x, t ? r.w : r.y, xfm);
        };
#pragma unroll
        for (int f = 0; f < 4; ++f) raw[0][f] = lds_read(0, 0, f);
#pragma unroll
        for (int f = 0; f < 4; ++f) frag[0][f] = dec(0, f);
        for (int kt = 0; kt < nk; ++kt) {
            const int next = slot + 1 == NST ? 0 : slot + 1;
#pragma unroll
            for (int st = 0; st < 4; ++st) {
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    acc[k >> 1][k & 1] = mfma_exact<PKIND>(frag[st & 1][k >> 1], frag[st & 1][2 + (k & 1)], acc[k >> 1][k & 1]);
                    if (st == 2 && k == 0) wait_next();
                    if (st == 0) raw[1][k] = lds_read(slot, 1, k);
                    if (st == 2) raw[0][k] = lds_read(next, 0, k);
                    frag[(st + 1) & 1][k] = dec((st + 1) & 3, k);
                    if (st < 2 && st * 4 + k < LOADS) issue_one(st * 4 + k, to);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            issue_advance();
            to = to + 1 == NST ? 0 : to + 1;
            slot = next;
        }
    } else {
        // codes straight into the 8-bit / 4-bit MFMA, one 64-code step each (operand layout: see gemm_dma_kernel.h)
        v8i frag8[2][4];
        auto lds_read8 = [&](int s, int f) -> v8i {
            const uint8_t* base = ring + s * STAGE;
            const int row = 32 * (f & 1) + l32;
            union { v8i v; uint4 q[2]; } u;
            if (is_w(f) && W4) {
                u.q[0] = *reinterpret_cast<const uint4*>(base + XTILE + w4_off(row, g));
                u.q[1] = make_uint4(0, 0, 0, 0);
            } else {
                if (is_w(f)) base += XTILE;
                u.q[0] = *reinterpret_cast<const uint4*>(base + lds_off<64>(row, g));
                u.q[1] = *reinterpret_cast<const uint4*>(base + lds_off<64>(row, 2 + g));
            }
            return u.v;
        };
#pragma unroll
        for (int f = 0; f < 4; ++f) frag8[0][f] = lds_read8(0, f);
        auto step = [&](int cur) {
            const int next = slot + 1 == NST ? 0 : slot + 1;
#pragma unroll
            for (int idx = 0; idx < LOADS; ++idx) issue_one(idx, to);
            issue_advance();
            wait_next();
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                acc[k >> 1][k & 1] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
                    frag8[cur][k >> 1], frag8[cur][2 + (k & 1)], acc[k >> 1][k & 1], PFMT, QFMT, 0, 0, 0, 0);
                frag8[cur ^ 1][k] = lds_read8(next, k);
                __builtin_amdgcn_sched_barrier(0);
            }
            to = to + 1 == NST ? 0 : to + 1;
            slot = next;
        };
        for (int kt = 0; kt + 1 < nk; kt += 2) {
            step(0);
            step(1);
        }
        if (nk & 1) step(0);
    }
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));                      // no load may land in LDS from here on
    asm volatile("" ::: "memory");

    // ---- add the four partial tiles: every wavefront leaves its own in LDS (its own ring: [block][quad of registers][lane]),
    // wavefront w adds up block (w / 2, w % 2), in the order of K
    float4* mine = reinterpret_cast<float4*>(smem + wave * WAVE_LDS) + lane;
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int q = 0; q < 4; ++q)
            mine[(b * 4 + q) * 64] = make_float4(acc[b >> 1][b & 1][4 * q], acc[b >> 1][b & 1][4 * q + 1], acc[b >> 1][b & 1][4 * q + 2],
                                                 acc[b >> 1][b & 1][4 * q + 3]);
    __syncthreads();
    float out[16];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        float4 v[4];
#pragma unroll
        for (int w = 0; w < 4; ++w) v[w] = (reinterpret_cast<const float4*>(smem + w * WAVE_LDS) + lane)[(wave * 4 + q) * 64];
        out[4 * q] = ((v[0].x + v[1].x) + v[2].x) + v[3].x;
        out[4 * q + 1] = ((v[0].y + v[1].y) + v[2].y) + v[3].y;
        out[4 * q + 2] = ((v[0].z + v[1].z) + v[2].z) + v[3].z;
        out[4 * q + 3] = ((v[0].w + v[1].w) + v[2].w) + v[3].w;
    }

    // ---- epilogue of a 32 x 32 block: register r is row 8 (r / 4) + 4 g + r % 4 of operand P, the lane column l32 of operand Q
    const int pb = 32 * (wave >> 1) + 4 * g, qb = 32 * (wave & 1) + l32;
    float* const yout = a.splits > 1 ? a.partial + (size_t)sl * ((size_t)a.M * a.N) : a.y;
    const bool accum = a.accumulate && a.splits == 1;
    if constexpr (P_IS_W) {
        // NCHW: the lane is a pixel, registers are channels; 32 lanes write 128 consecutive bytes (two pieces across images)
        float* table = reinterpret_cast<float*>(smem + 4 * WAVE_LDS) + wave * 64;
        table[(g << 5) | l32] = g ? my_bias : sxa * my_scale;                               // [scales][biases] of the block's channels
        const int hw = a.Ho * a.Wo;
        const int m = m0 + qb;
        if (m < a.M) {
            const int bi = m / hw;
            float* yp = yout + (size_t)bi * a.N * hw + (m - bi * hw);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float4 s4 = *reinterpret_cast<const float4*>(table + 8 * q + 4 * g);
                const float4 b4 = *reinterpret_cast<const float4*>(table + 32 + 8 * q + 4 * g);
                const float sc[4] = {s4.x, s4.y, s4.z, s4.w}, bv[4] = {b4.x, b4.y, b4.z, b4.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int n = n0 + pb + 8 * q + e;
                    if (n < a.N) {
                        const float v = out[4 * q + e] * sc[e] + bv[e];
                        float* at = yp + (size_t)n * hw;
                        *at = accum ? v + *at : v;
                    }
                }
            }
        }
    } else {
        const int n = n0 + qb;
        const float sc = sxa * my_scale, bv = my_bias;
        const int mb = m0 + pb;
        if (QOUT && a.splits == 1) {
            const QParams qy{a.ym, a.yb, a.yem, a.yc};
            const float ry = inv_scale(a.sy, a.sy_dev);
            uint32_t sel1, sel2;
            const int qpos = l32 & 3;
            transpose_selectors(qpos, sel1, sel2);
            const int no = a.act == FPQ_ACT_GEGLU ? ((n0 + qb - l32) >> 1) + l32 : n;       // output column of this lane
            const bool lane_out = a.act == FPQ_ACT_GEGLU ? l32 < 16 : true;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float v[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = n < a.N ? out[4 * q + e] * sc + bv : 0.0f;
                if (a.act == FPQ_ACT_SILU) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = act_silu(v[e]);
                } else if (a.act == FPQ_ACT_GEGLU) {
                    // lanes 0-15 of each 32 hold the values, lanes 16-31 the gates of the same outputs
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] *= act_gelu(lane_xor16(v[e]));
                }
                uint32_t w;
                if (a.ykind == 1)
                    w = codes_of4<1>(v[0], v[1], v[2], v[3], ry, qy);
                else if (a.ykind == 2)
                    w = codes_of4<2>(v[0], v[1], v[2], v[3], ry, qy);
                else
                    w = codes_of4<0>(v[0], v[1], v[2], v[3], ry, qy);
                if (a.act != FPQ_ACT_GEGLU && n >= a.N) w = 0;                              // padding columns: code 0
                // 4 x 4 bytes inside each quad of lanes: afterwards the lane has row 8 q + 4 g + qpos, four columns from no - qpos
                const uint32_t row = quad_transpose_bytes(w, sel1, sel2);
                const int m = mb + 8 * q + qpos;
                if (lane_out && m < a.M && no - qpos < a.ldq)                               // ldq % 4 == 0
                    *reinterpret_cast<uint32_t*>(a.yq + (size_t)m * a.ldq + (no - qpos)) = row;
            }
        } else {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int m = mb + 8 * (r >> 2) + (r & 3);
                if (n < a.N && m < a.M) {
                    const float v = out[r] * sc + bv;
                    float* at = yout + (size_t)m * a.N + n;
                    *at = accum ? v + *at : v;
                }
            }
        }
    }
}

template <int NST, int XKIND, int WKIND, int ACC, bool CONV, bool QOUT>
__global__ __launch_bounds__(256, (NST <= 2 ? 2 : 1)) void gemm_wk_kernel(const WaveArgs<CONV> a)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    gemm_wk_tile<NST, XKIND, WKIND, ACC, CONV, QOUT>(a, blockIdx.x, smem);
}

template <int NST, int XKIND, int WKIND, int ACC, bool CONV, bool QOUT>
static int launch_wk_one(const GemmArgs& a, hipStream_t st)
{
    constexpr int smem = 4 * wk_wave_lds(NST, kind_is_4bit(WKIND)) + 1024;   // + scales and biases of NCHW blocks
    const int items = ((a.M + 63) / 64) * ((a.N + 63) / 64) * a.splits;
    auto kern = gemm_wk_kernel<NST, XKIND, WKIND, ACC, CONV, QOUT>;
    if (smem > 64 * 1024) {
        static std::atomic<uint64_t> allowed{0};   // per instantiation
        if (!allow_dynamic_lds(reinterpret_cast<const void*>(kern), smem, allowed)) return FPQ_ERR_LAUNCH;
    }
    hipLaunchKernelGGL(kern, dim3(items), dim3(256), smem, st, wave_args<CONV>(a));
    if (a.splits > 1) return launch_splitk_reduce(a, st);
    return hipGetLastError() == hipSuccess ? FPQ_OK : FPQ_ERR_LAUNCH;
}

template <int XKIND, int WKIND, int ACC, bool QOUT>
static int launch_wk_shape(const GemmArgs& a, hipStream_t st)
{
    if (a.tile == TILE_WAVE_K4)
        return a.conv_out ? launch_wk_one<4, XKIND, WKIND, ACC, true, QOUT>(a, st) : launch_wk_one<4, XKIND, WKIND, ACC, false, QOUT>(a, st);
    return a.conv_out ? launch_wk_one<2, XKIND, WKIND, ACC, true, QOUT>(a, st) : launch_wk_one<2, XKIND, WKIND, ACC, false, QOUT>(a, st);
}

}  // namespace fpq
