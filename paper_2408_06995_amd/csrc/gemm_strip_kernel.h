// Quantized linear layer / 1 x 1 convolution on ExMy codes for gfx950, K of at most 320 codes: weights stay in registers.
//
// With a short K the result is most of the traffic and a tile of the LDS ring is three K steps long, so a kernel that walks
// (tile, K step) spends its time on start-up: it waits for a step's loads, which retire behind the stores of the tile before, and the
// four wavefronts of a workgroup meet at a barrier each step.  Here a wavefront keeps the weights of a strip of 64 columns over all of
// K as MFMA operands in registers (K = 320: 160 of its 256) and walks down the rows in blocks of 32:
//   - a code of the activations is read from LDS and converted once for two MFMAs, a weight once per workgroup life;
//   - a block's activations are one contiguous piece of memory (32 rows x K codes) that the wavefront itself loads into its own LDS
//     ring: after the weights are in place there is no barrier, and the two wavefronts of a SIMD drift apart, so that one multiplies
//     while the other stores;
//   - the loads of block i + 1 go out before the stores of block i, and the wait for them counts those stores instead of draining them.
// Two workgroups per compute unit: 2 x 4 wavefronts x 20 KB of ring are all 160 KB of LDS at K = 320, which is where the limit
// on K comes from (the registers give out at the same point).
#pragma once
#include <utility>

#include "gemm_dma_kernel.h"

namespace fpq {

enum StripOut : int { STRIP_ROWS = 0, STRIP_NCHW = 1, STRIP_CODES = 2 };

constexpr int strip_block_bytes(int nk64) { return 32 * 64 * nk64; }   // activations of one block: 32 rows x 64 nk64 codes
constexpr int strip_stages(int nk64) { return nk64 >= 4 ? 2 : nk64 == 3 ? 3 : 4; }
constexpr int strip_lds_bytes(int nk64) { return 4 * strip_stages(nk64) * strip_block_bytes(nk64); }

// Value of lane r of each row of 16 lanes, in all lanes of that row.
template <int R>
__device__ __forceinline__ float row_lane(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x150 + R, 0xF, 0xF, true));
}

template <class F, int... R>
__device__ __forceinline__ void for_constants(std::integer_sequence<int, R...>, F f)
{
    (f(std::integral_constant<int, R>{}), ...);
}

// NK64: K rounded up to 64 codes.  P = operand along the accumulator registers,
// Q = along the lanes: results in rows of N want lanes along the columns, NCHW results and codes (four columns to a word) lanes
// along the rows.
template <int NK64, int XKIND, int WKIND, int ACC, int OUT>
__global__ __launch_bounds__(256, 2) void gemm_strip_kernel(const GemmArgs a)
{
    constexpr bool P_IS_W = OUT != STRIP_ROWS;
    constexpr bool W4 = kind_is_4bit(WKIND);
    constexpr int NC = 4 * NK64;                              // 16-byte chunks per row of activations
    constexpr int G = NC % 16 == 0 ? 16 : NC % 8 == 0 ? 8 : 4;// gcd(NC, 16): see swz
    constexpr int NWC = W4 ? NC / 2 : NC;                     // and per row of weights
    constexpr int GW = W4 ? (NWC % 16 == 0 ? 16 : NWC % 8 == 0 ? 8 : NWC % 4 == 0 ? 4 : 2) : G;
    constexpr int NST = strip_stages(NK64);
    constexpr int BLOCK = strip_block_bytes(NK64);
    constexpr int LOADS = BLOCK / 1024;
    constexpr int STORES = OUT == STRIP_CODES ? 1 : 32;       // of a block of a whole strip, at least
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l32 = lane & 31, g = lane >> 5;

    // Workgroups: (chunk of the row blocks, strip), strips innermost; chunk c has the groups of four blocks c, c + chunks, ..., so that
    // all of them write near each other.  Ids go round-robin over the 8 XCDs; each takes a contiguous run of (chunk, strip), so that
    // strips that read the same activations share an L2.
    const int strips = (a.N + 63) / 64;
    int q = blockIdx.x;
    {
        const int per = gridDim.x >> 3;
        if (q < (per << 3)) q = (q & 7) * per + (q >> 3);
    }
    const int chunk = q / strips;
    const int n0 = (q - chunk * strips) * 64;
    const int nblocks = (a.M + 31) / 32;
    const int step = 4 * (gridDim.x / strips);
    int blk = 4 * chunk + wave;                               // this wavefront's blocks: blk, blk + step, ...

    const v4i xrsrc = make_rsrc(a.x, a.x_bytes);
    const unsigned lds0 = (unsigned)(size_t)((__attribute__((address_space(3))) void*)smem);
    const uint8_t* ring = smem + wave * (NST * BLOCK);
    const unsigned ring0 = lds0 + wave * (NST * BLOCK);
    constexpr unsigned OOB = 0x80000000u;

    // Rows lie NC chunks apart in LDS; chunk c of a row sits at c ^ swz(row), which stays inside the row (G divides NC) and makes the
    // chunks c of any 16 consecutive rows fall on all 64 banks: rows are a multiple of G apart mod 16, swz fills the gaps.
    auto swz = [](int row) { return (row / (16 / G)) & (G - 1); };
    auto wswz = [](int row) { return (row / (16 / GW)) & (GW - 1); };

    // ---- weights and scales of the strip, through the last stage of the ring: wavefront w brings rows 16 w .. + 15, the first two also
    // the 64 scales and biases.
    {
        const v4i wrsrc = make_rsrc(a.wrows, a.w_bytes);
        const unsigned wrow_bytes = W4 ? (unsigned)a.Kpad / 2 : (unsigned)a.Kpad;
        const unsigned to = ring0 + (NST - 1) * BLOCK;
#pragma unroll
        for (int i = 0; i < (16 * NWC + 63) / 64; ++i) {
            const int p = 64 * i + lane, row = p / NWC, c = (p - row * NWC) ^ wswz(row);
            const int n = n0 + 16 * wave + row;
            dma16(wrsrc, row < 16 && n < a.N ? (unsigned)n * wrow_bytes + 16u * c : OOB, to + 1024 * i);
        }
        if (wave < 2) {
            const v4i srsrc = make_rsrc(wave == 0 ? a.sw : a.bias, wave == 0 || a.bias ? (unsigned)a.N * 4u : 0u);
            dma16(srsrc, lane < 16 ? (unsigned)(n0 * 4 + lane * 16) : OOB, to + BLOCK / 2);
        }
    }

    // ---- activations: load i covers LDS chunks 64 i .. + 63 of a block; two halves of 16 rows look alike
    unsigned xoff[NK64];
#pragma unroll
    for (int i = 0; i < NK64; ++i) {
        const int p = 64 * i + lane, row = p / NC, c = (p - row * NC) ^ swz(row);
        xoff[i] = 16 * c < a.Cp ? (unsigned)row * (unsigned)a.Cp + 16u * c : OOB;   // K beyond the row: zeros
    }
    int live = -1;                                            // what dma16_live wants
    // rows beyond M lie beyond the buffer: zeros
    auto issue = [&](int block, int stage) {
        const unsigned base = (unsigned)block * (32u * (unsigned)a.Cp);
        live = block < nblocks ? -1 : 1;
#pragma unroll
        for (int i = 0; i < LOADS; ++i) {
            const unsigned at = base + (i >= NK64 ? 16u * (unsigned)a.Cp : 0u);
            const unsigned off = xoff[i % NK64];
            dma16_live(xrsrc, off == OOB ? OOB : off + at, ring0 + stage * BLOCK + 1024 * i, live);
        }
    };
#pragma unroll
    for (int s = 0; s < NST - 1; ++s) issue(blk + step * s, s);

    const float sxa = (a.sx_dev ? a.sx_dev[0] : a.sx) * a.alpha;
    const GenFmt wfm{a.we, a.wm, a.wb}, xfm{a.xe, a.xm, a.xb};
    v8bf w[ACC == FPQ_ACC_FP32 ? 2 : 1][ACC == FPQ_ACC_FP32 ? 4 * NK64 : 1];
    v8i w8[ACC == FPQ_ACC_FP32 ? 1 : 2][ACC == FPQ_ACC_FP32 ? 1 : NK64];
    float sc[2], bv[2];

    __builtin_amdgcn_s_waitcnt(vmcnt_imm((NST - 1) * LOADS));
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    {
        const uint8_t* last = smem + (NST - 1) * BLOCK;       // of wavefront 0; the others' lie NST blocks apart
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int row = 32 * j + l32;
            const uint8_t* at = last + (row >> 4) * (NST * BLOCK) + (row & 15) * (NWC * 16);
            const int sz = wswz(row & 15);
            if constexpr (ACC == FPQ_ACC_FP32) {
#pragma unroll
                for (int c = 0; c < 2 * NK64; ++c) {          // 32 codes: lane half g takes 16 of them, two MFMA steps
                    if constexpr (W4) {
                        const uint2 v = *reinterpret_cast<const uint2*>(at + ((c ^ sz) << 4) + g * 8);
                        w[j][2 * c] = decode8<WKIND>(v.x, 0u, wfm);
                        w[j][2 * c + 1] = decode8<WKIND>(v.y, 0u, wfm);
                    } else {
                        const uint4 v = *reinterpret_cast<const uint4*>(at + (((2 * c + g) ^ sz) << 4));
                        w[j][2 * c] = decode8<WKIND>(v.x, v.y, wfm);
                        w[j][2 * c + 1] = decode8<WKIND>(v.z, v.w, wfm);
                    }
                }
            } else {
#pragma unroll
                for (int c = 0; c < NK64; ++c) {              // 64 codes: the operand layout of the instruction, see gemm_dma_kernel.h
                    union { v8i v; uint4 h[2]; } u;
                    if constexpr (W4) {
                        u.h[0] = *reinterpret_cast<const uint4*>(at + (((2 * c + g) ^ sz) << 4));
                        u.h[1] = make_uint4(0, 0, 0, 0);
                    } else {
                        u.h[0] = *reinterpret_cast<const uint4*>(at + (((4 * c + g) ^ sz) << 4));
                        u.h[1] = *reinterpret_cast<const uint4*>(at + (((4 * c + 2 + g) ^ sz) << 4));
                    }
                    w8[j][c] = u.v;
                }
            }
            // lanes along the columns: the lane's own scale; along the rows: lane r of each 16 holds that of register r
            const int col = 32 * j + (P_IS_W ? 8 * ((lane & 15) >> 2) + 4 * g + (lane & 3) : l32);
            sc[j] = sxa * *reinterpret_cast<const float*>(last + BLOCK / 2 + 4 * col);
            bv[j] = *reinterpret_cast<const float*>(last + NST * BLOCK + BLOCK / 2 + 4 * col);
        }
    }
    __builtin_amdgcn_s_waitcnt(0xC07F);                       // lgkmcnt(0): everything has left the last stage
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");

    // ---- one block: acc[j] = rows 32 blk .. + 31 of the activations times columns 32 j .. + 31 of the strip
    v16f acc[2];
    constexpr int PKIND = P_IS_W ? WKIND : XKIND;
    auto compute = [&](int stage) {
        // what depends on the lane is worked out anew for each block, here and in the epilogue: with the weights there are no
        // registers to keep it in
        int fresh = lane;
        asm volatile("" : "+v"(fresh));
        const int l32 = fresh & 31, g = fresh >> 5;
        const uint8_t* at = ring + stage * BLOCK + l32 * (NC * 16);
        // chunk k + g of the lane's row (k even): the bits of k that swz can reach are exchanged in one xor, the others are an offset
        const int xsw = (g ^ swz(l32)) << 4;
        auto chunk_at = [&](int k) { return (k & ~(G - 1)) * 16 + (xsw ^ ((k & (G - 1)) << 4)); };
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[j][r] = 0.0f;
        if constexpr (ACC == FPQ_ACC_FP32) {
            // the slots of gemm_dma_kernel: behind the two MFMAs of a step the conversion for the next step and, every other step, the
            // LDS read two chunks ahead
            uint4 raw[2];
            v8bf frag[2];
            auto read = [&](int c) { return *reinterpret_cast<const uint4*>(at + chunk_at(2 * c)); };
            auto dec = [&](int st) {
                const uint4 r = raw[(st >> 1) & 1];
                return (st & 1) ? decode8<XKIND>(r.z, r.w, xfm) : decode8<XKIND>(r.x, r.y, xfm);
            };
            raw[0] = read(0);
            raw[1] = read(1);
            frag[0] = dec(0);
#pragma unroll
            for (int st = 0; st < 4 * NK64; ++st) {
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[j] = P_IS_W ? mfma_exact<PKIND>(w[j][st], frag[st & 1], acc[j]) : mfma_exact<PKIND>(frag[st & 1], w[j][st], acc[j]);
                if (st + 1 < 4 * NK64) frag[(st + 1) & 1] = dec(st + 1);
                if ((st & 1) == 0 && st >= 2 && st / 2 + 1 < 2 * NK64) raw[(st / 2 + 1) & 1] = read(st / 2 + 1);
                __builtin_amdgcn_sched_barrier(0);
            }
        } else {
            constexpr int PF = mfma_fmt(P_IS_W ? WKIND : XKIND), QF = mfma_fmt(P_IS_W ? XKIND : WKIND);
            v8i f8[2];
            auto read8 = [&](int c) {
                union { v8i v; uint4 h[2]; } u;
                u.h[0] = *reinterpret_cast<const uint4*>(at + chunk_at(4 * c));
                u.h[1] = *reinterpret_cast<const uint4*>(at + chunk_at(4 * c + 2));
                return u.v;
            };
            f8[0] = read8(0);
#pragma unroll
            for (int c = 0; c < NK64; ++c) {
                if (c + 1 < NK64) f8[(c + 1) & 1] = read8(c + 1);
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[j] = P_IS_W ? __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(w8[j][c], f8[c & 1], acc[j], PF, QF, 0, 0, 0, 0)
                                    : __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(f8[c & 1], w8[j][c], acc[j], PF, QF, 0, 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };

    // ---- results of a block.  Register r = 4 q + e is row (P = activations) or column (P = weights) 8 q + 4 g + e.
    const bool whole_strip = n0 + 64 <= a.N;
    // Rows (planes) of whole 128-byte lines leave with streaming stores; where lines are shared, streaming stores send them to memory
    // in pieces (33000 x 64 -> 1001: 70 us, 37 us with stores that meet in the L2; rows of whole lines 20 to 35 % the other way).
    const bool whole_lines = ((OUT == STRIP_NCHW ? a.Ho * a.Wo : a.N) & 31) == 0;
    const QParams qy{a.ym, a.yb, a.yem, a.yc};
    float ry = 0.0f;                                          // the same in every lane: a scalar register
    if (OUT == STRIP_CODES)
        ry = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, inv_scale(a.sy, a.sy_dev))));
    const int hw = OUT == STRIP_NCHW ? a.Ho * a.Wo : 1;
    auto epilogue = [&](int m0) {
        int fresh = lane;
        asm volatile("" : "+v"(fresh));
        const int l32 = fresh & 31, g = fresh >> 5;
        if constexpr (OUT == STRIP_ROWS) {
            const unsigned lane_off = (unsigned)(4 * g * a.N + l32);
            if (m0 + 32 <= a.M) {
                auto store_all = [&](auto streaming) {
                    auto put = [&](int r, int j) {
                        float* rowp = a.y + (size_t)(m0 + 8 * (r >> 2) + (r & 3)) * a.N + n0;   // uniform
                        const float v = acc[j][r] * sc[j] + bv[j];
                        if constexpr (decltype(streaming)::value)
                            store_out(rowp + lane_off + 32 * j, v);
                        else
                            rowp[lane_off + 32 * j] = v;
                    };
                    if (whole_strip) {
#pragma unroll
                        for (int r = 0; r < 16; ++r) {
                            put(r, 0);
                            put(r, 1);
                        }
                    } else {
#pragma unroll
                        for (int j = 0; j < 2; ++j)
                            if (n0 + 32 * j + l32 < a.N) {
#pragma unroll
                                for (int r = 0; r < 16; ++r) put(r, j);
                            }
                    }
                };
                if (whole_lines)
                    store_all(std::true_type{});
                else
                    store_all(std::false_type{});
                return;
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int m = m0 + 8 * (r >> 2) + 4 * g + (r & 3);
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    if (m < a.M && n0 + 32 * j + l32 < a.N) a.y[(size_t)m * a.N + n0 + 32 * j + l32] = acc[j][r] * sc[j] + bv[j];
            }
        } else {
            const int m = m0 + l32;
            // scale and bias of register r come from lane r of the row of 16 (all lanes have to take part); spread anew for each block, or 64 registers would hold them
            asm volatile("" : "+v"(sc[0]), "+v"(sc[1]), "+v"(bv[0]), "+v"(bv[1]));
            auto value = [&](auto rc, int j) {
                constexpr int R = decltype(rc)::value;
                return acc[j][R] * row_lane<R>(sc[j]) + row_lane<R>(bv[j]);
            };
            if constexpr (OUT == STRIP_NCHW) {
                // the lane is a pixel, registers are channels: 32 lanes write 128 consecutive bytes of a channel
                const int bi = m / hw;
                unsigned plane = (unsigned)hw;                // per lane: uniform, the offsets of all planes would be kept in (spilled)
                asm volatile("" : "+v"(plane));               // scalar registers, also through the block loop
                float* yp = a.y + ((size_t)bi * a.N + n0 + 4 * g) * plane + (m - bi * hw);
                auto store_all = [&](auto whole, auto streaming) {
                    for_constants(std::make_integer_sequence<int, 32>{}, [&](auto rc) {
                        constexpr int R = decltype(rc)::value, C = 8 * (R >> 2) + (R & 3);
                        const float v = value(std::integral_constant<int, R & 15>{}, R >> 4);
                        if constexpr (decltype(whole)::value && decltype(streaming)::value)
                            store_out(yp, v);
                        else if constexpr (decltype(whole)::value)
                            *yp = v;
                        else if (m < a.M && n0 + C + 4 * g < a.N)
                            *yp = v;
                        yp += (R & 3) == 3 ? 5 * (size_t)plane : (size_t)plane;
                        if ((R & 3) == 3) __builtin_amdgcn_sched_barrier(0);   // or the addresses of all of them come first, and spill
                    });
                };
                if (whole_strip && m0 + 32 <= a.M && whole_lines)
                    store_all(std::true_type{}, std::true_type{});
                else if (whole_strip && m0 + 32 <= a.M)
                    store_all(std::true_type{}, std::false_type{});
                else
                    store_all(std::false_type{}, std::false_type{});
            } else {
                // a register group q = four consecutive columns of the lane's row = one word of codes
                auto codes = [&](auto kind, auto activation) {
                    constexpr int YK = decltype(kind)::value, ACT = decltype(activation)::value;
                    // (one group at a time, or the values of all of them come first, and spill)
                    constexpr int WORDS = ACT == FPQ_ACT_GEGLU ? 2 : 4;
                    uint32_t word[2][4];
                    for_constants(std::make_integer_sequence<int, 2 * WORDS>{}, [&](auto kc) {
                        constexpr int J = decltype(kc)::value / WORDS, K = decltype(kc)::value % WORDS;
                        float v[4];
                        for_constants(std::make_integer_sequence<int, 4>{}, [&](auto ec) {
                            constexpr int R = 4 * K + decltype(ec)::value;
                            float x = value(std::integral_constant<int, R>{}, J);
                            if constexpr (ACT == FPQ_ACT_SILU) x = act_silu(x);
                            // columns 0 .. 15 of a block of 32 are values, 16 .. 31 their gates
                            if constexpr (ACT == FPQ_ACT_GEGLU) x *= act_gelu(value(std::integral_constant<int, R + 8>{}, J));
                            v[decltype(ec)::value] = x;
                        });
                        word[J][K] = codes_of4<YK>(v[0], v[1], v[2], v[3], ry, qy);
                        __builtin_amdgcn_sched_barrier(0);
                    });
                    // lane halves hold words g, 2 + g, ... of a row: one exchange gives each half 16 consecutive bytes
                    typedef unsigned v2u __attribute__((ext_vector_type(2)));
                    typedef unsigned v4u __attribute__((ext_vector_type(4)));
                    if (ACT == FPQ_ACT_GEGLU) {
                        const v2u p = __builtin_amdgcn_permlane32_swap(word[0][0], word[1][0], false, false);
                        const v2u s = __builtin_amdgcn_permlane32_swap(word[0][1], word[1][1], false, false);
                        const int no = (n0 >> 1) + 16 * g;
                        const v4u o = {p.x, p.y, s.x, s.y};
                        if (m < a.M && no < a.ldq) *reinterpret_cast<v4u*>(a.yq + (size_t)m * a.ldq + no) = o;
                    } else {
#pragma unroll
                        for (int j = 0; j < 2; ++j) {
                            if (!whole_strip) {               // columns N .. ldq - 1 get code 0
#pragma unroll
                                for (int k = 0; k < 4; ++k) {
                                    const int left = a.N - (n0 + 32 * j + 8 * k + 4 * g);
                                    word[j][k] = left >= 4 ? word[j][k] : left <= 0 ? 0u : word[j][k] & ((1u << (8 * left)) - 1u);
                                }
                            }
                            const v2u p = __builtin_amdgcn_permlane32_swap(word[j][0], word[j][2], false, false);
                            const v2u s = __builtin_amdgcn_permlane32_swap(word[j][1], word[j][3], false, false);
                            const int no = n0 + 32 * j + 16 * g;
                            const v4u o = {p.x, p.y, s.x, s.y};
                            if (m < a.M && no < a.ldq) *reinterpret_cast<v4u*>(a.yq + (size_t)m * a.ldq + no) = o;
                        }
                    }
                };
                if (a.ykind == 1) {
                    if (a.act == FPQ_ACT_GEGLU)
                        codes(std::integral_constant<int, 1>{}, std::integral_constant<int, FPQ_ACT_GEGLU>{});
                    else if (a.act == FPQ_ACT_SILU)
                        codes(std::integral_constant<int, 1>{}, std::integral_constant<int, FPQ_ACT_SILU>{});
                    else
                        codes(std::integral_constant<int, 1>{}, std::integral_constant<int, 0>{});
                } else {
                    codes(std::integral_constant<int, 0>{}, std::integral_constant<int, 0>{});
                }
            }
        }
    };

    // ---- the loads of block i + NST - 1 go out ahead of block i.  Younger than the loads of block i are then NST - 1 groups of loads
    // and the stores of the NST - 1 blocks before it (fewer at the start; those of strips that are not whole are not counted on).
    // (Issued between a block's last read and its stores instead, they give the stores the time of one more block to drain, but hold
    // them up: 16384 x 320 -> 960 through the 8-bit MFMA 14.3 us, 13.2 us as it is.)
    int stage = 0, to = NST - 1, done = 0;
    for (; blk < nblocks; blk += step) {
        issue(blk + step * (NST - 1), to);
        constexpr int ALL = (NST - 1) * (LOADS + STORES);
        if (whole_strip && done >= NST - 1)
            __builtin_amdgcn_s_waitcnt(vmcnt_imm(ALL < 63 ? ALL : 63));
        else
            __builtin_amdgcn_s_waitcnt(vmcnt_imm((NST - 1) * LOADS));
        asm volatile("" ::: "memory");
        compute(stage);
        epilogue(32 * blk);
        ++done;
        to = stage;
        stage = stage + 1 == NST ? 0 : stage + 1;
    }
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));                 // no load may land in LDS after the workgroup has gone
}

// Workgroups per strip.  Two workgroups fit on a compute unit; one takes the time of its blocks per wavefront and about one and a half
// more for the weights.
static inline int strip_chunks(int64_t M, int64_t N)
{
    const int64_t groups = (M + 127) / 128, strips = (N + 63) / 64;
    int64_t best = 1;
    double least = 1e30;
    for (int rounds = 1; rounds <= 4; ++rounds) {
        int64_t chunks = 512 * rounds / strips;
        if (chunks < 1) chunks = 1;
        const int64_t per = (groups + chunks - 1) / chunks;
        chunks = (groups + per - 1) / per;
        const double cost = (double)((chunks * strips + 511) / 512) * ((double)per + 1.5);
        if (cost < least) { least = cost; best = chunks; }
    }
    return (int)best;
}

template <int NK64, int XKIND, int WKIND, int ACC, int OUT>
static int launch_strip_one(const GemmArgs& a, hipStream_t st)
{
    constexpr int smem = strip_lds_bytes(NK64);
    auto kern = gemm_strip_kernel<NK64, XKIND, WKIND, ACC, OUT>;
    if (smem > 64 * 1024) {
        static std::atomic<uint64_t> allowed{0};   // per instantiation
        if (!allow_dynamic_lds(reinterpret_cast<const void*>(kern), smem, allowed)) return FPQ_ERR_LAUNCH;
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)(strip_chunks(a.M, a.N) * ((a.N + 63) / 64))), dim3(256), smem, st, a);
    return hipGetLastError() == hipSuccess ? FPQ_OK : FPQ_ERR_LAUNCH;
}

template <int XKIND, int WKIND, int ACC, int OUT>
static int launch_strip_k(const GemmArgs& a, hipStream_t st)
{
    switch ((a.Kreal + 63) / 64) {
        case 1: return launch_strip_one<1, XKIND, WKIND, ACC, OUT>(a, st);
        case 2: return launch_strip_one<2, XKIND, WKIND, ACC, OUT>(a, st);
        case 3: return launch_strip_one<3, XKIND, WKIND, ACC, OUT>(a, st);
        case 4: return launch_strip_one<4, XKIND, WKIND, ACC, OUT>(a, st);
        case 5: return launch_strip_one<5, XKIND, WKIND, ACC, OUT>(a, st);
        default: return FPQ_ERR_UNSUPPORTED;
    }
}

}  // namespace fpq
