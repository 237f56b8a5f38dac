// The same-bitwidth integer baseline the paper compares against (Section IV-A, Eq. (4)): uniform quantizer with scale
// s = (max - min) / (2^b - 1) and zero point z = -round(min / s), and a linear layer on its codes with the 8-bit integer
// matrix instruction of gfx950 (v_mfma_i32_32x32x32_i8, exact 32-bit sums).
//
// The matrix instruction multiplies signed bytes, the codes are unsigned (0 .. 2^b - 1) with a zero point, so the
// operands are offset: activations enter as a' = q - 128, 8-bit weights as b' = q - 128 (stored that way when packed),
// 4-bit weights as b' = q (0 .. 15 fits a signed byte).  With za = zx - 128 and zb = zw - 128 (or zw):
//   sum_k (qx - zx)(qw - zw) = sum_k a' b'  -  zb * sum_k a'  -  za * sum_k b'  +  K * za * zb,
// all in 32-bit integers (K <= 32768 keeps the result below 2^31; intermediate wrap-around cancels).  The row sums of b'
// are computed when the weights are packed, those of a' by the layer kernel on its way through the codes.
#include "fpq_dev.h"
#include "fpq_host.h"
#include "gemm_dma_kernel.h"

namespace fpq {

typedef v4i v4i32;
typedef int v16i32 __attribute__((ext_vector_type(16)));

// ---------------------------------------------------------------------------------- min / max -> (s, z)

__device__ __forceinline__ void block_minmax(float& lo, float& hi)
{
    __shared__ float plo[4], phi[4];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        lo = fminf(lo, __shfl_xor(lo, off, 64));
        hi = fmaxf(hi, __shfl_xor(hi, off, 64));
    }
    if ((threadIdx.x & 63) == 0) { plo[threadIdx.x >> 6] = lo; phi[threadIdx.x >> 6] = hi; }
    __syncthreads();
    lo = fminf(fminf(plo[0], plo[1]), fminf(plo[2], plo[3]));
    hi = fmaxf(fmaxf(phi[0], phi[1]), fmaxf(phi[2], phi[3]));
    __syncthreads();
}

// Eq. (4): s = fl32(fl32(max - min) / (2^b - 1)) (1 for a constant tensor), z = -round(fl32(min * fl32(1 / s))).
__device__ __forceinline__ void int_params_of(float lo, float hi, int levels, float& s, int& z)
{
    const float rng = __fsub_rn(hi, lo);
    s = (rng == 0.0f) ? 1.0f : __fdiv_rn(rng, (float)levels);
    const float r = __fdiv_rn(1.0f, s);
    z = -(int)rintf(__fmul_rn(lo, r));
}

__global__ __launch_bounds__(256) void int_minmax_partial_kernel(const float* __restrict__ x, size_t n, float* __restrict__ partial)
{
    float lo = INFINITY, hi = -INFINITY;
    const size_t nthreads = (size_t)gridDim.x * 256, tid = (size_t)blockIdx.x * 256 + threadIdx.x;
    auto take = [&](float v) {
        lo = fminf(lo, v);
        hi = fmaxf(hi, v);
    };
    auto take4 = [&](const float4& v) { take(v.x), take(v.y), take(v.z), take(v.w); };
    // 16 bytes per lane, four loads in flight; a start that is not 16-byte aligned leaves up to three elements to single loads
    size_t head = (16 - (reinterpret_cast<uintptr_t>(x) & 15)) / 4 & 3;
    if (head > n) head = n;
    const float4* x4 = reinterpret_cast<const float4*>(x + head);
    const size_t n4 = (n - head) >> 2;
    size_t i = tid;
    for (; i + 3 * nthreads < n4; i += 4 * nthreads) {
        const float4 a = x4[i], b = x4[i + nthreads], c = x4[i + 2 * nthreads], d = x4[i + 3 * nthreads];
        take4(a), take4(b), take4(c), take4(d);
    }
    for (; i < n4; i += nthreads) take4(x4[i]);
    if (tid < head) take(x[tid]);
    if (head + 4 * n4 + tid < n) take(x[head + 4 * n4 + tid]);
    block_minmax(lo, hi);
    if (threadIdx.x == 0) { partial[2 * blockIdx.x] = lo; partial[2 * blockIdx.x + 1] = hi; }
}

__global__ __launch_bounds__(256) void int_minmax_final_kernel(const float* __restrict__ partial, int nparts, int levels, int empty,
                                                               fpq_int_params* __restrict__ out)
{
    float lo = INFINITY, hi = -INFINITY;
    for (int i = threadIdx.x; i < nparts; i += 256) { lo = fminf(lo, partial[2 * i]); hi = fmaxf(hi, partial[2 * i + 1]); }
    block_minmax(lo, hi);
    if (threadIdx.x == 0) {
        if (empty) lo = hi = 0.0f;
        float s; int z;
        int_params_of(lo, hi, levels, s, z);
        out->scale = s;
        out->zero_point = z;
        out->min = lo;
        out->max = hi;
    }
}

static int int_minmax_parts(size_t n)
{
    size_t g = (n + 4095) / 4096;
    return (int)(g < 1 ? 1 : (g > 1024 ? 1024 : g));
}

int launch_int_params(const float* x, size_t n, int bits, fpq_int_params* out, float* partial, hipStream_t st)
{
    const int parts = int_minmax_parts(n);
    hipLaunchKernelGGL(int_minmax_partial_kernel, dim3(parts), dim3(256), 0, st, x, n, partial);
    hipLaunchKernelGGL(int_minmax_final_kernel, dim3(1), dim3(256), 0, st, partial, parts, (1 << bits) - 1, n == 0 ? 1 : 0, out);
    return hipGetLastError() == hipSuccess ? FPQ_OK : FPQ_ERR_LAUNCH;
}

// ---------------------------------------------------------------------------------- quantize

// q = clamp(round(fl32(x * r)) + z; 0, 2^b - 1), ties to even; NaN gives code 0.
__device__ __forceinline__ uint32_t int_code(float x, float r, int z, int qmax)
{
    const float y = rintf(__fmul_rn(x, r));
    // |y| can exceed the int range: clamp in float first (z is small against 2^30)
    const float yc = fminf(fmaxf(y, -1073741824.0f), 1073741824.0f);
    const long long q = (long long)(int)yc + (long long)z;
    return (uint32_t)(q < 0 ? 0 : (q > qmax ? qmax : q));
}

__global__ __launch_bounds__(256) void int_quantize_kernel(const float* __restrict__ x, size_t n, int qmax, float scale, int zp,
                                                           const fpq_int_params* __restrict__ params_dev,
                                                           uint8_t* __restrict__ codes)
{
    const float s = params_dev ? params_dev->scale : scale;
    const int z = params_dev ? params_dev->zero_point : zp;
    const float r = __fdiv_rn(1.0f, s);
    const size_t nthreads = (size_t)gridDim.x * 256;
    const size_t tid = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (((reinterpret_cast<uintptr_t>(x) & 15) | (reinterpret_cast<uintptr_t>(codes) & 3)) == 0) {
        const size_t n4 = n >> 2;
        for (size_t i = tid; i < n4; i += nthreads) {
            const float4 v = reinterpret_cast<const float4*>(x)[i];
            reinterpret_cast<uint32_t*>(codes)[i] = int_code(v.x, r, z, qmax) | (int_code(v.y, r, z, qmax) << 8) |
                                                   (int_code(v.z, r, z, qmax) << 16) | (int_code(v.w, r, z, qmax) << 24);
        }
        for (size_t j = (n4 << 2) + tid; j < n; j += nthreads) codes[j] = (uint8_t)int_code(x[j], r, z, qmax);
    } else {
        for (size_t j = tid; j < n; j += nthreads) codes[j] = (uint8_t)int_code(x[j], r, z, qmax);
    }
}

int launch_int_quantize(const float* x, size_t n, int bits, float scale, int zp, const fpq_int_params* params_dev, uint8_t* codes,
                        hipStream_t st)
{
    if (n == 0) return FPQ_OK;
    size_t g = (n / 4 + 1023) / 1024;
    g = g < 1 ? 1 : (g > 2048 ? 2048 : g);
    hipLaunchKernelGGL(int_quantize_kernel, dim3((unsigned)g), dim3(256), 0, st, x, n, (1 << bits) - 1, scale, zp, params_dev, codes);
    return hipGetLastError() == hipSuccess ? FPQ_OK : FPQ_ERR_LAUNCH;
}

// ---------------------------------------------------------------------------------- weights: per-channel (s, z), codes, row sums

// One block per output channel.  Packed row: Kpad bytes of b' = q - 128 (8-bit), or Kpad / 2 bytes holding b' = q as
// nibbles (4-bit), where byte j of every 4-byte word carries k = 8 w + j in its low and k = 8 w + 4 + j in its high nibble
// (w = the word's index), so that masking the low and the high nibbles of a word yields two words of four consecutive k.
// Padding (k >= K) is b' = 0: it adds nothing to the products nor to the row sum.
template <bool FOUR_BIT>
__global__ __launch_bounds__(256) void int_pack_weights_kernel(const float* __restrict__ w, int K, int Kpad, int bits,
                                                               uint8_t* __restrict__ rows, float* __restrict__ scale_out,
                                                               int32_t* __restrict__ zp_out, int32_t* __restrict__ rowsum_out,
                                                               uint8_t* __restrict__ codes_out)
{
    const int n = blockIdx.x;
    const float* row = w + (size_t)n * K;
    float lo = INFINITY, hi = -INFINITY;
    for (int i = threadIdx.x; i < K; i += 256) { lo = fminf(lo, row[i]); hi = fmaxf(hi, row[i]); }
    block_minmax(lo, hi);
    float s; int z;
    const int qmax = (1 << bits) - 1;
    int_params_of(lo, hi, qmax, s, z);
    if (threadIdx.x == 0) { scale_out[n] = s; zp_out[n] = z; }
    const float r = __fdiv_rn(1.0f, s);
    int sum = 0;
    if (FOUR_BIT) {
        uint32_t* dst = reinterpret_cast<uint32_t*>(rows + (size_t)n * (Kpad / 2));
        for (int wd = threadIdx.x; wd < Kpad / 8; wd += 256) {
            uint32_t word = 0;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int k = 8 * wd + j;
                uint32_t q = 0;
                if (k < K) {
                    q = int_code(row[k], r, z, qmax);
                    if (codes_out) codes_out[(size_t)n * K + k] = (uint8_t)q;
                    sum += (int)q;
                }
                word |= q << (j < 4 ? 8 * j : 8 * (j - 4) + 4);
            }
            dst[wd] = word;
        }
    } else {
        uint32_t* dst = reinterpret_cast<uint32_t*>(rows + (size_t)n * Kpad);
        for (int wd = threadIdx.x; wd < Kpad / 4; wd += 256) {
            uint32_t word = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int k = 4 * wd + j;
                if (k < K) {
                    const uint32_t q = int_code(row[k], r, z, qmax);
                    if (codes_out) codes_out[(size_t)n * K + k] = (uint8_t)q;
                    sum += (int)q - 128;
                    word |= (q ^ 0x80u) << (8 * j);
                }
            }
            dst[wd] = word;
        }
    }
    __shared__ int part[4];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off, 64);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = sum;
    __syncthreads();
    if (threadIdx.x == 0) rowsum_out[n] = part[0] + part[1] + part[2] + part[3];
}

int launch_int_pack_weights(const float* w, int64_t N, int64_t K, int bits, uint8_t* rows, float* scale_out, int32_t* zp_out,
                            int32_t* rowsum_out, uint8_t* codes_out, hipStream_t st)
{
    const int Kpad = (int)padded_k(K, 1);
    if (bits == 4)
        hipLaunchKernelGGL(int_pack_weights_kernel<true>, dim3((unsigned)N), dim3(256), 0, st, w, (int)K, Kpad, bits, rows, scale_out,
                           zp_out, rowsum_out, codes_out);
    else
        hipLaunchKernelGGL(int_pack_weights_kernel<false>, dim3((unsigned)N), dim3(256), 0, st, w, (int)K, Kpad, bits, rows, scale_out,
                           zp_out, rowsum_out, codes_out);
    return hipGetLastError() == hipSuccess ? FPQ_OK : FPQ_ERR_LAUNCH;
}

// ---------------------------------------------------------------------------------- the layer

struct IGemmArgs {
    const uint8_t* x;        // activation codes [M, K], K % 16 == 0
    const uint8_t* wrows;    // packed weight rows
    const int32_t* wsum;     // [N] row sums of b'
    const float* sw;         // [N]
    const int32_t* zw;       // [N]
    const float* bias;       // [N] or null
    const fpq_int_params* px_dev;   // activation scale / zero point on the device, or null
    float sx;
    int zx;
    float* y;
    int M, N, K, Kpad;
};

// A workgroup of four wavefronts (2 x 2) owns a BX x BW tile and walks K in steps of 128 codes through NST LDS stages that buffer loads
// fill without registers (dma16; codes beyond the rows or K arrive as 0).  A step's loads go out NST - 1 steps ahead, behind the
// barrier that frees its stage, and there is one barrier per step; two to five workgroups share a compute unit, so that one
// stores while another multiplies.  Activations are the row operand (accumulator registers run along m), weights the lane operand, so a
// half-wave stores 128 consecutive bytes of an output row.
// The row sums of the activation codes, which the zero points need, are taken from the fragments as they pass (one dot4 per four
// codes, in the shadow of the matrix instructions) instead of by a kernel of their own.
// No unit is busy throughout (2048 x 1280 -> 10240, counters: matrix unit 0.31 of the cycles, vector instructions 0.43, LDS 0.17; wavefronts
// wait for 0.35 of theirs): the two workgroups of a compute unit meet at a barrier per step, and 84 MB of results leave in 43 us.  Staged
// through registers, with single workgroups walking along the columns, 77 us; 41 us (35 us with 4-bit weights).
template <int BX, int BW, int NST, bool W4>
__global__ __launch_bounds__(256, 2) void igemm_kernel(const IGemmArgs a)
{
    constexpr int XROWB = 128, WROWB = W4 ? 64 : 128;
    constexpr int XTILE = BX * XROWB, WTILE = BW * WROWB, STAGE = XTILE + WTILE;
    constexpr int XLD = XTILE / 4096, WLD = WTILE / 4096, LOADS = XLD + WLD;     // loads per wavefront and step
    constexpr int TP = BX / 2, TQ = BW / 2, MI = TP / 32, NI = TQ / 32;
    static_assert(XTILE % 4096 == 0 && WTILE % 4096 == 0, "a tile splits evenly over the wavefronts' loads");
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    const int lane = threadIdx.x & 63, l32 = lane & 31, g = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int tiles_w = (a.N + BW - 1) / BW;
    // ids go round-robin over the 8 XCDs: each takes a contiguous run of tiles, which share activation rows
    int tile = blockIdx.x;
    {
        const int per = gridDim.x >> 3;
        if (tile < (per << 3)) tile = (tile & 7) * per + (tile >> 3);
    }
    // bands of eight tile rows, rows innermost: the workgroups that run together on an XCD then share weights as well as activations
    // (columns innermost, each of 64 workgroups would fetch weights of its own)
    const int tiles_x = (a.M + BX - 1) / BX;
    const int band = tile / (8 * tiles_w), rows = tiles_x - 8 * band < 8 ? tiles_x - 8 * band : 8;
    const int at = tile - band * 8 * tiles_w;
    const int tw = at / rows, tx = 8 * band + at - tw * rows;
    const int m0 = tx * BX, n0 = tw * BW;

    // buffers of this tile's rows alone: rows beyond M or N are beyond the buffer
    const unsigned wrow_bytes = W4 ? (unsigned)a.Kpad / 2 : (unsigned)a.Kpad;
    const v4i xrsrc = make_rsrc(a.x + (size_t)m0 * a.K, (unsigned)(a.M - m0 < BX ? a.M - m0 : BX) * (unsigned)a.K);
    const v4i wrsrc = make_rsrc(a.wrows + (size_t)n0 * wrow_bytes, (unsigned)(a.N - n0 < BW ? a.N - n0 : BW) * wrow_bytes);
    const unsigned lds0 = (unsigned)(size_t)((__attribute__((address_space(3))) void*)smem);
    constexpr unsigned OOB = 0x80000000u;
    // load i covers rows 8 (4 i + wave) .. + 7 of 128 bytes (weights of 64 bytes: 16 rows); the swizzle of lds_off is applied by
    // choosing the chunk that a lane fetches
    const int xc = (lane & 7) ^ ((wave * 4 + (lane >> 4)) & 7);
    unsigned xoff[XLD], woff[WLD];
#pragma unroll
    for (int i = 0; i < XLD; ++i) xoff[i] = (unsigned)((4 * i + wave) * 8 + (lane >> 3)) * (unsigned)a.K + 16u * xc;
#pragma unroll
    for (int i = 0; i < WLD; ++i)
        woff[i] = W4 ? (unsigned)((4 * i + wave) * 16 + (lane >> 2)) * wrow_bytes + 16u * ((lane & 3) ^ ((lane >> 4) & 3))
                     : (unsigned)((4 * i + wave) * 8 + (lane >> 3)) * wrow_bytes + 16u * xc;
    const int nk = a.Kpad / 128;
    auto issue = [&](int kt, int stage) {
        const int live = kt < nk ? -1 : 1;                    // beyond the last step one lane keeps the counts of the waits
        const bool in_row = kt * 128 + xc * 16 < a.K;
#pragma unroll
        for (int i = 0; i < XLD; ++i)
            dma16_live(xrsrc, in_row ? xoff[i] + kt * 128 : OOB, lds0 + stage * STAGE + (4 * i + wave) * 1024, live);
#pragma unroll
        for (int i = 0; i < WLD; ++i)
            dma16_live(wrsrc, kt < nk ? woff[i] + kt * WROWB : OOB, lds0 + stage * STAGE + XTILE + (4 * i + wave) * 1024, live);
    };
#pragma unroll
    for (int s = 0; s < NST - 1; ++s) issue(s, s);

    v16i32 acc[MI][NI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0;
    unsigned xs[MI];                                          // sums of the codes this lane has read of row l32 of block i
#pragma unroll
    for (int i = 0; i < MI; ++i) xs[i] = 0;
    const int wp = wave >> 1, wq = wave & 1;
    const int prow0 = wp * TP + l32, qrow0 = wq * TQ + l32;

    int stage = 0, to = NST - 1;
    for (int kt = 0; kt < nk; ++kt) {
        // this step's loads have landed (younger: those of the NST - 2 steps after it); behind the barrier that holds for all
        // wavefronts, and all have read the stage of the step before, which the loads issued next overwrite
        __builtin_amdgcn_s_waitcnt(vmcnt_imm((NST - 2) * LOADS));
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        issue(kt + NST - 1, to);
        const uint8_t* xt = smem + stage * STAGE;
        const uint8_t* wt = xt + XTILE;
        // four chunks of 32 codes; lane half g takes 16 codes of a chunk, the same ones of both operands
        v4i32 af[2][MI], bf[2][NI];
        auto read = [&](int c) {
#pragma unroll
            for (int i = 0; i < MI; ++i) {
                // two chunks of 4-bit weights are one 16-byte piece: their halves are 32 codes apart
                const int k = W4 ? 4 * (c >> 1) + 2 * g + (c & 1) : 2 * c + g;
                const uint4 v = *reinterpret_cast<const uint4*>(xt + lds_off<XROWB>(prow0 + 32 * i, k));
                af[c & 1][i] = v4i32{(int)v.x, (int)v.y, (int)v.z, (int)v.w};
            }
#pragma unroll
            for (int j = 0; j < NI; ++j) {
                const int row = qrow0 + 32 * j;
                if (W4) {
                    // 16 codes = 8 bytes = two words: low nibbles, then high nibbles of each
                    const uint2 v = *reinterpret_cast<const uint2*>(wt + lds_off<WROWB>(row, 2 * (c >> 1) + g) + 8 * (c & 1));
                    bf[c & 1][j] = v4i32{(int)(v.x & 0x0f0f0f0fu), (int)((v.x >> 4) & 0x0f0f0f0fu), (int)(v.y & 0x0f0f0f0fu),
                                         (int)((v.y >> 4) & 0x0f0f0f0fu)};
                } else {
                    const uint4 v = *reinterpret_cast<const uint4*>(wt + lds_off<WROWB>(row, 2 * c + g));
                    bf[c & 1][j] = v4i32{(int)v.x, (int)v.y, (int)v.z, (int)v.w};
                }
            }
        };
        read(0);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            if (c + 1 < 4) read(c + 1);
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    const unsigned q = (unsigned)af[c & 1][i][w];
                    xs[i] = __builtin_amdgcn_udot4(q, 0x01010101u, xs[i], false);
                    af[c & 1][i][w] = (int)(q ^ 0x80808080u);  // unsigned code -> signed a' = q - 128
                }
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int j = 0; j < NI; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(af[c & 1][i], bf[c & 1][j], acc[i][j], 0, 0, 0);
        }
        to = stage;
        stage = stage + 1 == NST ? 0 : stage + 1;
    }
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));                 // no load may land in LDS from here on
    asm volatile("" ::: "memory");
    __syncthreads();

    // ---- epilogue: fold the zero points out with the row sums, scale, store.  The row sums cross from lanes to registers in LDS.
    unsigned* sums = reinterpret_cast<unsigned*>(smem) + wave * TP;
#pragma unroll
    for (int i = 0; i < MI; ++i) {
        const unsigned both = xs[i] + (unsigned)__shfl_xor((int)xs[i], 32, 64);
        if (g == 0) sums[32 * i + l32] = both - 128u * (unsigned)a.K;          // sum of a'
    }
    __syncthreads();
    const float sx = a.px_dev ? a.px_dev->scale : a.sx;
    const int za = (a.px_dev ? a.px_dev->zero_point : a.zx) - 128;
    float sc[NI], bv[NI];
    unsigned zb[NI], colterm[NI];
#pragma unroll
    for (int j = 0; j < NI; ++j) {
        const int n = n0 + wq * TQ + 32 * j + l32;
        const bool in = n < a.N;
        zb[j] = in ? (unsigned)(a.zw[n] - (W4 ? 0 : 128)) : 0u;
        colterm[j] = in ? (unsigned)a.K * (unsigned)za * zb[j] - (unsigned)za * (unsigned)a.wsum[n] : 0u;
        sc[j] = in ? sx * a.sw[n] : 0.0f;
        bv[j] = in && a.bias ? a.bias[n] : 0.0f;
    }
    const int mw = m0 + wp * TP, nw = n0 + wq * TQ;
    auto store_all = [&](auto whole, auto streaming) {
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint4 s4 = *reinterpret_cast<const uint4*>(sums + 32 * i + 8 * q + 4 * g);
                const unsigned s[4] = {s4.x, s4.y, s4.z, s4.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int m = mw + 32 * i + 8 * q + 4 * g + e;
#pragma unroll
                    for (int j = 0; j < NI; ++j) {
                        // unsigned arithmetic: intermediate values may wrap, the result fits (K <= 32768)
                        const int total = (int)((unsigned)acc[i][j][4 * q + e] - zb[j] * s[e] + colterm[j]);
                        const float v = (float)total * sc[j] + bv[j];
                        float* at = a.y + (size_t)m * a.N + nw + 32 * j + l32;
                        if constexpr (decltype(streaming)::value)
                            store_out(at, v);
                        else if (decltype(whole)::value || (m < a.M && nw + 32 * j + l32 < a.N))
                            *at = v;
                    }
                }
            }
    };
    // streaming stores where rows are whole cache lines; lines shared by two rows are put together in the L2
    const bool whole_tile = m0 + BX <= a.M && n0 + BW <= a.N;
    if (whole_tile && (a.N & 31) == 0)
        store_all(std::true_type{}, std::true_type{});
    else if (whole_tile)
        store_all(std::true_type{}, std::false_type{});
    else
        store_all(std::false_type{}, std::false_type{});
}

template <int BX, int BW, int NST, bool W4>
static int launch_igemm_one(const IGemmArgs& a, hipStream_t st)
{
    constexpr int smem = NST * (BX * 128 + BW * (W4 ? 64 : 128));
    const int64_t tiles = (int64_t)((a.M + BX - 1) / BX) * ((a.N + BW - 1) / BW);
    auto kern = igemm_kernel<BX, BW, NST, W4>;
    if (smem > 64 * 1024) {
        static std::atomic<uint64_t> allowed{0};
        if (!allow_dynamic_lds(reinterpret_cast<const void*>(kern), smem, allowed)) return FPQ_ERR_LAUNCH;
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)tiles), dim3(256), smem, st, a);
    return hipGetLastError() == hipSuccess ? FPQ_OK : FPQ_ERR_LAUNCH;
}

int launch_int_gemm(const uint8_t* x, float sx, int zx, const fpq_int_params* px_dev, const uint8_t* wrows, const int32_t* wsum,
                    int wbits, const float* sw, const int32_t* zw, const float* bias, float* y, int64_t M, int64_t N, int64_t K,
                    hipStream_t st)
{
    if (M <= 0 || N <= 0) return FPQ_OK;
    IGemmArgs a{x, wrows, wsum, sw, zw, bias, px_dev, sx, zx, y, (int)M, (int)N, (int)K, (int)padded_k(K, 1)};
    switch (int_tile(M, N, K, a.Kpad, wbits)) {
    case INT_128x128: return wbits == 4 ? launch_igemm_one<128, 128, 2, true>(a, st) : launch_igemm_one<128, 128, 2, false>(a, st);
    case INT_64x128: return wbits == 4 ? launch_igemm_one<64, 128, 2, true>(a, st) : launch_igemm_one<64, 128, 2, false>(a, st);
    case INT_64x64_S3: return wbits == 4 ? launch_igemm_one<64, 64, 3, true>(a, st) : launch_igemm_one<64, 64, 3, false>(a, st);
    default: return wbits == 4 ? launch_igemm_one<64, 64, 2, true>(a, st) : launch_igemm_one<64, 64, 2, false>(a, st);
    }
}

}  // namespace fpq
