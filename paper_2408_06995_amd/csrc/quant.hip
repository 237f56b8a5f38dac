// Streaming kernels of libfpq: absmax calibration, the activation quantizer (flat and
// NCHW -> channels-last), dequantize, and the offline weight quantizer / packer.
// All are HBM-bound: 16-byte coalesced loads, the ExMy encode in registers, packed stores.
#include "fpq_dev.h"
#include "fpq_host.h"

namespace fpq {

// ------------------------------------------------------------------------------ absmax

__device__ __forceinline__ float wave_max(float v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = fmaxf(v, __shfl_xor(v, off, 64));
    return v;
}

__device__ __forceinline__ float block_max(float v)
{
    __shared__ float part[4];
    v = wave_max(v);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = v;
    __syncthreads();
    v = fmaxf(fmaxf(part[0], part[1]), fmaxf(part[2], part[3]));
    __syncthreads();
    return v;
}

// r = fl32(1 / scale) for a quantize kernel, in two halves (all threads of the block call both): the partial maxima go out first, the
// caller's own first loads right behind them, and the wait for the partials, the barriers and the division then run while those are
// on their way.  (One after the other, a block spent half of its life on the fold: its loads, four in a row, and nothing else.)
// Loads ahead of fold_end are not conditional (an index beyond the end becomes the last one): behind a branch, the compiler's wait for
// the partials would be one for all loads.
struct Fold {
    float part[kAbsmaxParts / 256];
};
__device__ __forceinline__ Fold fold_begin(const ScaleSrc& s)
{
    Fold f;
#pragma unroll
    for (int u = 0; u < kAbsmaxParts / 256; ++u) {
        f.part[u] = s.partials != nullptr ? s.partials[min((int)threadIdx.x + 256 * u, s.nparts - 1)] : 0.0f;
    }
    return f;
}
__device__ __forceinline__ float fold_end(const ScaleSrc& s, const Fold& f)
{
    if (s.partials == nullptr) return inv_scale(s.host, s.dev);
    float v = f.part[0];
#pragma unroll
    for (int u = 1; u < kAbsmaxParts / 256; ++u) v = fmaxf(v, f.part[u]);
    v = block_max(v);
    const float sc = (v == 0.0f) ? 1.0f : __fdiv_rn(v, s.maxval);
    if (s.publish && blockIdx.x == 0 && blockIdx.y == 0 && blockIdx.z == 0 && threadIdx.x == 0) {
        s.publish[0] = sc;
        s.publish[1] = v;
    }
    return __fdiv_rn(1.0f, sc);
}

// Four codes in one word, byte e = value e.  The formats that the hardware converts (YKIND 1: (4, 3, 7), 2: (5, 2, 15), see hw_kind)
// take one conversion per pair after the clip, the same rounding on the same grid, signs of zeros included: 14 vector instructions
// for four values against about 60 of the arithmetic encoder, which at 10 M elements take as long as half of the reads.
template <int YKIND>
__device__ __forceinline__ uint32_t quantize4(float v0, float v1, float v2, float v3, float r, const QParams& q)
{
    if constexpr (YKIND == 0) {
        return quantize_nearest(v0, r, q) | (quantize_nearest(v1, r, q) << 8) | (quantize_nearest(v2, r, q) << 16) |
               (quantize_nearest(v3, r, q) << 24);
    } else {
        auto clip = [&](float x) {
            const float y = __fmul_rn(x, r);
            return copysignf(fminf(fabsf(y), q.c), y);
        };
        int w;
        if constexpr (YKIND == 1) {
            w = __builtin_amdgcn_cvt_pk_fp8_f32(clip(v0), clip(v1), 0, false);
            w = __builtin_amdgcn_cvt_pk_fp8_f32(clip(v2), clip(v3), w, true);
        } else {
            w = __builtin_amdgcn_cvt_pk_bf8_f32(clip(v0), clip(v1), 0, false);
            w = __builtin_amdgcn_cvt_pk_bf8_f32(clip(v2), clip(v3), w, true);
        }
        return (uint32_t)w;
    }
}

// The format's conversion instruction, if there is one (any max value up to the hardware's own: the clip comes first).
int hw_kind(const QParams& q)
{
    if (q.em == 7 && q.m == 3 && q.b == 7 && q.c <= 448.0f) return 1;
    if (q.em == 7 && q.m == 2 && q.b == 15 && q.c <= 57344.0f) return 2;
    return 0;
}

// Tensors from this many elements (64 MB of fp32) on take the contiguous-share / streaming-load kernels.
constexpr size_t kStreamElems = (size_t)16 << 20;
// ... and the flat quantizer with a given scale from here on, where a tensor no longer fits the 32 MB of L2 (10 M elements: E4M3 8.9 us
// grid-strided, 7.6 us in shares, E2M1 9.3 and 7.8 us; 8 M: 5.7 us both, E2M1 5.4 and 5.9 us).
constexpr size_t kStreamElemsGiven = (size_t)9 << 20;

typedef float v4f __attribute__((ext_vector_type(4)));

// Streaming 16-byte load for the last reader of the activations (the quantize kernels): ~10 % more
// bandwidth than a plain load, and the codes just written are not displaced from the caches.  The absmax
// pass uses plain loads, so that what fits the last-level cache is still there for the quantize pass.
__device__ __forceinline__ float4 load_stream(const float4* p)
{
    const v4f v = __builtin_nontemporal_load(reinterpret_cast<const v4f*>(p));
    return make_float4(v.x, v.y, v.z, v.w);
}

__device__ __forceinline__ float max4(float v, const float4& a)
{
    return fmaxf(v, fmaxf(fmaxf(fabsf(a.x), fabsf(a.y)), fmaxf(fabsf(a.z), fabsf(a.w))));
}

// Pass 1: each block folds one contiguous share of x into one partial maximum of |x| (contiguous shares
// and eight 16-byte loads in flight per lane measured fastest: ~6.6 TB/s against ~5.3 grid-strided; 168 MB 35.4 us, 38.7 us with
// loads behind conditions).
__global__ __launch_bounds__(256) void absmax_partial_kernel(const float* __restrict__ x, size_t n,
                                                             float* __restrict__ partial)
{
    float v = 0.0f;
    if ((reinterpret_cast<uintptr_t>(x) & 15) == 0) {
        const float4* x4 = reinterpret_cast<const float4*>(x);
        const size_t n4 = n >> 2;
        const size_t per = (n4 + gridDim.x - 1) / gridDim.x;
        const size_t b0 = (size_t)blockIdx.x * per;
        const size_t e = b0 + per < n4 ? b0 + per : n4;
        // eight loads in flight per lane whatever the length of the share (beyond its end the last element again: a load behind a
        // condition would be waited for before the next); plain loads: the quantize pass that follows re-reads x
        for (size_t base = b0 + threadIdx.x; base < e; base += 8 * 256) {
            float4 a[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) a[u] = x4[base + u * 256 < e ? base + u * 256 : e - 1];
#pragma unroll
            for (int u = 0; u < 8; ++u) v = max4(v, a[u]);
        }
        const size_t tid = (size_t)blockIdx.x * 256 + threadIdx.x;
        for (size_t j = (n4 << 2) + tid; j < n; j += (size_t)gridDim.x * 256) v = fmaxf(v, fabsf(x[j]));
    } else {
        const size_t tid = (size_t)blockIdx.x * 256 + threadIdx.x;
        for (size_t j = tid; j < n; j += (size_t)gridDim.x * 256) v = fmaxf(v, fabsf(x[j]));
    }
    v = block_max(v);
    if (threadIdx.x == 0) partial[blockIdx.x] = v;
}

// Pass 1 for tensors below kStreamElems: each block folds a grid-strided share of x (measured ~1 us
// faster per call than the contiguous-share kernel on the small and cache-resident tensors).
__global__ __launch_bounds__(256) void absmax_partial_strided_kernel(const float* __restrict__ x, size_t n,
                                                             float* __restrict__ partial)
{
    float v = 0.0f;
    const size_t tid = (size_t)blockIdx.x * 256 + threadIdx.x;
    const size_t nthreads = (size_t)gridDim.x * 256;
    if ((reinterpret_cast<uintptr_t>(x) & 15) == 0) {
        const float4* x4 = reinterpret_cast<const float4*>(x);
        const size_t n4 = n >> 2;
        size_t i = tid;
        for (; i + 3 * nthreads < n4; i += 4 * nthreads) {
            float4 a = x4[i], b = x4[i + nthreads], c = x4[i + 2 * nthreads], d = x4[i + 3 * nthreads];
            v = fmaxf(v, fmaxf(fmaxf(fabsf(a.x), fabsf(a.y)), fmaxf(fabsf(a.z), fabsf(a.w))));
            v = fmaxf(v, fmaxf(fmaxf(fabsf(b.x), fabsf(b.y)), fmaxf(fabsf(b.z), fabsf(b.w))));
            v = fmaxf(v, fmaxf(fmaxf(fabsf(c.x), fabsf(c.y)), fmaxf(fabsf(c.z), fabsf(c.w))));
            v = fmaxf(v, fmaxf(fmaxf(fabsf(d.x), fabsf(d.y)), fmaxf(fabsf(d.z), fabsf(d.w))));
        }
        for (; i < n4; i += nthreads) {
            float4 a = x4[i];
            v = fmaxf(v, fmaxf(fmaxf(fabsf(a.x), fabsf(a.y)), fmaxf(fabsf(a.z), fabsf(a.w))));
        }
        for (size_t j = (n4 << 2) + tid; j < n; j += nthreads) v = fmaxf(v, fabsf(x[j]));
    } else {
        for (size_t j = tid; j < n; j += nthreads) v = fmaxf(v, fabsf(x[j]));
    }
    v = block_max(v);
    if (threadIdx.x == 0) partial[blockIdx.x] = v;
}

// Pass 2: one block folds the partials and writes absmax and scale = absmax / maxval.
__global__ __launch_bounds__(256) void absmax_final_kernel(const float* __restrict__ partial, int nparts,
                                                           float maxval, float* __restrict__ absmax_out,
                                                           float* __restrict__ scale_out)
{
    float v = 0.0f;
    for (int i = threadIdx.x; i < nparts; i += 256) v = fmaxf(v, partial[i]);
    v = block_max(v);
    if (threadIdx.x == 0) {
        absmax_out[0] = v;
        if (scale_out) scale_out[0] = (v == 0.0f) ? 1.0f : __fdiv_rn(v, maxval);
    }
}

int launch_absmax_partials(const float* x, size_t n, float* partial, hipStream_t st);

int launch_absmax(const float* x, size_t n, float maxval, float* absmax_out, float* scale_out,
                  float* partial, hipStream_t st)
{
    int nparts = absmax_parts(n);
    launch_absmax_partials(x, n, partial, st);
    hipLaunchKernelGGL(absmax_final_kernel, dim3(1), dim3(256), 0, st, partial, nparts, maxval, absmax_out,
                       scale_out);
    return hipGetLastError() == hipSuccess ? FPQ_OK : FPQ_ERR_LAUNCH;
}

// Pass 1 alone, for the dynamic-scale path of the layer entry points (the quantize kernel folds the partials).
int launch_absmax_partials(const float* x, size_t n, float* partial, hipStream_t st)
{
    const int nparts = absmax_parts(n);
    if (nparts > 0) {
        if (n >= kStreamElems)
            hipLaunchKernelGGL(absmax_partial_kernel, dim3(nparts), dim3(256), 0, st, x, n, partial);
        else
            hipLaunchKernelGGL(absmax_partial_strided_kernel, dim3(nparts), dim3(256), 0, st, x, n, partial);
    }
    return hipGetLastError() == hipSuccess ? FPQ_OK : FPQ_ERR_LAUNCH;
}

// ------------------------------------------------------------------------------ quantize (flat)

template <bool FOUR_BIT, int YKIND>
__device__ __forceinline__ void store_codes(uint8_t* codes, size_t i, const float4& v, float r, const QParams& q)
{
    if (FOUR_BIT) {
        reinterpret_cast<uint16_t*>(codes)[i] = (uint16_t)(quantize_nearest(v.x, r, q) | (quantize_nearest(v.y, r, q) << 4) |
                                                           (quantize_nearest(v.z, r, q) << 8) | (quantize_nearest(v.w, r, q) << 12));
    } else {
        reinterpret_cast<uint32_t*>(codes)[i] = quantize4<YKIND>(v.x, v.y, v.z, v.w, r, q);
    }
}

// Four elements per lane and step: one 16-byte streaming load, four encodes, one 4-byte (8-bit codes) or
// 2-byte (4-bit codes) store.  Each block walks one contiguous share with four loads in flight per lane.
template <bool FOUR_BIT, int YKIND, bool FOLD>
__global__ __launch_bounds__(256) void quantize_vec_kernel(const float4* __restrict__ x4, size_t n4, QParams q,
                                                           ScaleSrc ss, uint8_t* __restrict__ codes)
{
    Fold f;
    if constexpr (FOLD) f = fold_begin(ss);
    const size_t per = (n4 + gridDim.x - 1) / gridDim.x;
    const size_t b0 = (size_t)blockIdx.x * per;
    const size_t e = b0 + per < n4 ? b0 + per : n4;
    size_t i = b0 + threadIdx.x;
    float4 a[4];
    auto load = [&]() {
#pragma unroll
        for (int u = 0; u < 4; ++u) a[u] = load_stream(x4 + (i + u * 256 < e ? i + u * 256 : e - 1));
    };
    load();
    const float r = FOLD ? fold_end(ss, f) : inv_scale(ss.host, ss.dev);
    while (i < e) {   // four loads in flight per lane
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (i + u * 256 < e) store_codes<FOUR_BIT, YKIND>(codes, i + u * 256, a[u], r, q);
        i += 4 * 256;
        if (i < e) load();
    }
}

// The same for smaller tensors, grid-strided with plain loads, one round of four loads per lane: the grid covers the tensor.
// 32768 x 320: 11.3 us with the fold in front of the loads and the arithmetic encoder, 7.9 us.
template <bool FOUR_BIT, int YKIND, bool FOLD>
__global__ __launch_bounds__(256) void quantize_vec_strided_kernel(const float4* __restrict__ x4, size_t n4, QParams q,
                                                           ScaleSrc ss, uint8_t* __restrict__ codes)
{
    Fold f;
    if constexpr (FOLD) f = fold_begin(ss);
    const size_t nthreads = (size_t)gridDim.x * 256;
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    float4 a[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) a[u] = x4[i + u * nthreads < n4 ? i + u * nthreads : n4 - 1];
    const float r = FOLD ? fold_end(ss, f) : inv_scale(ss.host, ss.dev);
#pragma unroll
    for (int u = 0; u < 4; ++u)
        if (i + u * nthreads < n4) store_codes<FOUR_BIT, YKIND>(codes, i + u * nthreads, a[u], r, q);
}

// One output byte per lane: any alignment, tails.  first = index of the first element handled.
template <bool FOUR_BIT>
__global__ __launch_bounds__(256) void quantize_scalar_kernel(const float* __restrict__ x, size_t first, size_t n,
                                                              QParams q, ScaleSrc ss,
                                                              uint8_t* __restrict__ codes)
{
    const float r = fold_end(ss, fold_begin(ss));
    const size_t per = FOUR_BIT ? 2 : 1;
    size_t j = first / per + (size_t)blockIdx.x * 256 + threadIdx.x;  // output byte
    const size_t nbytes = (n + per - 1) / per;
    const size_t nthreads = (size_t)gridDim.x * 256;
    for (; j < nbytes; j += nthreads) {
        if (FOUR_BIT) {
            uint32_t lo = quantize_nearest(x[2 * j], r, q);
            uint32_t hi = (2 * j + 1 < n) ? quantize_nearest(x[2 * j + 1], r, q) : 0u;
            codes[j] = (uint8_t)(lo | (hi << 4));
        } else {
            codes[j] = (uint8_t)quantize_nearest(x[j], r, q);
        }
    }
}

static int grid_for(size_t work_items, int per_block)
{
    size_t g = (work_items + per_block - 1) / per_block;
    if (g < 1) g = 1;
    if (g > 4096) g = 4096;
    return (int)g;
}

int launch_quantize(const float* x, size_t n, const QParams& q, bool four_bit, const ScaleSrc& ss, uint8_t* codes,
                    hipStream_t st)
{
    if (n == 0) return FPQ_OK;
    bool aligned = (reinterpret_cast<uintptr_t>(x) & 15) == 0 && (reinterpret_cast<uintptr_t>(codes) & 3) == 0;
    size_t n4 = aligned ? (n >> 2) : 0;
    if (n4) {
        static_assert(kStreamElems <= (size_t)4096 * 4 * 256 * 4, "the grid of the strided kernel covers what it is given");
        int g = grid_for(n4, 256 * 4);
        const float4* x4 = reinterpret_cast<const float4*>(x);
        // a given scale leaves nothing to fold, and its branches ahead of the first load cost formats without a conversion instruction 3 to
        // 8 % (E2M1, 5 M elements: 4.4 us, 3.9 us)
        const int kind = four_bit ? 4 : hw_kind(q);
        auto pick = [&](auto fold) {
            constexpr bool F = decltype(fold)::value;
            if (n >= (F ? kStreamElems : kStreamElemsGiven))
                return kind == 4   ? quantize_vec_kernel<true, 0, F>
                       : kind == 1 ? quantize_vec_kernel<false, 1, F>
                       : kind == 2 ? quantize_vec_kernel<false, 2, F> : quantize_vec_kernel<false, 0, F>;
            return kind == 4   ? quantize_vec_strided_kernel<true, 0, F>
                   : kind == 1 ? quantize_vec_strided_kernel<false, 1, F>
                   : kind == 2 ? quantize_vec_strided_kernel<false, 2, F> : quantize_vec_strided_kernel<false, 0, F>;
        };
        auto kern = ss.partials ? pick(std::true_type{}) : pick(std::false_type{});
        hipLaunchKernelGGL(kern, dim3(g), dim3(256), 0, st, x4, n4, q, ss, codes);
    }
    size_t first = n4 << 2;
    if (first < n) {
        int g = grid_for(n - first, 256);
        if (four_bit)
            hipLaunchKernelGGL(quantize_scalar_kernel<true>, dim3(g), dim3(256), 0, st, x, first, n, q, ss, codes);
        else
            hipLaunchKernelGGL(quantize_scalar_kernel<false>, dim3(g), dim3(256), 0, st, x, first, n, q, ss, codes);
    }
    return hipGetLastError() == hipSuccess ? FPQ_OK : FPQ_ERR_LAUNCH;
}

// Dynamic per-tensor scale of a tensor so small that one workgroup holds it in registers (up to 16 Ki elements: the
// time-embedding vectors of the U-Net): all loads in flight at once (sixteen 16-byte loads per lane at most), maximum
// of |x|, scale, and the codes from the registers, in one launch.  Bit-identical to the two-launch form.
__global__ __launch_bounds__(256) void quantize_dynamic_small_kernel(const float4* __restrict__ x4, int n4, QParams q,
                                                                     float maxval, float* __restrict__ publish,
                                                                     uint8_t* __restrict__ codes)
{
    float4 v[16];
    float m = 0.0f;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        const int i = e * 256 + threadIdx.x;
        v[e] = i < n4 ? x4[i] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        m = max4(m, v[e]);
    }
    m = block_max(m);
    const float sc = (m == 0.0f) ? 1.0f : __fdiv_rn(m, maxval);
    if (threadIdx.x == 0) {
        publish[0] = sc;
        publish[1] = m;
    }
    const float r = __fdiv_rn(1.0f, sc);
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        const int i = e * 256 + threadIdx.x;
        if (i < n4) {
            const uint32_t c0 = quantize_nearest(v[e].x, r, q), c1 = quantize_nearest(v[e].y, r, q);
            const uint32_t c2 = quantize_nearest(v[e].z, r, q), c3 = quantize_nearest(v[e].w, r, q);
            reinterpret_cast<uint32_t*>(codes)[i] = c0 | (c1 << 8) | (c2 << 16) | (c3 << 24);
        }
    }
}

// FPQ_OK when the one-launch form ran, FPQ_ERR_UNSUPPORTED when it does not apply (size, alignment).
int launch_quantize_dynamic_small(const float* x, size_t n, const QParams& q, float maxval, float* publish, uint8_t* codes,
                                  hipStream_t st)
{
    if (n == 0 || n > 16384 || (n & 3) || (reinterpret_cast<uintptr_t>(x) & 15) || (reinterpret_cast<uintptr_t>(codes) & 3))
        return FPQ_ERR_UNSUPPORTED;
    hipLaunchKernelGGL(quantize_dynamic_small_kernel, dim3(1), dim3(256), 0, st, reinterpret_cast<const float4*>(x),
                       (int)(n >> 2), q, maxval, publish, codes);
    return hipGetLastError() == hipSuccess ? FPQ_OK : FPQ_ERR_LAUNCH;
}

// ------------------------------------------------------------------- grouped dynamic-scale quantizer

// Dynamic per-tensor scales of a group of activation tensors in two launches for the whole group (blockIdx.y picks the
// problem): per-block partial maxima of |x|, then every block of the second kernel folds its problem's partials into
// scale = absmax / maxval (the same arithmetic as the single-tensor form, so the codes are the same bit for bit),
// block 0 of a problem publishes [scale, absmax] where the layer kernel reads its scale, and the elements are encoded.
// Each tensor has a multiple of 16 elements and is 16-byte aligned (rows of K % 16 == 0 codes).
__global__ __launch_bounds__(256) void absmax_grouped_kernel(const GroupedArgs g)
{
    const GroupedProblem& q = g.p[blockIdx.y];
    const float4* x4 = reinterpret_cast<const float4*>(q.x32);
    const int n4 = (q.M * q.K) >> 2;
    float v = 0.0f;
    constexpr int step = kGroupAbsmaxParts * 256;
    for (int i = blockIdx.x * 256 + threadIdx.x; i < n4; i += 8 * step) {      // eight loads in flight: 2 x 616 x 768 9.7 us, 4.9 us
        float4 a[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) a[u] = x4[min(i + u * step, n4 - 1)];
#pragma unroll
        for (int u = 0; u < 8; ++u) v = max4(v, a[u]);
    }
    v = block_max(v);
    if (threadIdx.x == 0) q.partials[blockIdx.x] = v;
}

template <int YKIND>
__global__ __launch_bounds__(256) void quantize_grouped_kernel(const GroupedArgs g, QParams qx, float maxval)
{
    const GroupedProblem& q = g.p[blockIdx.y];
    float v = threadIdx.x < kGroupAbsmaxParts ? q.partials[threadIdx.x] : 0.0f;
    const float4* x4 = reinterpret_cast<const float4*>(q.x32);
    uint32_t* codes = reinterpret_cast<uint32_t*>(const_cast<uint8_t*>(q.xcodes));
    const int n4 = (q.M * q.K) >> 2, step = gridDim.x * 256;
    int i = blockIdx.x * 256 + threadIdx.x;
    float4 a[4];
    auto load = [&]() {
#pragma unroll
        for (int u = 0; u < 4; ++u) a[u] = x4[min(i + u * step, n4 - 1)];
    };
    load();                                    // on their way while the maxima are folded
    v = block_max(v);
    const float sc = (v == 0.0f) ? 1.0f : __fdiv_rn(v, maxval);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        float* pub = const_cast<float*>(q.sx_dev);
        pub[0] = sc;
        pub[1] = v;
    }
    const float r = __fdiv_rn(1.0f, sc);
    while (i < n4) {
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (i + u * step < n4) codes[i + u * step] = quantize4<YKIND>(a[u].x, a[u].y, a[u].z, a[u].w, r, qx);
        i += 4 * step;
        if (i < n4) load();
    }
}

int launch_quantize_dynamic_grouped(const GroupedArgs& g, const QParams& qx, float maxval, hipStream_t st)
{
    if (g.count <= 0) return FPQ_OK;
    size_t most = 0;
    for (int i = 0; i < g.count; ++i) {
        const size_t n4 = ((size_t)g.p[i].M * g.p[i].K) >> 2;
        most = n4 > most ? n4 : most;
    }
    hipLaunchKernelGGL(absmax_grouped_kernel, dim3(kGroupAbsmaxParts, (unsigned)g.count), dim3(256), 0, st, g);
    size_t gx = (most + 1023) / 1024;          // four 16-byte loads per lane
    gx = gx < 1 ? 1 : (gx > 256 ? 256 : gx);
    const int kind = hw_kind(qx);
    auto kern = kind == 1 ? quantize_grouped_kernel<1> : kind == 2 ? quantize_grouped_kernel<2> : quantize_grouped_kernel<0>;
    hipLaunchKernelGGL(kern, dim3((unsigned)gx, (unsigned)g.count), dim3(256), 0, st, g, qx, maxval);
    return hipGetLastError() == hipSuccess ? FPQ_OK : FPQ_ERR_LAUNCH;
}

// ------------------------------------------------------------------- quantize NCHW -> NHWC codes

// 16 bytes from any 4-byte address (planes and rows of sizes that are no multiple of four elements).
typedef float v4f_any __attribute__((ext_vector_type(4), aligned(4)));
__device__ __forceinline__ float4 load_any(const float* p, bool stream)
{
    const v4f_any* at = reinterpret_cast<const v4f_any*>(p);
    const v4f_any v = stream ? __builtin_nontemporal_load(at) : *at;
    return make_float4(v.x, v.y, v.z, v.w);
}

// Keeps the first `left` codes of a word, the others become code 0 (whatever the scale).
__device__ __forceinline__ uint32_t first_codes(uint32_t w, int left)
{
    return left >= 4 ? w : left <= 0 ? 0u : w & ((1u << (8 * left)) - 1u);
}

// One block turns a patch of GROUPS x 4 channels x 1024 / GROUPS pixels of one image, or of 64 pixels of IMAGES images: reads run along
// pixels (contiguous in NCHW), the codes cross an LDS tile, writes run along channels (contiguous in [B,H,W,Cp]).
// A thread has four pixels of four channels, its four loads in flight together and ahead of the fold of the scale; the four codes
// of a pixel are one word.  Channels C..Cp-1 receive code 0.  Rows of the tile are GROUPS + 1 words, so that the words of a wavefront
// fall on different LDS banks (with 64 channels; on half and a quarter of them with 32 and 16).
// 8 x 320 x 64 x 64: 12.6 us with byte stores, loads behind the fold and the arithmetic encoder, 10.0 us; 3 x 200 x 75 x 53, whose
// planes are no multiple of 16 bytes: 9.9 us with single-element loads, 4.6 us.  Sixteen channel groups whatever C is cost images of few
// channels their time (8 x 3 x 256 x 256 11.5 us, in a format without a conversion instruction 19.1 us; with four groups 4.9 and 5.3 us).
template <int YKIND, int GROUPS, int IMAGES>
__global__ __launch_bounds__(256) void quantize_nhwc_kernel(const float* __restrict__ x, int B, int C, int Cp, int HW,
                                                            QParams q, ScaleSrc ss, bool stream,
                                                            uint8_t* __restrict__ codes)
{
    constexpr int QUADS = 256 / GROUPS, LDW = GROUPS + 1, PARTS = GROUPS / 4, OWN = 4 * QUADS / IMAGES;   // OWN: pixels of an image
    __shared__ uint32_t tile[4 * QUADS * LDW];
    const Fold f = fold_begin(ss);
    const int c0 = blockIdx.y * (4 * GROUPS), p0 = blockIdx.x * OWN;
    const int pq = threadIdx.x % QUADS, cg = threadIdx.x / QUADS;     // pixel quad, channel group
    const int ch = c0 + 4 * cg, p = p0 + 4 * pq % OWN, left = C - ch;
    const int img = 4 * pq / OWN;
    float4 v[4];                                                      // of channel ch + k
    // A quad that runs over the end of its plane goes on into the next; the last one of the tensor is read from four elements before
    // its end.  Narrow patches' groups without a channel read the tensor's first quad and encode nothing.
    const size_t last = (size_t)B * C * HW - 4;
    const bool some = GROUPS == 16 || left > 0;                       // (few patches of 64 channels have groups without any)
    auto at = [&](int b, int k) { return some ? ((size_t)b * C + min(ch + k, C - 1)) * HW + p : 0; };
    auto load = [&](int b) {
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = load_any(x + (at(b, k) < last ? at(b, k) : last), stream);
    };
    // images from b = IMAGES blockIdx.z, IMAGES (blockIdx.z + gridDim.z), ... on (the grid's third dimension stops at 65535)
    int b = IMAGES * blockIdx.z;
    load(b + img);
    const float r = fold_end(ss, f);
    for (;;) {
        if (p < HW && (IMAGES == 1 || b + img < B) && at(b + img, 3) > last) {
#pragma unroll
            for (int k = 0; k < 4; ++k)
                for (size_t late = last; late < at(b + img, k); ++late) v[k] = make_float4(v[k].y, v[k].z, v[k].w, 0.0f);
        }
        uint32_t* to = tile + 4 * pq * LDW + cg;
        if (some) {
            to[0] = first_codes(quantize4<YKIND>(v[0].x, v[1].x, v[2].x, v[3].x, r, q), left);
            to[LDW] = first_codes(quantize4<YKIND>(v[0].y, v[1].y, v[2].y, v[3].y, r, q), left);
            to[2 * LDW] = first_codes(quantize4<YKIND>(v[0].z, v[1].z, v[2].z, v[3].z, r, q), left);
            to[3 * LDW] = first_codes(quantize4<YKIND>(v[0].w, v[1].w, v[2].w, v[3].w, r, q), left);
        } else if (ch < Cp) {
            to[0] = to[LDW] = to[2 * LDW] = to[3 * LDW] = 0u;
        }
        __syncthreads();
        const int row = threadIdx.x / PARTS, part = threadIdx.x % PARTS;
        const int out_b = b + row / OWN, out_p = p0 + row % OWN, out_ch = c0 + part * 16;
        if ((IMAGES == 1 || out_b < B) && out_p < HW && out_ch < Cp) {
            const uint32_t* t4 = tile + row * LDW + part * 4;
            *reinterpret_cast<uint4*>(codes + ((size_t)out_b * HW + out_p) * (size_t)Cp + out_ch) = make_uint4(t4[0], t4[1], t4[2], t4[3]);
        }
        b += IMAGES * gridDim.z;
        if (b >= B) break;
        load(b + img);
        __syncthreads();   // the tile is rewritten for the next image
    }
}

// Rows of C elements to rows of Cp codes (a linear layer whose K is no multiple of 16; images of one pixel are the same, and those of
// one channel are rows of one element): a word of four codes per lane, four of them in flight.  Channels C..Cp-1 receive code 0.
// 4000 x 1001 -> 320, the whole call: 131 us as images of one pixel each (a block for 64 elements), 21 us; 30000 x 100 -> 64: 74 and
// 10 us.
template <int YKIND>
__global__ __launch_bounds__(256) void quantize_rows_kernel(const float* __restrict__ x, uint32_t words, int C, int wpr,
                                                            QParams q, ScaleSrc ss, uint32_t* __restrict__ codes)
{
    const Fold f = fold_begin(ss);
    const uint32_t nthreads = gridDim.x * 256;
    uint32_t i = blockIdx.x * 256 + threadIdx.x;                      // words < 2^29: no sum wraps
    float4 v[4];
    int left[4];
    auto load = [&]() {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t at = i + u * nthreads, row = at / (uint32_t)wpr;
            const int k = 4 * (int)(at - row * (uint32_t)wpr);
            left[u] = at < words ? C - k : 0;
            const float* src = x + (size_t)row * C + k;
            if (left[u] >= 4) {
                v[u] = load_any(src, false);
            } else if (left[u] > 0) {
                v[u].x = src[0];
                v[u].y = left[u] > 1 ? src[1] : 0.0f;
                v[u].z = left[u] > 2 ? src[2] : 0.0f;
                v[u].w = 0.0f;
            } else {
                v[u] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            }
        }
    };
    load();
    const float r = fold_end(ss, f);
    while (i < words) {
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (i + u * nthreads < words)
                codes[i + u * nthreads] = first_codes(quantize4<YKIND>(v[u].x, v[u].y, v[u].z, v[u].w, r, q), left[u]);
        i += 4 * nthreads;
        load();
    }
}

template <int GROUPS, int IMAGES>
static void launch_nhwc_patches(const float* x, int B, int C, int Cp, int HW, const QParams& q, const ScaleSrc& ss, uint8_t* codes,
                                hipStream_t st)
{
    constexpr int pixels = 1024 / GROUPS / IMAGES;
    const int kind = hw_kind(q), images = (int)(((int64_t)B + IMAGES - 1) / IMAGES);
    const dim3 grid((HW + pixels - 1) / pixels, (Cp + 4 * GROUPS - 1) / (4 * GROUPS), images < 65535 ? images : 65535);
    auto kern = kind == 1   ? quantize_nhwc_kernel<1, GROUPS, IMAGES>
                : kind == 2 ? quantize_nhwc_kernel<2, GROUPS, IMAGES> : quantize_nhwc_kernel<0, GROUPS, IMAGES>;
    hipLaunchKernelGGL(kern, grid, dim3(256), 0, st, x, B, C, Cp, HW, q, ss, (size_t)B * C * HW >= kStreamElems, codes);
}

int launch_quantize_nhwc(const float* x, int64_t B, int64_t C, int64_t H, int64_t W, const QParams& q,
                         const ScaleSrc& ss, uint8_t* codes, hipStream_t st)
{
    const int Cp = (int)padded_channels(C), HW = (int)(H * W), kind = hw_kind(q);
    // One channel: planes of fewer than 64 pixels as rows (100000 of 2 x 2: 6.6 us, a patch per image 49.9 us); from 64 on in patches, where
    // a lane has four pixels and not a quarter of one (4 x 1024 x 1024: 19.8 us, rows 31.2 us; 30000 x 8 x 8: 11.2 and 18.5 us).
    // Where 64-channel patches would be more than two per compute unit, patches have the channels that Cp fills, and of small planes
    // several images (20000 x 3 x 8 x 8: 8.4 us, an image each 22.5 us; fewer patches are one round of latencies, which the narrow
    // ones' exchange through LDS makes longer: 8 x 32 x 32 x 32 2.22 us, narrow 2.37).
    const bool narrow = B * ((HW + 63) / 64) > 512;
    if (HW == 1 || (C == 1 && HW < 64)) {
        const uint32_t words = (uint32_t)(B * HW * (Cp / 4));
        auto kern = kind == 1 ? quantize_rows_kernel<1> : kind == 2 ? quantize_rows_kernel<2> : quantize_rows_kernel<0>;
        hipLaunchKernelGGL(kern, dim3(grid_for(words, 1024)), dim3(256), 0, st, x, words, (int)C, Cp / 4, q, ss,
                           reinterpret_cast<uint32_t*>(codes));
    } else if (narrow && Cp <= 16) {                                  // at least four elements
        HW > 64 ? launch_nhwc_patches<4, 1>(x, (int)B, (int)C, Cp, HW, q, ss, codes, st)
                : launch_nhwc_patches<4, 4>(x, (int)B, (int)C, Cp, HW, q, ss, codes, st);
    } else if (narrow && Cp <= 32) {
        HW > 64 ? launch_nhwc_patches<8, 1>(x, (int)B, (int)C, Cp, HW, q, ss, codes, st)
                : launch_nhwc_patches<8, 2>(x, (int)B, (int)C, Cp, HW, q, ss, codes, st);
    } else {
        launch_nhwc_patches<16, 1>(x, (int)B, (int)C, Cp, HW, q, ss, codes, st);
    }
    return hipGetLastError() == hipSuccess ? FPQ_OK : FPQ_ERR_LAUNCH;
}

// ------------------------------------------------------------------------------ dequantize

__global__ __launch_bounds__(256) void dequantize_kernel(const uint8_t* __restrict__ codes, size_t n, int e, int m,
                                                         int b, float scale, float* __restrict__ out)
{
    size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    const size_t nthreads = (size_t)gridDim.x * 256;
    for (; i < n; i += nthreads) out[i] = __fmul_rn(decode_code(codes[i], e, m, b), scale);
}

int launch_dequantize(const uint8_t* codes, size_t n, int e, int m, int b, float scale, float* out, hipStream_t st)
{
    if (n == 0) return FPQ_OK;
    hipLaunchKernelGGL(dequantize_kernel, dim3(grid_for(n, 256)), dim3(256), 0, st, codes, n, e, m, b, scale, out);
    return hipGetLastError() == hipSuccess ? FPQ_OK : FPQ_ERR_LAUNCH;
}

// ------------------------------------------------------------------------------ pack weights

// One block per output channel n.  The row's scale is its absmax / c unless given; every element
// is quantized (Eq. (12) with its mask entry, or Eq. (8) without a mask) and written to the packed
// row in (kh, kw, ci) order with ci padded to Cp and the row padded to Kpad, padding = code 0.
// A lane builds one 4-byte word of the packed row: 4 codes, or 8 codes for 4-bit formats.
template <bool FOUR_BIT>
__global__ __launch_bounds__(256) void pack_weights_kernel(const float* __restrict__ w, int Cin, int taps, int Cp,
                                                           int Kpad, QParams q, const float* __restrict__ scale_in,
                                                           const uint8_t* __restrict__ mask,
                                                           uint8_t* __restrict__ packed_rows,
                                                           float* __restrict__ scale_out,
                                                           uint8_t* __restrict__ codes_out)
{
    const int n = blockIdx.x;
    const size_t K = (size_t)Cin * taps;
    const float* row = w + (size_t)n * K;
    const uint8_t* mrow = mask ? mask + (size_t)n * K : nullptr;
    float s;
    if (scale_in) {
        s = scale_in[n];
    } else {
        float v = 0.0f;
        for (size_t i = threadIdx.x; i < K; i += 256) v = fmaxf(v, fabsf(row[i]));
        v = block_max(v);
        s = (v == 0.0f) ? 1.0f : __fdiv_rn(v, q.c);
    }
    if (threadIdx.x == 0) scale_out[n] = s;
    const float r = __fdiv_rn(1.0f, s);
    constexpr int GW = FOUR_BIT ? 8 : 4;
    const size_t row_bytes = FOUR_BIT ? (size_t)Kpad / 2 : (size_t)Kpad;
    uint32_t* dst = reinterpret_cast<uint32_t*>(packed_rows + (size_t)n * row_bytes);
    for (int g = threadIdx.x; g < Kpad / GW; g += 256) {
        const int kp0 = g * GW;
        const int tap = kp0 / Cp;
        const int ci0 = kp0 - tap * Cp;
        uint32_t word = 0;
#pragma unroll
        for (int j = 0; j < GW; ++j) {
            const int ci = ci0 + j;
            uint32_t code = 0;
            if (tap < taps && ci < Cin) {
                const size_t src = (size_t)ci * taps + tap;   // [Cin, kh, kw] within the row
                code = mrow ? quantize_mask(row[src], r, mrow[src], q) : quantize_nearest(row[src], r, q);
                if (codes_out) codes_out[(size_t)n * K + src] = (uint8_t)code;
            }
            word |= code << (FOUR_BIT ? 4 * j : 8 * j);
        }
        dst[g] = word;
    }
}

int launch_pack_weights(const float* w, int64_t N, int64_t Cin, int taps, const QParams& q, bool four_bit,
                        const float* scale_in, const uint8_t* mask, uint8_t* packed_rows, float* scale_out,
                        uint8_t* codes_out, hipStream_t st)
{
    int Cp = (int)padded_channels(Cin);
    int Kpad = (int)padded_k(Cin, taps);
    if (four_bit)
        hipLaunchKernelGGL(pack_weights_kernel<true>, dim3((unsigned)N), dim3(256), 0, st, w, (int)Cin, taps, Cp, Kpad,
                           q, scale_in, mask, packed_rows, scale_out, codes_out);
    else
        hipLaunchKernelGGL(pack_weights_kernel<false>, dim3((unsigned)N), dim3(256), 0, st, w, (int)Cin, taps, Cp,
                           Kpad, q, scale_in, mask, packed_rows, scale_out, codes_out);
    return hipGetLastError() == hipSuccess ? FPQ_OK : FPQ_ERR_LAUNCH;
}

}  // namespace fpq
