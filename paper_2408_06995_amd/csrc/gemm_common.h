// Device helpers shared by the GEMM / implicit-GEMM kernels of libfpq: LDS tile geometry and the
// code -> bf16 decoders (Eq. (5) of the paper, with the subnormal row of Eq. (9)).
#pragma once
#include "fpq_dev.h"
#include "fpq_host.h"

namespace fpq {

typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));

// ---------------------------------------------------------------------------------- activations (codes out)

// x * sigmoid(x) with the hardware exponential and reciprocal: relative error below 1e-6.  For very negative x the
// exponential overflows to +inf and the product is -0: the exact value is below the smallest fp32 number there.
__device__ __forceinline__ float act_silu(float x) { return x * __frcp_rn(1.0f + __expf(-x)); }

// g * Phi(g), Phi the standard normal distribution function = 1 - erfc(g / sqrt 2) / 2, with
// erfc(z) = t (a1 + t (a2 + t (a3 + t (a4 + t a5)))) exp(-z^2), t = 1 / (1 + p z), z >= 0 (Abramowitz & Stegun
// 7.1.26, absolute error of the formula 1.5e-7); the result is max(g, 0) - |g| erfc(|g| / sqrt 2) / 2, so nothing cancels on the
// negative side.  Fourteen instructions, two of them transcendental: the factor 1/2 is in the coefficients, exp(-g^2 / 2) =
// 2^-(s s), and the hardware's reciprocal, within one unit of its last place, does no harm: the largest error over |g| is 3.1e-7 over all
// floats between 1e-30 and 1e30, 3.1e-7 with the correctly rounded one, 3.2e-7 of g (1 - erfc / 2) on the positive side with that one
// (an error of a whole unit in every reciprocal would give 3.6e-7; 4e-7 is what callers may count on).  The bound on |g| keeps infinity times 0 out; the
// exponential is 0 long before.  A negative g whose result underflows gives -0; NaN stays NaN (the plain maximum drops it).
__device__ __forceinline__ float act_gelu(float g)
{
    const float m = fminf(fabsf(g), 1e18f);
    const float s = m * 0.84932180028801907f;                          // sqrt(log2(e) / 2)
    const float t = __builtin_amdgcn_rcpf(fmaf(0.23164188f, m, 1.0f));   // p / sqrt(2)
    float p = fmaf(t, 0.5f * 1.061405429f, 0.5f * -1.453152027f);
    p = fmaf(t, p, 0.5f * 1.421413741f);
    p = fmaf(t, p, 0.5f * -0.284496736f);
    p = fmaf(t, p, 0.5f * 0.254829592f);
    const float half_erfc = (t * p) * __builtin_amdgcn_exp2f(-s * s);
    return fmaf(-m, half_erfc, __builtin_elementwise_maximum(g, -0.0f));
}

// The same as real function calls, for the rarely taken, fully unrolled element-wise paths (edge tiles, the
// register-staged kernels), where inlining them a few hundred times over makes the kernels spill.
__device__ __attribute__((noinline)) float act_silu_call(float x) { return act_silu(x); }
__device__ __attribute__((noinline)) float act_gelu_call(float g) { return act_gelu(g); }

// The value of the lane 16 away inside each group of 32 lanes (ds_swizzle, bit-mask mode: xor 0x10).
__device__ __forceinline__ float lane_xor16(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_ds_swizzle(__builtin_bit_cast(int, v), 0x401F));
}

// ---------------------------------------------------------------------------------- LDS geometry

// Byte offset of 16-byte chunk c of a tile row.  Rows are ROWB (128 or 64) bytes; the chunk index
// is xor-ed with bits of the row so that the lanes of a half-wave, which read the same chunk of 32
// consecutive rows, spread over all LDS banks.
template <int ROWB>
__device__ __forceinline__ int lds_off(int row, int c)
{
    if (ROWB == 128) return row * 128 + ((c ^ ((row >> 1) & 7)) << 4);
    return row * 64 + ((c ^ ((row >> 2) & 3)) << 4);
}

// ---------------------------------------------------------------------------------- convolution geometry

__device__ __forceinline__ int divide(int n, const Divisor& d) { return (int)(__umulhi(2u * (unsigned)n, d.mul) >> d.shift); }

// Output pixel m: byte offset of its tap (0, 0), channel 0 in the channels-last codes (wraps below zero for halo rows), and its taps that
// lie inside the image, bit r kw + c.  Valid kernel columns and rows are ranges; a multiplication repeats the one's bits at the
// other's: about 25 instructions where a loop over nine taps and two divisions by the compiler take 120 (they are all that a workgroup
// does before its first load goes out).
__device__ __forceinline__ void conv_row(const ConvArgs& a, int m, unsigned& base, unsigned& taps)
{
    const int bi = divide(m, a.by_hw), rem = m - bi * (a.Ho * a.Wo);
    const int ho = divide(rem, a.by_wo), wo = rem - ho * a.Wo;
    const int hi0 = ho * a.stride - a.pad, wi0 = wo * a.stride - a.pad;
    base = (unsigned)(((bi * a.H + hi0) * a.W + wi0) * a.Cp);
    const int c0 = min(max(-wi0, 0), a.kw), c1 = min(max(a.W - wi0, 0), a.kw);
    const int r0 = min(max(-hi0, 0), a.kh), r1 = min(max(a.H - hi0, 0), a.kh);
    taps = (a.tap_rows & ((1u << (r1 * a.kw)) - (1u << (r0 * a.kw)))) * ((1u << c1) - (1u << c0));
}

// ---------------------------------------------------------------------------------- code -> bf16

// Eight codes (two dwords for one-code-per-byte operands, one dword for 4-bit operands) to the
// bf16x8 fragment of one MFMA k-step.  KIND selects the decoder.
struct GenFmt {
    int e, m, b;
};

__device__ __forceinline__ uint32_t generic_pair(uint32_t c0, uint32_t c1, const GenFmt& f)
{
    // fp32 bit pattern with the code's exponent/mantissa fields in place has the value
    // 2^(p-127) (1 + f/2^m) for p >= 1 and the fp32 subnormal f 2^(-126-m) for p = 0; multiplying by
    // 2^(127-b) (as 2^64 * 2^(63-b), both representable for |b| <= 64) yields Eq. (5) and its
    // subnormal row alike.  The result has at most 7 significant bits, so the upper half of the
    // fp32 word is its exact bf16.
    const uint32_t magmask = (1u << (f.e + f.m)) - 1u;
    const float k1 = __uint_as_float((uint32_t)(127 + 64) << 23);        // 2^64
    const float k2 = __uint_as_float((uint32_t)(127 + 63 - f.b) << 23);  // 2^(63-b)
    float v0 = __uint_as_float((c0 & magmask) << (23 - f.m)) * k1 * k2;
    float v1 = __uint_as_float((c1 & magmask) << (23 - f.m)) * k1 * k2;
    uint32_t b0 = (__float_as_uint(v0) >> 16) | (((c0 >> (f.e + f.m)) & 1u) << 15);
    uint32_t b1 = (__float_as_uint(v1) >> 16) | (((c1 >> (f.e + f.m)) & 1u) << 15);
    return b0 | (b1 << 16);
}

// Codes of a format with e <= 4 as halves: the exponent and mantissa fields, shifted into place, are a half whose value is
// Eq. (5) times 2^(b - 15), the subnormal row included (a half's own subnormals); the factor goes into the epilogue.
// Given words with a code in the top bits of each half, one arithmetic shift moves the fields down and one mask takes the
// copies of the sign away: with the byte permute three vector instructions per pair, where the arithmetic decode of
// generic_pair takes about fourteen.  Halves of at most 8 significant bits multiply exactly into fp32.
typedef short v2s __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t half_pair(uint32_t top, short shift, uint32_t mask)
{
    const v2s s = {shift, shift};
    return __builtin_bit_cast(uint32_t, (v2s)(__builtin_bit_cast(v2s, top) >> s)) & mask;
}

template <int KIND>
__device__ __forceinline__ v8bf decode8(uint32_t lo, uint32_t hi, const GenFmt& f)
{
    union {
        v8bf v;
        v2bf p[4];
        uint32_t u[4];
    } o;
    if constexpr (KIND == OPK_FP8) {
        o.p[0] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(lo, 1.0f, false);
        o.p[1] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(lo, 1.0f, true);
        o.p[2] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(hi, 1.0f, false);
        o.p[3] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(hi, 1.0f, true);
    } else if constexpr (KIND == OPK_BF8) {
        o.p[0] = __builtin_amdgcn_cvt_scalef32_pk_bf16_bf8(lo, 1.0f, false);
        o.p[1] = __builtin_amdgcn_cvt_scalef32_pk_bf16_bf8(lo, 1.0f, true);
        o.p[2] = __builtin_amdgcn_cvt_scalef32_pk_bf16_bf8(hi, 1.0f, false);
        o.p[3] = __builtin_amdgcn_cvt_scalef32_pk_bf16_bf8(hi, 1.0f, true);
    } else if constexpr (KIND == OPK_FP4) {   // eight 4-bit codes in lo
        o.p[0] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(lo, 1.0f, 0);
        o.p[1] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(lo, 1.0f, 1);
        o.p[2] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(lo, 1.0f, 2);
        o.p[3] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(lo, 1.0f, 3);
    } else if constexpr (KIND == OPK_GENERIC8) {
        o.u[0] = generic_pair(lo & 0xffu, (lo >> 8) & 0xffu, f);
        o.u[1] = generic_pair((lo >> 16) & 0xffu, lo >> 24, f);
        o.u[2] = generic_pair(hi & 0xffu, (hi >> 8) & 0xffu, f);
        o.u[3] = generic_pair((hi >> 16) & 0xffu, hi >> 24, f);
    } else if constexpr (KIND == OPK_HALF8 || KIND == OPK_HALF4) {
        const int em = f.e + f.m;
        const short shift = (short)(5 - f.e);
        const uint32_t one = 0x8000u | (((1u << em) - 1u) << (10 - f.m));
        const uint32_t mask = one | (one << 16);
        if constexpr (KIND == OPK_HALF8) {
            const uint32_t a = lo << (7 - em), b = hi << (7 - em);            // sign in bit 7 of every byte
            o.u[0] = half_pair(__builtin_amdgcn_perm(a, a, 0x010c000cu), shift, mask);   // bytes 0, 1 into the halves' upper bytes
            o.u[1] = half_pair(__builtin_amdgcn_perm(a, a, 0x030c020cu), shift, mask);
            o.u[2] = half_pair(__builtin_amdgcn_perm(b, b, 0x010c000cu), shift, mask);
            o.u[3] = half_pair(__builtin_amdgcn_perm(b, b, 0x030c020cu), shift, mask);
        } else {                                                              // eight 4-bit codes in lo
            const uint32_t odd = lo << (3 - em), even = odd << 4;             // sign in bit 7 of every byte, codes 2j + 1 / 2j
            o.u[0] = half_pair(__builtin_amdgcn_perm(odd, even, 0x040c000cu), shift, mask);
            o.u[1] = half_pair(__builtin_amdgcn_perm(odd, even, 0x050c010cu), shift, mask);
            o.u[2] = half_pair(__builtin_amdgcn_perm(odd, even, 0x060c020cu), shift, mask);
            o.u[3] = half_pair(__builtin_amdgcn_perm(odd, even, 0x070c030cu), shift, mask);
        }
    } else {   // OPK_GENERIC4: eight 4-bit codes in lo
        o.u[0] = generic_pair(lo & 0xfu, (lo >> 4) & 0xfu, f);
        o.u[1] = generic_pair((lo >> 8) & 0xfu, (lo >> 12) & 0xfu, f);
        o.u[2] = generic_pair((lo >> 16) & 0xfu, (lo >> 20) & 0xfu, f);
        o.u[3] = generic_pair((lo >> 24) & 0xfu, lo >> 28, f);
    }
    return o.v;
}

// Grouped linear layers: blockIdx.y picks the problem, blockIdx.x the output tile within it (the grid is as wide as
// the problem with the most tiles; workgroups beyond a problem's own tile count leave at once).
__device__ __forceinline__ GemmArgs grouped_problem_args(const GroupedArgs& g, int pi)
{
    GemmArgs a = g.common;
    const GroupedProblem& q = g.p[pi];
    a.x = q.xcodes;
    a.wrows = q.wrows;
    a.sw = q.sw;
    a.bias = q.bias;
    a.sx_dev = q.sx_dev;
    a.y = q.y;
    a.M = q.M; a.N = q.N; a.Kpad = q.Kpad; a.Kreal = q.K;
    a.B = q.M; a.H = 1; a.W = 1; a.Cp = q.K; a.Ho = 1; a.Wo = 1;
    a.x_bytes = (uint32_t)q.M * (uint32_t)q.K;              // below 2^31
    a.w_bytes = q.w_bytes;
    return a;
}

constexpr bool kind_is_4bit(int k) { return k == OPK_FP4 || k == OPK_GENERIC4 || k == OPK_HALF4; }

// One 32 x 32 x 16 step of the fp32-accumulate mode on fragments of decode8 (both operands are halves or both bf16).
typedef _Float16 v8h __attribute__((ext_vector_type(8)));
template <int KIND>
__device__ __forceinline__ v16f mfma_exact(v8bf a, v8bf b, v16f c)
{
    if constexpr (KIND == OPK_HALF8 || KIND == OPK_HALF4)
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(v8h, a), __builtin_bit_cast(v8h, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
// Format selector of the f8f6f4 MFMA: 0 = E4M3, 1 = E5M2, 4 = E2M1.
constexpr int mfma_fmt(int k) { return k == OPK_FP8 ? 0 : (k == OPK_BF8 ? 1 : 4); }

}  // namespace fpq
