// Gradient-based rounding learning for low-bitwidth weights (Section V-B, Eq. (10)-(14)): one gradient-descent step
// on the per-weight parameters alpha of a linear layer, on calibration activations in full precision.
//
//   y' = clamp(fl32(W * fl32(1 / sw[n])), -c, c),  s = step of Eq. (9) at y',  fl = floor(y' / s)
//   Wq(alpha) = clamp(s (fl + sigmoid(alpha)), -c, c) * sw[n]                                   (Eq. (12), soft)
//   loss = mean((A Wq^T - A W^T)^2) + reg_weight * mean(1 - (2 |sigmoid(alpha) - 0.5|)^20)     (Eq. (11), (13), (14))
//
// The step runs as: D = Wq(alpha) - W (elementwise, with the regulariser's sum);  R = A D^T (the output error
// A Wq^T - A W^T in one product, with the sums of R^2);  G = (2 / (M N)) R^T A = d mse / d Wq;
// alpha -= lr (G * dWq/dalpha + reg_weight * dreg/dalpha) and the losses: four launches.  The two products are dense fp32
// contractions, computed on the bf16 matrix instruction with every fp32 operand split into three bf16 parts (sgemm_kernel).
#include <type_traits>

#include "fpq_dev.h"
#include "fpq_host.h"

namespace fpq {

namespace {

typedef float v16f __attribute__((ext_vector_type(16)));

__device__ __forceinline__ float sigmoid_f(float a) { return 1.0f / (1.0f + expf(-a)); }

// The weight on the format's axis: clipped value y', step s of Eq. (9) (a power of two) and floor(y' / s).
struct OnAxis {
    float yc, s, fl;
};
__device__ __forceinline__ OnAxis on_axis(float w, float r, const QParams& q)
{
    OnAxis o;
    o.yc = fminf(fmaxf(__fmul_rn(w, r), -q.c), q.c);
    const uint32_t ab = __float_as_uint(o.yc) & 0x7fffffffu;
    const int P = max((int)(ab >> 23) - 127 + q.b, 1);
    const int es = P - q.b - q.m;
    o.s = __uint_as_float((uint32_t)(127 + es) << 23);
    o.fl = floorf(__fmul_rn(o.yc, __uint_as_float((uint32_t)(127 - es) << 23)));   // exact: |y' / s| < 2^(m+1)
    return o;
}

__device__ __forceinline__ float block_sum(float v)
{
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    __shared__ float wsum[4];
    __syncthreads();
    if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = v;
    __syncthreads();
    return wsum[0] + wsum[1] + wsum[2] + wsum[3];
}

// Position of a grid-strided index in a matrix of K columns (in units of V neighbouring elements of a row), kept by addition:
// one division per thread.
template <int V>
struct Walk {
    size_t i, n, step;
    int row, col, drow, dcol, K;
    __device__ Walk(size_t n_, int K_) : n(n_ / V), K(K_ / V)
    {
        i = (size_t)blockIdx.x * 256 + threadIdx.x;
        step = (size_t)gridDim.x * 256;
        row = (int)((uint32_t)i / (uint32_t)K);            // N K < 2^31
        col = (int)((uint32_t)i - (uint32_t)row * (uint32_t)K);
        drow = (int)((uint32_t)step / (uint32_t)K);
        dcol = (int)((uint32_t)step - (uint32_t)drow * (uint32_t)K);
    }
    __device__ bool more() const { return i < n; }
    __device__ void next()
    {
        i += step;
        row += drow;
        col += dcol;
        if (col >= K) { col -= K; ++row; }
    }
};
template <int V>
struct Pack {                                              // V floats, one load or store
    float v[V];
};
template <int V>
__device__ __forceinline__ Pack<V> get(const float* p, size_t i)
{
    Pack<V> r;
    if (V == 4) {
        const float4 a = reinterpret_cast<const float4*>(p)[i];
        r.v[0] = a.x; r.v[1 % V] = a.y; r.v[2 % V] = a.z; r.v[3 % V] = a.w;
    } else {
        r.v[0] = p[i];
    }
    return r;
}
template <int V>
__device__ __forceinline__ void put(float* p, size_t i, const Pack<V>& r)
{
    if (V == 4)
        reinterpret_cast<float4*>(p)[i] = make_float4(r.v[0], r.v[1 % V], r.v[2 % V], r.v[3 % V]);
    else
        p[i] = r.v[0];
}

// D = Wq(alpha) - W and the per-block sums of the regulariser 1 - (2 |sigmoid - 0.5|)^20.
template <int V>
__global__ __launch_bounds__(256) void rl_soft_kernel(const float* __restrict__ w, const float* __restrict__ sw,
                                                      const float* __restrict__ alpha, size_t n, int K, QParams q,
                                                      float* __restrict__ d, float* __restrict__ reg_partial)
{
    float reg = 0.0f;
    for (Walk<V> k(n, K); k.more(); k.next()) {
        const float s_n = sw[k.row], r_n = __fdiv_rn(1.0f, s_n);
        const Pack<V> wi = get<V>(w, k.i), al = get<V>(alpha, k.i);
        Pack<V> out;
#pragma unroll
        for (int e = 0; e < V; ++e) {
            const OnAxis o = on_axis(wi.v[e], r_n, q);
            const float sg = sigmoid_f(al.v[e]);
            const float qv = fminf(fmaxf(o.s * (o.fl + sg), -q.c), q.c);
            out.v[e] = qv * s_n - wi.v[e];
            const float u = 2.0f * fabsf(sg - 0.5f);
            const float u2 = u * u, u4 = u2 * u2, u8 = u4 * u4, u16 = u8 * u8;
            reg += 1.0f - u16 * u4;
        }
        put<V>(d, k.i, out);
    }
    reg = block_sum(reg);
    if (threadIdx.x == 0) reg_partial[blockIdx.x] = reg;
}

// loss_out[0] = sum(sq partials) / count_mse, loss_out[1] = sum(reg partials) / count_reg  (double across blocks),
// by one workgroup of the update kernel
struct LossArgs {
    const float* sq;
    int nsq;
    double count_mse;
    const float* reg;
    int nreg;
    double count_reg;
    float* out;
};
__device__ void write_losses(const LossArgs& l)
{
    __shared__ double acc[2][256];
    double a = 0.0, b = 0.0;
    for (int i = threadIdx.x; i < l.nsq; i += 256) a += (double)l.sq[i];
    for (int i = threadIdx.x; i < l.nreg; i += 256) b += (double)l.reg[i];
    acc[0][threadIdx.x] = a;
    acc[1][threadIdx.x] = b;
    __syncthreads();
    for (int off = 128; off > 0; off >>= 1) {
        if ((int)threadIdx.x < off) {
            acc[0][threadIdx.x] += acc[0][threadIdx.x + off];
            acc[1][threadIdx.x] += acc[1][threadIdx.x + off];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        l.out[0] = (float)(acc[0][0] / l.count_mse);
        l.out[1] = (float)(acc[1][0] / l.count_reg);
    }
}

// alpha -= lr * (g * dWq/dalpha + reg_weight * dreg/dalpha); the gradient itself goes to grad_out when asked for.
// The last workgroup writes the losses.
template <int V>
__global__ __launch_bounds__(256) void rl_update_kernel(const float* __restrict__ w, const float* __restrict__ sw,
                                                        float* __restrict__ alpha, const float* __restrict__ g, int gslices,
                                                        size_t n, int K, QParams q, float lr, float reg_scale,
                                                        float* __restrict__ grad_out, LossArgs losses)
{
    if (blockIdx.x == gridDim.x - 1) write_losses(losses);
    for (Walk<V> k(n, K); k.more(); k.next()) {
        const float s_n = sw[k.row], r_n = __fdiv_rn(1.0f, s_n);
        const Pack<V> wi = get<V>(w, k.i), al = get<V>(alpha, k.i);
        Pack<V> gi = get<V>(g, k.i), next, grad;             // d mse / d Wq: the slices of the product, in order
        int z = 1;
        for (; z + 4 <= gslices; z += 4) {                   // four loads in flight
            Pack<V> t[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) t[u] = get<V>(g + (size_t)(z + u) * n, k.i);
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int e = 0; e < V; ++e) gi.v[e] += t[u].v[e];
        }
        for (; z < gslices; ++z) {
            const Pack<V> t = get<V>(g + (size_t)z * n, k.i);
#pragma unroll
            for (int e = 0; e < V; ++e) gi.v[e] += t.v[e];
        }
#pragma unroll
        for (int e = 0; e < V; ++e) {
            const OnAxis o = on_axis(wi.v[e], r_n, q);
            const float a = al.v[e];
            const float sg = sigmoid_f(a);
            const float ds = sg * sigmoid_f(-a);            // sigmoid' = sigmoid(a) sigmoid(-a): 1 - sigmoid would cancel for large a
            const float pre = o.s * (o.fl + sg);
            const float dwq = (pre > -q.c && pre < q.c) ? o.s * ds * s_n : 0.0f;   // the outer clamp passes no gradient
            const float dv = sg - 0.5f;
            const float u = 2.0f * fabsf(dv);
            const float u2 = u * u, u4 = u2 * u2, u8 = u4 * u4, u16 = u8 * u8;
            const float dlam = -20.0f * (u16 * u2 * u) * 2.0f * (dv > 0.0f ? 1.0f : (dv < 0.0f ? -1.0f : 0.0f)) * ds;
            grad.v[e] = gi.v[e] * dwq + reg_scale * dlam;
            next.v[e] = a - lr * grad.v[e];
        }
        if (grad_out) put<V>(grad_out, k.i, grad);
        put<V>(alpha, k.i, next);
    }
}

// alpha with sigmoid(alpha) = the weight's fractional position between its grid neighbours, kept inside [eps, 1 - eps].
__global__ __launch_bounds__(256) void rl_init_kernel(const float* __restrict__ w, const float* __restrict__ sw, size_t n,
                                                      int K, QParams q, float eps, float* __restrict__ alpha)
{
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) {
        const float s_n = sw[i / K];
        const OnAxis o = on_axis(w[i], __fdiv_rn(1.0f, s_n), q);
        const float inv_s = 1.0f / o.s;                                  // exact: a power of two
        const float frac = fminf(fmaxf(o.yc * inv_s - o.fl, eps), 1.0f - eps);   // exact before the clip
        alpha[i] = logf(frac / (1.0f - frac));
    }
}

__global__ __launch_bounds__(256) void rl_mask_kernel(const float* __restrict__ alpha, size_t n, uint8_t* __restrict__ mask)
{
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256)
        mask[i] = alpha[i] >= 0.0f ? 1 : 0;                               // sigmoid(alpha) >= 0.5
}

// A convolution enters rounding learning as the linear layer on its patch matrix: row (b, ho, wo) of a holds the
// receptive field of that output pixel in the order of the flattened weight [Cout, (ci, kh, kw)], zeros where the
// field reaches into the padding.  Lanes run along the row (the kw taps of one (ci, kh) are neighbours in x).
__global__ __launch_bounds__(256) void rl_im2col_kernel(const float* __restrict__ x, int C, int H, int W, int kh, int kw,
                                                        int stride, int pad, int Ho, int Wo, size_t rows,
                                                        float* __restrict__ a)
{
    const int K = C * kh * kw;
    const size_t total = rows * (size_t)K;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (size_t)gridDim.x * 256) {
        const size_t row = i / K;
        const int k = (int)(i - row * K);
        const int ci = k / (kh * kw), t = k - ci * (kh * kw), r = t / kw, c = t - r * kw;
        const int wo = (int)(row % Wo), ho = (int)((row / Wo) % Ho);
        const size_t b = row / ((size_t)Wo * Ho);
        const int h = ho * stride - pad + r, w = wo * stride - pad + c;
        a[i] = (h >= 0 && h < H && w >= 0 && w < W) ? x[((b * C + ci) * H + h) * (size_t)W + w] : 0.0f;
    }
}

// ---------------------------------------------------------------------------------- fp32 contraction
//
// C[i, j] = scale * sum_k P(i, k) Q(j, k), i < I, j < J, k < Kc, with P(i, k) = p[i * pi + k * pk] and the same for Q:
// KCONTIG = true:  pk = 1 (rows of P and Q run along k: C = P Q^T),
// KCONTIG = false: pi = 1 (rows of the stored matrices run along i / j: C = P'^T Q' with P' = [Kc, I], Q' = [Kc, J]).
//
// Every fp32 operand x is split into three bf16 parts, x = h + m + l: h = bf16(x), m = bf16(x - h), l = x - h - m, each
// difference exact, the last one representable (24 significant bits = 8 + 8 + 8; the split of Henry, Tang and Heinecke,
// "Leveraging the bfloat16 artificial intelligence datatype for higher-precision computations", ARITH 2019).  Of the nine products
// of a pair the six largest go to the matrix unit (bf16 products are exact in fp32, sums are fp32): hh, hm, mh, mm, hl, lh.  The
// three left out are at most 2^-24 of |x y| together, 5.5e-9 (2^-27.4) in the root mean square over normal deviates, where one fp32
// rounding, of which every addition makes one of the whole partial sum, has 2.5e-8.  The rate of the fp32 matrix instruction is 1/16
// of the bf16 one: six bf16 steps take 3/8 of the time of an fp32 one.
// An operand that is infinite, or rounds to bf16's infinity, has parts that are NaN: an output that is no finite number is computed
// once more by plain fp32 multiply-adds, so that it is what the operands themselves make it.  The last part meets bf16's smallest
// number below 2^-110: smaller operands keep fewer than 24 bits.
//
// A workgroup of four wavefronts (2 x 2) owns a T x T tile of C (T = 128 or 64) and walks k in steps of 16 through three LDS
// buffers; the split happens in registers between the global load and the LDS store.  Per step and wavefront at T = 128:
// 24 MFMAs (768 cycles) on 12 LDS reads.  The unit of loads and stores is a quad, 4 consecutive k of one row:
//   KCONTIG: a thread loads a quad with one 16-byte load, four neighbouring threads the 64 bytes of a row and step;
//   else: a thread loads 4 k x W neighbouring rows (W = 4 or 2, one load per k) and has W quads.
// LDS holds, per part, the first eight k of all rows (16 bytes a row), then the others.  Without KCONTIG row W i + e of the
// tile is kept at place e T / W + i, so that both the stores of a wavefront (e fixed, i running) and its operand reads (32 places
// in a row) run along the banks; the result's rows and columns are renamed accordingly.
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
typedef float v2f __attribute__((ext_vector_type(2)));

struct Split {
    uint32_t h, m, l;       // the parts of two neighbouring elements
};
__device__ __forceinline__ uint32_t bf16_pair(float a, float b)
{
    const v2f v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, v2bf));      // round to nearest even
}
__device__ __forceinline__ Split split_pair(float a, float b)
{
    Split s;
    s.h = bf16_pair(a, b);
    const float ra = a - __uint_as_float(s.h << 16), rb = b - __uint_as_float(s.h & 0xffff0000u);
    s.m = bf16_pair(ra, rb);
    const float qa = ra - __uint_as_float(s.m << 16), qb = rb - __uint_as_float(s.m & 0xffff0000u);
    s.l = bf16_pair(qa, qb);
    return s;
}

template <int T, bool KCONTIG, bool VEC, bool SUMSQ>
__global__ __launch_bounds__(256, 2) void sgemm_kernel(const float* __restrict__ p, long pstride, const float* __restrict__ qm,
                                                       long qstride, int I, int J, int Kc, float scale, float* __restrict__ c,
                                                       long cstride, int kslice, float* __restrict__ sq_partial)
{
    constexpr int BK = 16;
    constexpr int NB = T / 64;                     // 32-row blocks per wave and direction
    constexpr int HALF = T + 8;                    // 16-byte places of eight k (8 of padding shift the second half's banks)
    constexpr int PART = 2 * HALF;
    constexpr int W = KCONTIG ? 1 : T / 32;        // neighbouring rows per thread
    constexpr int PD = T == 64 ? 4 : 2;            // steps of the small tile are short against the latency of a load
    constexpr int NQ = KCONTIG ? 2 * NB : W;       // quads per thread and step
    extern __shared__ __attribute__((aligned(16))) uint4 tiles_lds[];           // [3 buffers][P, Q][3 parts][PART]
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int l32 = lane & 31, g = lane >> 5;
    const int wi = wave >> 1, wj = wave & 1;
    // Workgroup -> tile: ids go round-robin over the 8 XCDs; each takes a contiguous run of tiles (they share rows of P)
    const int tiles_j = (J + T - 1) / T, tiles = tiles_j * ((I + T - 1) / T);
    int bid = blockIdx.x;
    {
        const int per = tiles >> 3;
        if (bid < (per << 3)) bid = (bid & 7) * per + (bid >> 3);
    }
    const int i0 = bid / tiles_j * T, j0 = bid % tiles_j * T;
    // slice blockIdx.y of the contraction (kslice steps of k each, a multiple of BK) writes its own copy of C
    const int kbeg = blockIdx.y * kslice;
    const int kend = kbeg + kslice < Kc ? kbeg + kslice : Kc;
    c += (size_t)blockIdx.y * (size_t)I * cstride;

    v16f acc[NB][NB];
#pragma unroll
    for (int a = 0; a < NB; ++a)
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.0f;

    // This thread's quads.  KCONTIG: quad kq of rows (tid / 4) + 64 r of P, then of Q; else: quad kq of W rows of P (the first
    // two wavefronts) or of Q.
    const int half_tid = tid & 127;
    const bool for_q = !KCONTIG && __builtin_amdgcn_readfirstlane(tid >> 7);
    const int kq = KCONTIG ? tid & 3 : half_tid >> 5;
    const float* src[KCONTIG ? NQ : 1];            // row base (KCONTIG) or column base of this thread's quads
    const long stride = for_q ? qstride : pstride;
    if (KCONTIG) {
#pragma unroll
        for (int n = 0; n < NQ; ++n) {
            const int r = (tid >> 2) + 64 * (n % NB);
            src[n] = n < NB ? p + (long)min(i0 + r, I - 1) * pstride : qm + (long)min(j0 + r, J - 1) * qstride;   // rows outside
        }                                                                                                      // never leave the tile
    } else {
        const int o = (for_q ? j0 : i0) + W * (half_tid & 31), O = for_q ? J : I;
        src[0] = (for_q ? qm : p) + (VEC ? min(o, O - W) : o);
    }
    float reg[PD][NQ][4];                          // [set][quad][k]: the global loads run PD steps ahead of the stores
    // No branch around a load (the merge would wait for all that are in flight): k outside the matrix reads its last k instead
    // and becomes zero at the store.
    auto load = [&](auto tail, int k0, int set) {
        constexpr bool TAIL = decltype(tail)::value;
        const int k = k0 + 4 * kq;
        if (KCONTIG) {
#pragma unroll
            for (int n = 0; n < NQ; ++n) {
                if (VEC) {                         // 16-byte aligned rows of a multiple of 4 elements
                    const float4 a = *reinterpret_cast<const float4*>(src[n] + (TAIL ? min(k, Kc - 4) : k));
                    reg[set][n][0] = a.x; reg[set][n][1] = a.y; reg[set][n][2] = a.z; reg[set][n][3] = a.w;
                } else {
#pragma unroll
                    for (int t = 0; t < 4; ++t) reg[set][n][t] = src[n][TAIL ? min(k + t, Kc - 1) : k + t];
                }
            }
        } else {
            const int o = (for_q ? j0 : i0) + W * (half_tid & 31), O = for_q ? J : I;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const float* at = src[0] + (long)(TAIL ? min(k + t, Kc - 1) : k + t) * stride;
                if (VEC) {
                    if (W == 4) {
                        const float4 a = *reinterpret_cast<const float4*>(at);
                        reg[set][0][t] = a.x; reg[set][1][t] = a.y; reg[set][2][t] = a.z; reg[set][NQ - 1][t] = a.w;
                    } else {
                        const float2 a = *reinterpret_cast<const float2*>(at);
                        reg[set][0][t] = a.x; reg[set][1][t] = a.y;
                    }
                } else {
#pragma unroll
                    for (int e = 0; e < W; ++e) reg[set][e][t] = at[min(e, O - 1 - o)];     // e or, outside, the last row
                }
            }
        }
    };
    auto store = [&](auto tail, int k0, int buf, int set) {
        uint2* to = reinterpret_cast<uint2*>(tiles_lds + buf * 6 * PART);
        const int k = k0 + 4 * kq;
#pragma unroll
        for (int n = 0; n < NQ; ++n) {
            float v[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) v[t] = (!decltype(tail)::value || k + t < kend) ? reg[set][n][t] : 0.0f;
            const bool is_q = KCONTIG ? n >= NB : for_q;
            const int place = KCONTIG ? (tid >> 2) + 64 * (n % NB) : n * (T / W) + (half_tid & 31);
            uint2* d = to + 2 * ((is_q ? 3 * PART : 0) + (kq >> 1) * HALF + place) + (kq & 1);
            const Split a = split_pair(v[0], v[1]), b = split_pair(v[2], v[3]);
            d[0] = make_uint2(a.h, b.h);
            d[2 * PART] = make_uint2(a.m, b.m);
            d[4 * PART] = make_uint2(a.l, b.l);
        }
    };
    v8bf pa[2][3][NB], qb[2][3][NB];               // operand fragments, read a step ahead
    auto fragments = [&](int buf, int set) {
        const uint4* at = tiles_lds + buf * 6 * PART + g * HALF + l32;
#pragma unroll
        for (int t = 0; t < 3; ++t)
#pragma unroll
            for (int a = 0; a < NB; ++a) {
                pa[set][t][a] = __builtin_bit_cast(v8bf, at[t * PART + wi * (T / 2) + 32 * a]);
                qb[set][t][a] = __builtin_bit_cast(v8bf, at[(3 + t) * PART + wj * (T / 2) + 32 * a]);
            }
    };

    // Three LDS buffers, one barrier per step.  While step t is multiplied from registers, the fragments of step t + 1 are read
    // (its buffer was complete at the last barrier), tile t + 2, loaded PD steps ago, is split and stored (into the buffer that
    // step t's fragments were read from before the last barrier), and the loads of tile t + 2 + PD go out: nothing that a step waits
    // for was begun in it.
    constexpr std::true_type tail{};
    constexpr std::false_type inside{};
#pragma unroll
    for (int t = 0; t < PD; ++t) load(tail, kbeg + t * BK, t);
    store(tail, kbeg, 0, 0);
    load(tail, kbeg + PD * BK, 0);
    store(tail, kbeg + BK, 1, 1);
    load(tail, kbeg + (PD + 1) * BK, 1);
    __syncthreads();
    fragments(0, 0);
    __syncthreads();
    int b1 = 1, b2 = 2;                            // buffers of tiles t + 1 and t + 2
    auto step_from = [&](auto where, int k0, int t) {
        const int set = t & 1;
        fragments(b1, set ^ 1);
        store(where, k0 + 2 * BK, b2, (t + 2) % PD);
        load(where, k0 + (2 + PD) * BK, (t + 2) % PD);
        auto mul = [&](int tp, int tq) {
#pragma unroll
            for (int a = 0; a < NB; ++a)
#pragma unroll
                for (int b = 0; b < NB; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(pa[set][tp][a], qb[set][tq][b], acc[a][b], 0, 0, 0);
        };
        mul(2, 0);
        mul(0, 2);
        mul(1, 1);
        mul(1, 0);
        mul(0, 1);
        mul(0, 0);
#pragma unroll
        for (int z = 0; z < 6 * NB * NB; ++z) {    // spread the rest of the step between its MFMAs
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x080, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x002, 5, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        __syncthreads();
        __builtin_amdgcn_sched_barrier(0);
        const int b0 = b2;
        b2 = 3 - b1 - b2;
        b1 = b0;
    };
    // PD steps per round without a condition between them (a step beyond the end multiplies zeros): the compiler's wait
    // counts then see which loads are outstanding.
    int k0 = kbeg;
    for (; k0 + (2 * PD + 2) * BK <= kend; k0 += PD * BK) {
#pragma unroll
        for (int t = 0; t < PD; ++t) step_from(inside, k0 + t * BK, t);
    }
    for (; k0 < kend; k0 += PD * BK) {
#pragma unroll
        for (int t = 0; t < PD; ++t) step_from(tail, k0 + t * BK, t);
    }
    auto of_place = [&](int at) { return KCONTIG ? at : W * (at % (T / W)) + at / (T / W); };     // row of the tile kept there
    // acc[a][b][r]: row 8 (r / 4) + 4 g + r % 4 of the block (operand P), column l32 (operand Q)
    auto row_of = [&](int a, int r) { return i0 + of_place(wi * (T / 2) + 32 * a + 8 * (r >> 2) + 4 * g + (r & 3)); };
    auto col_of = [&](int b) { return j0 + of_place(wj * (T / 2) + 32 * b + l32); };
    float sq = 0.0f, finite = 0.0f;                // finite: 0, or NaN once an output was infinite or NaN
#pragma unroll
    for (int a = 0; a < NB; ++a)
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const int j = col_of(b);
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int i = row_of(a, r);
                const float v = scale * acc[a][b][r];
                if (i < I && j < J) {
                    finite = __fmaf_rn(v, 0.0f, finite);
                    if (SUMSQ) sq += v * v;
                    c[(long)i * cstride + j] = v;
                }
            }
        }
    if (!(finite == 0.0f)) {
        sq = 0.0f;
#pragma unroll 1
        for (int z = 0; z < NB * NB * 16; ++z) {
            const int i = row_of(z / (16 * NB), z & 15), j = col_of((z >> 4) % NB);
            if (i >= I || j >= J) continue;
            float v = c[(long)i * cstride + j];
            if (!(fabsf(v) < __builtin_huge_valf())) {
                float sum = 0.0f;
                for (int k = kbeg; k < kend && sum == sum; ++k)
                    sum = KCONTIG ? __fmaf_rn(p[(long)i * pstride + k], qm[(long)j * qstride + k], sum)
                                  : __fmaf_rn(p[(long)k * pstride + i], qm[(long)k * qstride + j], sum);
                v = scale * sum;
                c[(long)i * cstride + j] = v;
            }
            if (SUMSQ) sq += v * v;
        }
    }
    if (SUMSQ) {
        sq = block_sum(sq);
        if (tid == 0) sq_partial[blockIdx.x] = sq;
    }
}

// Tile of a product: 128 where that still gives every compute unit a workgroup.
int tile_of(long I, long J, int slices)
{
    return ((I + 127) / 128) * ((J + 127) / 128) * slices >= 256 ? 128 : 64;
}
long tiles_of(long I, long J, int T) { return ((I + T - 1) / T) * ((J + T - 1) / T); }

// The record of the devices that allow the kernel its LDS is one per kernel: kernels of one type share a static of a generic
// lambda over them.
template <int T, bool KCONTIG, bool VEC, bool SUMSQ>
int launch_sgemm_tile(const float* p, long pstride, const float* q, long qstride, int I, int J, int Kc, float scale, float* c,
                      long cstride, int slices, float* sq, hipStream_t st)
{
    constexpr int lds = 3 * 6 * 2 * (T + 8) * 16;
    auto kern = sgemm_kernel<T, KCONTIG, VEC, SUMSQ>;
    if (lds > 65536) {
        static std::atomic<uint64_t> allowed{0};
        if (!allow_dynamic_lds(reinterpret_cast<const void*>(kern), lds, allowed)) return FPQ_ERR_LAUNCH;
    }
    const int kslice = ((Kc + slices - 1) / slices + 15) / 16 * 16;
    hipLaunchKernelGGL(kern, dim3((unsigned)tiles_of(I, J, T), slices), dim3(256), lds, st, p, pstride, q, qstride, I, J, Kc, scale, c,
                       cstride, kslice, sq);
    return hipGetLastError() == hipSuccess ? FPQ_OK : FPQ_ERR_LAUNCH;
}

// slices > 1: the contraction is cut into that many pieces, piece z writes c + z * I * cstride (the caller adds them up)
template <bool KCONTIG, bool SUMSQ>
int launch_sgemm(const float* p, long pstride, const float* q, long qstride, int I, int J, int Kc, float scale, float* c,
                 long cstride, int slices, float* sq, hipStream_t st)
{
    // 16-byte loads: aligned bases and rows, and a multiple of 4 elements along the direction of the loads
    const bool vec = ((reinterpret_cast<uintptr_t>(p) | reinterpret_cast<uintptr_t>(q)) & 15) == 0 && pstride % 4 == 0 &&
                     qstride % 4 == 0 && (KCONTIG ? Kc % 4 == 0 : I % 4 == 0 && J % 4 == 0);
    const bool big = tile_of(I, J, slices) == 128;
    auto run = vec ? (big ? launch_sgemm_tile<128, KCONTIG, true, SUMSQ> : launch_sgemm_tile<64, KCONTIG, true, SUMSQ>)
                   : (big ? launch_sgemm_tile<128, KCONTIG, false, SUMSQ> : launch_sgemm_tile<64, KCONTIG, false, SUMSQ>);
    return run(p, pstride, q, qstride, I, J, Kc, scale, c, cstride, slices, sq, st);
}

// Slices of the gradient product (its contraction runs over the M calibration rows, its output is only [N, K]): enough
// to give the 128-row tile two workgroups per compute unit, each slice at least 128 rows deep, at most 16 copies and 64 MB.
int rl_slices(int64_t M, int64_t N, int64_t K)
{
    const int64_t tiles = ((N + 127) / 128) * ((K + 127) / 128);
    int64_t s = 512 / tiles;
    if (s > M / 128) s = M / 128;
    if (s > 16) s = 16;
    while (s > 1 && s * N * K > ((int64_t)16 << 20)) --s;
    return s < 1 ? 1 : (int)s;
}

int blocks_for(size_t n)
{
    const size_t b = (n + 1023) / 1024;
    return b < 1 ? 1 : (b > 1024 ? 1024 : (int)b);
}

}  // namespace

size_t rl_workspace_bytes(int64_t M, int64_t N, int64_t K)
{
    // D [N, K], R [M, N], 1024 + one per tile of R partial sums, G [slices][N, K]
    auto up = [](size_t v) { return (v + 255) / 256 * 256; };
    return up((size_t)N * K * 4) + up((size_t)M * N * 4) + 4096 + up((size_t)tiles_of(M, N, tile_of(M, N, 1)) * 4) +
           up((size_t)rl_slices(M, N, K) * N * K * 4);
}

int launch_rl_im2col(const float* x, int64_t B, int64_t C, int64_t H, int64_t W, int kh, int kw, int stride, int pad,
                     float* a, hipStream_t st)
{
    const int Ho = (int)((H + 2 * pad - kh) / stride + 1), Wo = (int)((W + 2 * pad - kw) / stride + 1);
    const size_t rows = (size_t)B * Ho * Wo;
    const size_t total = rows * (size_t)(C * kh * kw);
    size_t grid = (total + 1023) / 1024;
    if (grid > 8192) grid = 8192;
    hipLaunchKernelGGL(rl_im2col_kernel, dim3((unsigned)grid), dim3(256), 0, st, x, (int)C, (int)H, (int)W, kh, kw, stride, pad,
                       Ho, Wo, rows, a);
    return hipGetLastError() == hipSuccess ? FPQ_OK : FPQ_ERR_LAUNCH;
}

int launch_rl_init(const float* w, const float* sw, int64_t N, int64_t K, const QParams& q, float* alpha, hipStream_t st)
{
    const size_t n = (size_t)N * K;
    hipLaunchKernelGGL(rl_init_kernel, dim3(blocks_for(n)), dim3(256), 0, st, w, sw, n, (int)K, q, 1e-3f, alpha);
    return hipGetLastError() == hipSuccess ? FPQ_OK : FPQ_ERR_LAUNCH;
}

int launch_rl_mask(const float* alpha, size_t n, uint8_t* mask, hipStream_t st)
{
    hipLaunchKernelGGL(rl_mask_kernel, dim3(blocks_for(n)), dim3(256), 0, st, alpha, n, mask);
    return hipGetLastError() == hipSuccess ? FPQ_OK : FPQ_ERR_LAUNCH;
}

// 8192 rows, 1280 x 1280 weights: 726 us with the fp32 matrix instruction (its two products 320 and 363), 323 us with the
// split operands (155 and 173 in the profiler's trace; matrix unit busy 0.64 and 0.55 of the time, the rest is operand loads and the
// split).
int launch_rl_step(const float* w, const float* sw, int64_t N, int64_t K, const QParams& q, float* alpha, const float* a,
                   int64_t M, float lr, float reg_weight, float* loss_out, float* grad_out, void* workspace, hipStream_t st)
{
    auto up = [](size_t v) { return (v + 255) / 256 * 256; };
    uint8_t* ws = static_cast<uint8_t*>(workspace);
    float* d = reinterpret_cast<float*>(ws);
    float* r = reinterpret_cast<float*>(ws + up((size_t)N * K * 4));
    float* regp = reinterpret_cast<float*>(ws + up((size_t)N * K * 4) + up((size_t)M * N * 4));
    float* sqp = regp + 1024;
    const int nsq = (int)tiles_of(M, N, tile_of(M, N, 1));
    float* g = reinterpret_cast<float*>(reinterpret_cast<uint8_t*>(sqp) + up((size_t)nsq * 4));
    const int slices = rl_slices(M, N, K);
    const size_t nw = (size_t)N * K, nr = (size_t)M * N;
    const int bw = blocks_for(nw);
    // four neighbouring weights per thread where rows and bases allow it
    const bool v4 = K % 4 == 0 && ((reinterpret_cast<uintptr_t>(w) | reinterpret_cast<uintptr_t>(alpha) |
                                    reinterpret_cast<uintptr_t>(grad_out)) & 15) == 0;
    auto soft = v4 ? rl_soft_kernel<4> : rl_soft_kernel<1>;
    auto update = v4 ? rl_update_kernel<4> : rl_update_kernel<1>;
    hipLaunchKernelGGL(soft, dim3(bw), dim3(256), 0, st, w, sw, alpha, nw, (int)K, q, d, regp);
    // R[m, n] = sum_k A[m, k] D[n, k]
    int rc = launch_sgemm<true, true>(a, K, d, K, (int)M, (int)N, (int)K, 1.0f, r, N, 1, sqp, st);
    if (rc) return rc;
    // G[n, k] = (2 / (M N)) sum_m R[m, n] A[m, k]
    rc = launch_sgemm<false, false>(r, N, a, K, (int)N, (int)K, (int)M, (float)(2.0 / (double)nr), g, K, slices, nullptr, st);
    if (rc) return rc;
    const LossArgs losses{sqp, nsq, (double)nr, regp, bw, (double)nw, loss_out};
    hipLaunchKernelGGL(update, dim3(bw), dim3(256), 0, st, w, sw, alpha, g, slices, nw, (int)K, q, lr,
                       (float)((double)reg_weight / (double)nw), grad_out, losses);
    return hipGetLastError() == hipSuccess ? FPQ_OK : FPQ_ERR_LAUNCH;
}

}  // namespace fpq
