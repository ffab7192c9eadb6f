// The head part of the gated-convolution layer (d_h > 1) without its d_h^2 long convolutions.  Per head and position
//   O[j][t] = sum_i X1~[i][t] sum_s k[t - s] X2~[i][s] V~[j][s]
// and with the sum over i taken first
//   S[s][t] = sum_i X2~[i][s] X1~[i][t],   O[j][t] = sum_s V~[j][s] (k[t - s] S[s][t])
// every (s, t) pair costs two small products of inner length d_h and one multiplication by the kernel, where the
// convolutions cost d_h^2 transforms: at d_h = 16, n = 1024 13 GFLOP per 8 x 48 heads instead of 143.  Both
// products are MFMAs: S leaves the first one with its rows s where the second one wants its contraction index, so k S
// goes from accumulator to operand in registers.
#include "half16.h"
#include "kernels.h"

namespace monarch {

namespace hheads {

using h16::f32x4;
typedef __attribute__((ext_vector_type(4))) short s16x4;

constexpr int TU = 64;       // positions t of a wave: four column tiles
constexpr int PAD = 64;      // zeros before k[0]: the pairs s > t of the tiles on the diagonal

constexpr int ROW = 16;      // features of a position's row, zeros past d_h
constexpr int MIN_DH = 5;    // fewest features of a head, see hyena_heads_supported

__host__ __device__ __forceinline__ int steps(int n) { return (n + 31) / 32; }   // of 32 positions

__device__ __forceinline__ void load8(const float *p, float (&v)[8])
{
    const float4 a = reinterpret_cast<const float4 *>(p)[0], b = reinterpret_cast<const float4 *>(p)[1];
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}
__device__ __forceinline__ void load8(const bf16_t *p, float (&v)[8])
{
    const uint4 w = *reinterpret_cast<const uint4 *>(p);
    const uint32_t d[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        v[2 * e] = h16::lo32<bf16_t>(d[e]);
        v[2 * e + 1] = h16::hi32<bf16_t>(d[e]);
    }
}
__device__ __forceinline__ void store8(float *p, const float (&v)[8])
{
    reinterpret_cast<float4 *>(p)[0] = make_float4(v[0], v[1], v[2], v[3]);
    reinterpret_cast<float4 *>(p)[1] = make_float4(v[4], v[5], v[6], v[7]);
}
__device__ __forceinline__ void store8(bf16_t *p, const float (&v)[8])
{
    *reinterpret_cast<uint4 *>(p) = make_uint4(h16::pack16<bf16_t>(v[0], v[1]), h16::pack16<bf16_t>(v[2], v[3]),
                                               h16::pack16<bf16_t>(v[4], v[5]), h16::pack16<bf16_t>(v[6], v[7]));
}

// The short convolutions of the layer, their results in the order in which the products read them, positions padded to
// whole steps of 32 and features to 16 with zeros.  X1~, X2~: (B, heads, position, feature).  V~: (B, heads, step, g,
// feature, q, e), the position in the step being 16 q + 4 g + e: a lane's operand for a step is 8 consecutive elements
// (as (B, d, n) rows a wave's request touched 16 cache lines for 32 bytes of each: the product kernel 48 us instead of
// 42 us at B = 8, n = 1024, d = 768, d_h = 16).  A workgroup takes whole steps of one head of one of the three; a thread
// 8 consecutive positions of one feature, as the plain kernel.
template <typename T>
__global__ __launch_bounds__(256) void short_conv_kernel(const T *__restrict__ in, T *__restrict__ out, const T *__restrict__ ks,
                                                         const T *__restrict__ bias, int B, int d, int n, int taps, int dh)
{
    __shared__ __attribute__((aligned(16))) T tile[256 / MIN_DH / 4 * 4 * 8 * ROW];
    const int pieces = 256 / dh / 4 * 4, heads = d / dh;
    const int head = blockIdx.y % heads, b = blockIdx.y / heads, i3 = blockIdx.z;
    const int t0 = blockIdx.x * 8 * pieces, positions = 32 * steps(n);
    // neighbouring threads: features of a position (neighbours in the tile)
    const int i = (int)threadIdx.x % dh, p = (int)threadIdx.x / dh, t = t0 + 8 * p;
    const int left = (positions - t0 < 8 * pieces ? positions - t0 : 8 * pieces) * ROW;
    if (dh != ROW || t0 + 8 * pieces > n) {
        for (int e = threadIdx.x; e < left; e += 256) tile[e] = from_f32<T>(0.0f);
        __syncthreads();
    }
    if (p < pieces && t < n) {     // n is a multiple of 8
        const int c = head * dh + i, kr = i3 * d + c;
        float w[8], x[16], cur[8], prev[8];
#pragma unroll
        for (int tau = 0; tau < 8; ++tau) w[tau] = tau < taps ? to_f32(ks[(int64_t)kr * taps + tau]) : 0.0f;
        const float bv = bias ? to_f32(bias[kr]) : 0.0f;
        const T *src = in + (((int64_t)b * 3 + i3) * d + c) * n + t;
        load8(src, cur);
        load8(t > 0 ? src - 8 : src, prev);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            x[8 + e] = cur[e] + bv;
            x[e] = t > 0 ? prev[e] + bv : 0.0f;   // positions before the start of the row contribute nothing
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            float acc = 0.0f;
#pragma unroll
            for (int tau = 0; tau < 8; ++tau) acc = fmaf(w[tau], x[8 + e - tau], acc);
            const int at = 8 * p + e, q = (at >> 4) & 1, g = (at >> 2) & 3;
            tile[i3 < 2 ? at * ROW + i : ((at >> 5) * 64 + g * 16 + i) * 8 + q * 4 + (at & 3)] = from_f32<T>(acc);
        }
    }
    __syncthreads();
    constexpr int PE = 16 / sizeof(T);
    T *dst = out + ((((int64_t)i3 * B + b) * heads + head) * positions + t0) * ROW;
    for (int e = threadIdx.x * PE; e < left; e += 256 * PE) *reinterpret_cast<uint4 *>(dst + e) = *reinterpret_cast<const uint4 *>(tile + e);
}

// four features 4 g .. 4 g + 3 of a position
template <typename T> struct Frag;
template <> struct Frag<bf16_t> { typedef s16x4 type; };
template <> struct Frag<float> { typedef f32x4 type; };
template <typename F, typename T> __device__ __forceinline__ F load4(const T *p) { return *reinterpret_cast<const F *>(p); }

__device__ __forceinline__ f32x4 dot(s16x4 a, s16x4 b)
{
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, f32x4{0, 0, 0, 0}, 0, 0, 0);
}
__device__ __forceinline__ f32x4 dot(f32x4 a, f32x4 b)
{
    f32x4 c = {0, 0, 0, 0};   // contraction index of MFMA e: feature 4 g + e
#pragma unroll
    for (int e = 0; e < 4; ++e) c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], b[e], c, 0, 0, 0);
    return c;
}
// acc += V (two tiles of 16 positions s) times p: slot (g, e) of the contraction is position 4 g + e of its tile
__device__ __forceinline__ f32x4 apply(s16x4 v0, s16x4 v1, f32x4 p0, f32x4 p1, f32x4 acc)
{
    const uint2 a0 = __builtin_bit_cast(uint2, v0), a1 = __builtin_bit_cast(uint2, v1);
    const h16::op8 a = {a0.x, a0.y, a1.x, a1.y};
    const h16::op8 b = {h16::pack16<bf16_t>(p0[0], p0[1]), h16::pack16<bf16_t>(p0[2], p0[3]), h16::pack16<bf16_t>(p1[0], p1[1]),
                        h16::pack16<bf16_t>(p1[2], p1[3])};
    return h16::mfma<bf16_t>(a, b, acc);
}
__device__ __forceinline__ f32x4 apply(f32x4 v0, f32x4 v1, f32x4 p0, f32x4 p1, f32x4 acc)
{
#pragma unroll
    for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(v0[e], p0[e], acc, 0, 0, 0);
#pragma unroll
    for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(v1[e], p1[e], acc, 0, 0, 0);
    return acc;
}

// o[b][head d_h + j][t].  A wave takes 64 positions t of one (batch entry, head) and walks over s <= t in steps of 32
// (two row tiles).  The four waves of a workgroup share the head's kernel, held in LDS in fp32, and take the same t of
// different batch entries (equally long sums), the longest sums first and neighbouring workgroups different heads (with
// the t of a head in neighbouring workgroups two of the eight XCDs had all the longest sums: 72 against 48 us).  A
// lane's four kernel values of a tile pair depend on the distance of the tiles only: of the five distances of a step
// three are those of the step before, so a step reads two (8 words) from LDS for its 32 x 64 pairs.  Bounds at B = 8,
// n = 1024, d = 768, d_h = 16, bf16 (27 us, against 188 us for the convolutions and the sum over i): vector instructions
// (15 us: one multiplication per pair, half a conversion), then MFMA (8 us) and 50 MB of operands and results (10 us).
template <typename T>
__global__ __launch_bounds__(256, sizeof(T) == 4 ? 2 : 4) void heads_kernel(const T *__restrict__ x12v, const T *__restrict__ k, T *__restrict__ o, int B, int d,
                                                       int n, int klen, int dh)
{
    typedef typename Frag<T>::type F;
    extern __shared__ __attribute__((aligned(16))) float kz[];   // PAD zeros, k, zeros up to lag n + 63
    const int heads = d / dh, head = blockIdx.x, units = (n + TU - 1) / TU;
    const int longest = (units - 1 - (int)(blockIdx.y * 4 / B)) * TU;   // t0 of the first wave
    for (int e = threadIdx.x; e < longest + TU + PAD; e += 256) {
        const int lag = e - PAD;
        kz[e] = lag >= 0 && lag < klen ? to_f32(k[(int64_t)head * klen + lag]) : 0.0f;
    }
    __syncthreads();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, l16 = lane & 15, g = lane >> 4;
    const int unit = blockIdx.y * 4 + wave;
    if (unit >= B * units) return;
    const int b = unit % B, t0 = (units - 1 - unit / B) * TU;
    const int64_t plane = (int64_t)B * heads * steps(n) * (32 * ROW);
    const T *x1 = x12v + ((int64_t)b * heads + head) * steps(n) * (32 * ROW);
    F xf[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        int t = t0 + 16 * c + l16;
        if (t >= n) t = n - 1;   // (positions past the end: computed, never stored)
        xf[c] = load4<F>(x1 + t * ROW + 4 * g);
    }
    f32x4 acc[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[c] = f32x4{0, 0, 0, 0};
    const T *xs_at = x1 + plane + l16 * ROW + 4 * g, *vs_at = x1 + 2 * plane + 8 * lane;
    auto request = [&](int s0, F (&xs)[2], F (&vs)[2]) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            xs[q] = load4<F>(xs_at + (s0 + 16 * q) * ROW);
            vs[q] = load4<F>(vs_at + s0 * ROW + 4 * q);
        }
    };
    // the first s that a position of the unit reaches, in whole steps; the last one
    int s_begin = t0 - klen + 1;
    s_begin = s_begin > 0 ? s_begin / 32 * 32 : 0;
    const int s_end = t0 + TU < n ? t0 + TU : n;
    // kf[m]: the kernel values of tiles at distance 16 (m - 1) of the step, m - 1 = column tile - row tile
    f32x4 kf[5];
    auto kernel_values = [&](int lag) {   // lag of column l16 against row 0: row 4 g + r lies 4 g + r before it
        const float *q = kz + PAD + lag + l16 - 4 * g;
        return f32x4{q[0], q[-1], q[-2], q[-3]};
    };
#pragma unroll
    for (int m = 0; m < 3; ++m) kf[m] = kernel_values(t0 - s_begin + 16 * (m + 1));
    // a step's operands are requested three steps ahead (requested one step ahead, with the registers copied at the
    // step's end, a wave waited for L2 in every step: 42 instead of 27 us)
    F xs[4][2], vs[4][2];
    const int last = s_begin + (s_end - 1 - s_begin) / 32 * 32;
#pragma unroll
    for (int m = 0; m < 3; ++m) request(s_begin + 32 * m < s_end ? s_begin + 32 * m : last, xs[m], vs[m]);
    for (int s4 = s_begin; s4 < s_end; s4 += 128) {
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            const int s0 = s4 + 32 * m;
            request(s0 + 96 < s_end ? s0 + 96 : last, xs[(m + 3) & 3], vs[(m + 3) & 3]);
            if (s0 < s_end) {
                kf[4] = kf[2]; kf[3] = kf[1]; kf[2] = kf[0];
                kf[1] = kernel_values(t0 - s0);
                kf[0] = kernel_values(t0 - s0 - 16);
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const f32x4 p0 = dot(xs[m][0], xf[c]) * kf[c + 1], p1 = dot(xs[m][1], xf[c]) * kf[c];
                    acc[c] = apply(vs[m][0], vs[m][1], p0, p1, acc[c]);
                }
            }
        }
    }
    // rows j = 4 g + r of the accumulator, column t
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const int t = t0 + 16 * c + l16;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int j = 4 * g + r;
            if (j < dh && t < n) o[((int64_t)b * d + head * dh + j) * n + t] = from_f32<T>(acc[c][r]);
        }
    }
}

template <typename T>
static int run(const void *proj, void *x12v, void *o, const void *k_short, const void *b_in, const void *k_long, int B, int d, int n,
               int taps, int klen, int dh, hipStream_t s)
{
    const int heads = d / dh, tb = 256 / dh / 4 * 32;
    hipLaunchKernelGGL(short_conv_kernel<T>, dim3((n + tb - 1) / tb, B * heads, 3), dim3(256), 0, s, (const T *)proj, (T *)x12v,
                       (const T *)k_short, (const T *)b_in, B, d, n, taps, dh);
    MONARCH_HIP_CHECK(hipGetLastError());
    const int64_t units = (int64_t)B * ((n + TU - 1) / TU);
    hipLaunchKernelGGL(heads_kernel<T>, dim3(heads, (unsigned)((units + 3) / 4)), dim3(256), sizeof(float) * (n + 2 * PAD), s,
                       (const T *)x12v, (const T *)k_long, (T *)o, B, d, n, klen, dh);
    MONARCH_HIP_CHECK(hipGetLastError());
    return MONARCH_OK;
}

}  // namespace hheads

// The work is n^2 per head here and d_h^2 transforms there.  Whole layer, us, convolutions against this kernel, d = 768 (640 at
// d_h = 5), B n = 8192:
//   bf16   d_h = 16       8            6            5            fp32   d_h = 16       12           8            6
//   n =  128   327 : 134    220 : 154    197 : 165    144 : 135      745 :  391    648 : 407    555 : 429    508 : 459
//        512   532 : 114    312 : 129    256 : 151    197 : 143      771 :  405    666 : 429    560 : 472    509 : 528
//       1024   279 : 120    184 : 140    164 : 169    132 : 152      772 :  444    667 : 476    559 : 548    506 : 638
//       2048   477 : 139    305 : 173    253 : 198    191 : 185      767 :  525    662 : 581    557 : 726    501 : 864
//       4096   578 : 178    348 : 236    291 : 280    223 : 262     1080 :  806    905 : 914    744 : 1183   663 : 1438
//       8192  1348 : 253    441 : 362    309 : 439    237 : 419     3792 : 1135   2954 : 1336  2106 : 1864  1686 : 2379
// bf16, and fp32 beyond the convolution kernel of one launch (n = 8192; n = 4200, d_h = 8, d = 256 1125 : 362; splits whose rows it
// takes one by one): from 8 features on always, from 5 on up to n = 512.  fp32 within that kernel: n < 2 d_h^3, which
// parts the table and what lies between (d_h = 10: n = 1024 684 : 521, 2048 663 : 653; 7: 512 591 : 515; 6: 256 518 : 475;
// 5: 128 111 : 109, 256 377 : 377); at B = 1 the line lies a little lower (8: 1024 111 : 128, 12: 2048 187 : 205).  With
// 4 features (rows padded to 4) an earlier form gained nothing at n = 128 and lost from n = 1024 on (bf16 147 : 280).
// (The bf16 convolutions of 512 points, n = 136 to 256, and those of 1024 and 4096 with few rows have become up to twice as fast since; the table has
// none of them but with many rows, and the line of 5 to 7 features was not drawn again.)
bool hyena_heads_supported(int B, int n, int d, int klen, int nfft, const int *factors, int nf, int head_dim, monarch_dtype dt)
{
    if (conv_fft_supported(nfft) && fft_mfma_f32_supported(nfft, factors, nf, dt)) {
        if (n >= 2 * head_dim * head_dim * head_dim) return false;
    } else if (head_dim < 8 && n > 512) return false;
    if (head_dim < hheads::MIN_DH || head_dim > hheads::ROW || n < 8 || n % 8 || n > 8192) return false;
    if ((int64_t)n + klen - 1 > nfft) return false;   // a circular convolution that wraps
    return (int64_t)B * (d / head_dim) <= 65535 && (int64_t)B * ((n + hheads::TU - 1) / hheads::TU) <= 4 * 65535;
}

size_t hyena_heads_bytes(int B, int n, int d, int head_dim, monarch_dtype dt)
{
    return 3 * (size_t)B * (d / head_dim) * hheads::steps(n) * (32 * hheads::ROW) * dtype_size(dt);
}

int launch_hyena_heads(const void *proj, void *x12v, void *o, const void *k_short, const void *b_in, const void *k_long, int B, int d,
                       int n, int taps, int klen, int dh, monarch_dtype dt, hipStream_t s)
{
    if (dt == MONARCH_F32) return hheads::run<float>(proj, x12v, o, k_short, b_in, k_long, B, d, n, taps, klen, dh, s);
    return hheads::run<bf16_t>(proj, x12v, o, k_short, b_in, k_long, B, d, n, taps, klen, dh, s);
}

}  // namespace monarch
