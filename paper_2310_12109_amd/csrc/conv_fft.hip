// Fused gated convolution, fp32 arithmetic on tensors of any element type, for transform lengths 256 .. 8192 (powers of two),
// on the vector unit:
//   y = g_out o (F^-1 (F k' o F (g_in o u)'))[0 : n]
// Two rows of a channel (batch entries 2 p, 2 p + 1) are one complex row z = x0 + i x1 (the kernel is real), or one row
// fills both parts (per = 1); a slot of N / A threads holds it in registers, A values per thread, from the loads to the stores.  The Monarch factors of
// the transform are A, 16 and R (N = A 16 R): with t the thread, t = t2 + R j2,
//   over j  (n = t + 16 R j):  X1[k1][t]      times w_N^(t k1)
//   over j2:                   X2[k1][k2][t2] times w_(16 R)^(t2 k2)
//   over t2:                   X3[k1][k2][k3], frequency k1 + A k2 + 16 A k3, left where it is
// and the inverse runs the same steps backwards on conj(Z k_f) (conj o F o conj), so no permutation exists in either
// direction.  A factor of 16 or 32 is itself taken as 4 x 4 (x 2) in registers: 144 additions and 10 complex
// multiplications instead of the 256 multiply-adds of the dense factor, which is why this unit beats the fp32
// matrix instruction here (64 x 64 in two MFMA passes: 70 us of matrix products alone at the shape below; its error
// is also smaller).  Between the factors the values change threads through LDS: one exchange inside a wave (a k1 belongs to
// R neighbouring lanes), one across the slot, in padded layouts without bank conflicts: two barriers per pair of rows, and one
// after the kernel's spectrum, whose transform leaves the waves at work on their rows of LDS.
// B = 7, H = 384, n = 2004, N = 4096, both gates: 34 us (six MFMA passes through memory: 171), of it 17 us the rows at
// the rate of a copy and about as much vector instructions (1300 per thread and pair, 3 waves per SIMD); the two
// overlap only between workgroups.  B = 8, H = 768, n = 1024, N = 2048: 36 us (a 64 x 32 MFMA kernel: 75).  16-bit tensors,
// where no MFMA kernel of one launch takes the call: bf16, B = 37, H = 384, n = 136, N = 512: 21 us (passes through memory: 47); B = 8, H = 768, n = 1015, N = 2048: 34 (three chunk launches: 46);
// fp16, B = 8, H = 768, n = 1016, a circular kernel, N = 2048: 51 (shape-generic passes: 2307).  Three
// waves per SIMD: with 128 registers (four) the twiddles held in registers spill, 34 -> 47 us.  N = 8192 takes 32
// values per thread and one wave per SIMD: 84 us at B = 2, H = 768, n = 4096 (passes: 293), 98 with two waves and spills.
#include "const_roots.h"
#include "kernels.h"

namespace monarch {

namespace cfft {

template <int A, int R> struct Geo {
    static constexpr int M = 16 * R, N = A * M, T = M, U = A / 16;          // U: (k1, t2) problems of a thread
    static constexpr int SLOTS = T >= 256 ? 1 : 256 / T, THREADS = T * SLOTS;
    // float2 pitches of k1 and k2 and of a slot: no two lanes of a half wave in the same bank pair, for each access below
    static constexpr int Q = R == 1 ? 1 : R == 2 ? 3 : R + 1;
    static constexpr int P = R == 1 ? 17 : R == 2 ? 50 : R == 4 ? 84 : R == 8 ? 152 : 272;
    static constexpr int SLOT = A * P;
    static constexpr size_t LDS_BYTES = sizeof(float2) * (SLOTS * SLOT + M);
};

// w_N^(t k1), t < M, by [k1][t]: a wave reads consecutive entries
template <int A, int R> struct Twiddles { float2 w[A][16 * R]; };
template <int A, int R> constexpr Twiddles<A, R> make_twiddles()
{
    Twiddles<A, R> t{};
    for (int k = 0; k < A; ++k)
        for (int i = 0; i < 16 * R; ++i) {
            const croots::CosSin r = croots::unit_root(k * i, A * 16 * R);
            t.w[k][i].x = (float)r.c;
            t.w[k][i].y = (float)-r.s;
        }
    return t;
}
template <int A, int R> __device__ const Twiddles<A, R> g_twiddles = make_twiddles<A, R>();

__device__ __forceinline__ float2 operator+(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float2 operator-(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ float2 minus_i(float2 a) { return make_float2(a.y, -a.x); }
__device__ __forceinline__ float2 times(float2 a, float2 b)
{
    return make_float2(fmaf(a.x, b.x, -(a.y * b.y)), fmaf(a.x, b.y, a.y * b.x));
}
// exp(-2 pi i e / 32), a compile-time constant after unrolling
__device__ __forceinline__ float2 w32(int e)
{
    constexpr float c[9] = {1.0f, 0.98078528040323044913f, 0.92387953251128675613f, 0.83146961230254523708f, 0.70710678118654752440f,
                            0.55557023301960222474f, 0.38268343236508977173f, 0.19509032201612826785f, 0.0f};
    e &= 31;
    const int q = e >> 3, r = e & 7;   // quadrant, angle in it
    const float co = c[r], si = c[8 - r];
    return q == 0 ? make_float2(co, -si) : q == 1 ? make_float2(-si, -co) : q == 2 ? make_float2(-co, si) : make_float2(si, co);
}
__device__ __forceinline__ float2 turn(float2 v, int e)   // times exp(-2 pi i e / 32), e known at compile time
{
    e &= 31;
    if (e == 0) return v;
    if (e == 8) return minus_i(v);
    if (e == 16) return make_float2(-v.x, -v.y);
    if (e == 4) return make_float2(0.70710678118654752440f * (v.x + v.y), 0.70710678118654752440f * (v.y - v.x));
    if (e == 12) return make_float2(0.70710678118654752440f * (v.y - v.x), -0.70710678118654752440f * (v.x + v.y));
    return times(v, w32(e));
}

template <bool LOW> __device__ __forceinline__ void dft4(float2 &a, float2 &b, float2 &c, float2 &d)   // LOW: c = d = 0
{
    if constexpr (LOW) {
        const float2 s = a, t = b;
        a = s + t; b = s + minus_i(t); c = s - t; d = s - minus_i(t);
    } else {
        const float2 s = a + c, t = a - c, u = b + d, v = minus_i(b - d);
        a = s + u; b = t + v; c = s - u; d = t - v;
    }
}
// in place, natural order in and out; LOW: the upper half of the input is zero (and is not read)
template <int L, bool LOW = false> __device__ __forceinline__ void dft(float2 (&x)[L])
{
    if constexpr (L == 2) {
        const float2 a = x[0];
        x[0] = a + x[1]; x[1] = a - x[1];
    } else if constexpr (L == 4) {
        dft4<LOW>(x[0], x[1], x[2], x[3]);
    } else if constexpr (L == 8) {
        float2 a[4] = {x[0], x[2], x[4], x[6]}, b[4] = {x[1], x[3], x[5], x[7]};
        dft<4, LOW>(a); dft<4, LOW>(b);
#pragma unroll
        for (int k = 0; k < 4; ++k) { const float2 t = turn(b[k], 4 * k); x[k] = a[k] + t; x[k + 4] = a[k] - t; }
    } else if constexpr (L == 16) {
        float2 y[4][4];   // [b][ka]
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            y[b][0] = x[b]; y[b][1] = x[b + 4]; y[b][2] = x[b + 8]; y[b][3] = x[b + 12];
            dft4<LOW>(y[b][0], y[b][1], y[b][2], y[b][3]);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            float2 v[4];
#pragma unroll
            for (int b = 0; b < 4; ++b) v[b] = turn(y[b][k], 2 * b * k);
            dft4<false>(v[0], v[1], v[2], v[3]);
#pragma unroll
            for (int q = 0; q < 4; ++q) x[k + 4 * q] = v[q];
        }
    } else {
        static_assert(L == 32, "");
        float2 a[16], b[16];   // even and odd outputs
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            a[j] = LOW ? x[j] : x[j] + x[j + 16];
            b[j] = turn(LOW ? x[j] : x[j] - x[j + 16], j);
        }
        dft<16>(a); dft<16>(b);
#pragma unroll
        for (int j = 0; j < 16; ++j) { x[2 * j] = a[j]; x[2 * j + 1] = b[j]; }
    }
}

// HALF: n <= N / 2 and klen <= N / 2 (zero padding): the upper half of the loads and of the outputs does not exist.
template <typename E, int A, int R, bool HALF, bool GIN, bool GOUT>
__global__ __launch_bounds__((Geo<A, R>::THREADS), (A == 32 ? 1 : 3)) void conv_kernel(
    const E *__restrict__ u, const E *__restrict__ k, const E *__restrict__ g_in, const E *__restrict__ g_out,
    E *__restrict__ y, int B, int H, int n, int klen, int per, int splits, int items)
{
    typedef Geo<A, R> G;
    constexpr int M = G::M, T = G::T, U = G::U, P = G::P, Q = G::Q, JN = HALF ? A / 2 : A, PR = 16 / R;
    extern __shared__ __attribute__((aligned(16))) float2 lds[];
    const int t = threadIdx.x % T, slot = threadIdx.x / T;
    float2 *buf = lds + slot * G::SLOT, *tw2 = lds + G::SLOTS * G::SLOT;   // tw2: w_M^(t2 k2) at k2 R + t2
    if (threadIdx.x < M) tw2[threadIdx.x] = g_twiddles<A, R>.w[U * (threadIdx.x / R)][16 * (threadIdx.x % R)];   // w_N^(A t2 k2)
    const int64_t item = (int64_t)blockIdx.x * G::SLOTS + slot;
    const bool live_item = item < items;
    const int h = live_item ? (int)(item % H) : 0, split = live_item ? (int)(item / H) : 0;
    const int pairs = per == 2 ? (B + 1) / 2 : B;   // complex rows of a channel
    __syncthreads();

    // forward transform of v (value n = t + M j in v[j]) into z[unit][m R + k3].  It begins by storing to every k1 row of the
    // slot's buffer, so no wave of the slot may still be at work on a row there; it ends while the waves are, each on
    // its own rows.
    auto forward = [&](float2 (&v)[A], float2 (&z)[U][16]) {
        dft<A, HALF>(v);
#pragma unroll
        for (int k1 = 1; k1 < A; ++k1) v[k1] = times(v[k1], g_twiddles<A, R>.w[k1][t]);
#pragma unroll
        for (int k1 = 0; k1 < A; ++k1) buf[k1 * P + t] = v[k1];
        __syncthreads();
#pragma unroll
        for (int w = 0; w < U; ++w) {
            const int id = t + T * w, k1 = id / R, t2 = id % R;
            float2 *mine = buf + k1 * P;
            float2 (&x)[16] = z[w];
#pragma unroll
            for (int j = 0; j < 16; ++j) x[j] = mine[t2 + R * j];
            dft<16>(x);
            if constexpr (R > 1) {
#pragma unroll
                for (int k2 = 1; k2 < 16; ++k2) x[k2] = times(x[k2], tw2[k2 * R + t2]);
                // (the R lanes of a k1 are neighbours in one wave, whose LDS accesses stay in order)
#pragma unroll
                for (int k2 = 0; k2 < 16; ++k2) mine[k2 * Q + t2] = x[k2];
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int m = 0; m < PR; ++m) {
                    float2 s[R];
#pragma unroll
                    for (int e = 0; e < R; ++e) s[e] = mine[(t2 + R * m) * Q + e];
                    dft<R>(s);
#pragma unroll
                    for (int e = 0; e < R; ++e) x[m * R + e] = s[e];
                }
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
            }
        }
    };
    // the same backwards: z -> v (values n = t + M j in v[j])
    auto backward = [&](float2 (&z)[U][16], float2 (&v)[A]) {
#pragma unroll
        for (int w = 0; w < U; ++w) {
            const int id = t + T * w, k1 = id / R, t2 = id % R;
            float2 *mine = buf + k1 * P;
            float2 (&x)[16] = z[w];
            if constexpr (R > 1) {
#pragma unroll
                for (int m = 0; m < PR; ++m) {
                    float2 s[R];
#pragma unroll
                    for (int e = 0; e < R; ++e) s[e] = x[m * R + e];
                    dft<R>(s);
#pragma unroll
                    for (int e = 0; e < R; ++e) mine[(t2 + R * m) * Q + e] = s[e];
                }
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int k2 = 0; k2 < 16; ++k2) x[k2] = mine[k2 * Q + t2];
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int k2 = 1; k2 < 16; ++k2) x[k2] = times(x[k2], tw2[k2 * R + t2]);
            }
            dft<16>(x);
#pragma unroll
            for (int j = 0; j < 16; ++j) mine[t2 + R * j] = x[j];
        }
        __syncthreads();
        // (the rows are free, and a thread reads just the places that it will itself write in the next forward transform: no
        // barrier before that one)
#pragma unroll
        for (int k1 = 0; k1 < A; ++k1) v[k1] = buf[k1 * P + t];
#pragma unroll
        for (int k1 = 1; k1 < A; ++k1) v[k1] = times(v[k1], g_twiddles<A, R>.w[k1][t]);
        dft<A>(v);
    };

    float2 v[A], kf[U][16];
#pragma unroll
    for (int j = 0; j < A; ++j) {
        const int i = t + M * j;
        v[j] = make_float2(j < JN && i < klen ? to_f32(k[(int64_t)h * klen + i]) : 0.0f, 0.0f);
    }
    forward(v, kf);
#pragma unroll
    for (int w = 0; w < U; ++w)
#pragma unroll
        for (int e = 0; e < 16; ++e) kf[w][e] = make_float2(kf[w][e].x * (1.0f / G::N), kf[w][e].y * (1.0f / G::N));
    __syncthreads();   // forward after forward: every wave has left its rows (all slots, whether live or not)

    for (int p = split; p - split < pairs; p += splits) {   // as many rounds for every slot of the workgroup
        const bool live = live_item && p < pairs;
        if constexpr (G::SLOTS == 1) {
            if (!live) break;
        }
        const int b0 = live ? per * p : 0;
        const bool two = per == 2 && b0 + 1 < B;
        const int64_t r0 = ((int64_t)b0 * H + h) * n, r1 = two ? r0 + (int64_t)H * n : r0;
        // (requested here and not a pair ahead: the 32 more registers spill at three workgroups per compute unit, 34 -> 43 us)
#pragma unroll
        for (int j = 0; j < A; ++j) {
            const int i = t + M * j;
            v[j] = make_float2(0.0f, 0.0f);
            if (j < JN && i < n) {
                v[j] = make_float2(to_f32(u[r0 + i]), to_f32(u[r1 + i]));
                if (GIN) v[j] = make_float2(v[j].x * to_f32(g_in[r0 + i]), v[j].y * to_f32(g_in[r1 + i]));
            }
        }
        float2 z[U][16];
        forward(v, z);
#pragma unroll
        for (int w = 0; w < U; ++w)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const float2 q = times(z[w][e], kf[w][e]);
                z[w][e] = make_float2(q.x, -q.y);
            }
        backward(z, v);
        if (live) {
#pragma unroll
            for (int j = 0; j < JN; ++j) {
                const int i = t + M * j;
                if (i < n) {
                    y[r0 + i] = from_f32<E>(GOUT ? v[j].x * to_f32(g_out[r0 + i]) : v[j].x);
                    if (two) y[r1 + i] = from_f32<E>(GOUT ? -v[j].y * to_f32(g_out[r1 + i]) : -v[j].y);
                }
            }
        }
    }
}

template <typename E, int A, int R>
static int launch(const E *u, const E *k, const E *g_in, const E *g_out, E *y, int B, int H, int n, int klen,
                  int per, hipStream_t s)
{
    typedef Geo<A, R> G;
    // a slot transforms its channel's kernel once and then takes the pairs split, split + splits, ...: as many splits of a
    // channel's pairs as give every compute unit its three workgroups
    const int pairs = per == 2 ? (B + 1) / 2 : B;
    int64_t splits = ((int64_t)768 * G::SLOTS + H - 1) / H;
    if (splits > pairs) splits = pairs;
    const int64_t items = splits * H;
    if (items > INT32_MAX) return fail(MONARCH_ESHAPE, "B*H too large for one launch");
    const unsigned grid = (unsigned)((items + G::SLOTS - 1) / G::SLOTS);
    const bool half = n <= G::N / 2 && klen <= G::N / 2;
#define MONARCH_CFFT(HALF, GI, GO)                                                                                              \
    do {                                                                                                                        \
        auto kern = conv_kernel<E, A, R, HALF, GI, GO>;                                                                            \
        if (G::LDS_BYTES > 65536)                                                                                               \
            MONARCH_HIP_CHECK(hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)G::LDS_BYTES)); \
        hipLaunchKernelGGL(kern, dim3(grid), dim3(G::THREADS), G::LDS_BYTES, s, u, k, g_in, g_out, y, B, H, n, klen, per, (int)splits, (int)items); \
    } while (0)
    switch ((half ? 4 : 0) | (g_in ? 2 : 0) | (g_out ? 1 : 0)) {
    case 7: MONARCH_CFFT(true, true, true); break;
    case 6: MONARCH_CFFT(true, true, false); break;
    case 5: MONARCH_CFFT(true, false, true); break;
    case 4: MONARCH_CFFT(true, false, false); break;
    case 3: MONARCH_CFFT(false, true, true); break;
    case 2: MONARCH_CFFT(false, true, false); break;
    case 1: MONARCH_CFFT(false, false, true); break;
    default: MONARCH_CFFT(false, false, false); break;
    }
#undef MONARCH_CFFT
    MONARCH_HIP_CHECK(hipGetLastError());
    return MONARCH_OK;
}

}  // namespace cfft

bool conv_fft_supported(int nfft)
{
    return nfft >= 256 && nfft <= 8192 && (nfft & (nfft - 1)) == 0;
}

template <typename E>
static int launch_conv_fft_as(const void *u, const void *k, const void *g_in, const void *g_out, void *y, int B, int H, int n, int klen,
                              int nfft, int per, hipStream_t s)
{
    const E *ue = (const E *)u, *ke = (const E *)k, *gi = (const E *)g_in, *go = (const E *)g_out;
    E *ye = (E *)y;
    switch (nfft) {
    case 256: return cfft::launch<E, 16, 1>(ue, ke, gi, go, ye, B, H, n, klen, per, s);
    case 512: return cfft::launch<E, 16, 2>(ue, ke, gi, go, ye, B, H, n, klen, per, s);
    case 1024: return cfft::launch<E, 16, 4>(ue, ke, gi, go, ye, B, H, n, klen, per, s);
    case 2048: return cfft::launch<E, 16, 8>(ue, ke, gi, go, ye, B, H, n, klen, per, s);
    case 4096: return cfft::launch<E, 16, 16>(ue, ke, gi, go, ye, B, H, n, klen, per, s);
    default: return cfft::launch<E, 32, 16>(ue, ke, gi, go, ye, B, H, n, klen, per, s);
    }
}

int launch_conv_fft(const void *u, const void *k, const void *g_in, const void *g_out, void *y, int B, int H, int n, int klen,
                    int nfft, int per, monarch_dtype dt, hipStream_t s)
{
    if (dt == MONARCH_F32) return launch_conv_fft_as<float>(u, k, g_in, g_out, y, B, H, n, klen, nfft, per, s);
    if (dt == MONARCH_BF16) return launch_conv_fft_as<bf16_t>(u, k, g_in, g_out, y, B, H, n, klen, nfft, per, s);
    return launch_conv_fft_as<f16_t>(u, k, g_in, g_out, y, B, H, n, klen, nfft, per, s);
}

}  // namespace monarch
