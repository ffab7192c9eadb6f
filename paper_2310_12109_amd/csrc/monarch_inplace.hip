// Square order-2 Monarch products with blocks of 32 x 32 or 64 x 64 (N = 1024 or 4096) on the fp32 matrix
// instruction (16x16x4), fp32 or bf16 tensors, fp32 arithmetic:
//   monarch_matmul   y = P L P R P x                                    (Sec. 3.1)
//   monarch_mixer    y = g_out o M2 (K o M1 (g_in o u))                  (Sec. 3.2 Eq. 2 in its gated form)
//   monarch_matmul_backward                  dx = M^T dy, dR, dL            (what training the matrices of Sec. 3.1 needs)
// A workgroup holds a tile of rows in LDS (element hi b + lo of a row at hi SH + lo) and every block-diagonal
// factor works IN PLACE: block k reads the b elements of a row that it contracts (one digit of the index, the other
// digit being the block's number) and writes its b results to the same places.  With x at (c, k):
//   R: block k contracts c (stride SH)  ->  (r, k);     L: block r contracts k (stride 1)  ->  (r, s) = y[s b + r]
// so the three permutations of M = P L P R P cost nothing and the product ends transposed in the tile.  The mixer's
// second matrix takes that layout as it is (R2: block k' = s contracts c' = r with stride 1, L2: block r' contracts
// k' with stride SH) and ends in natural order.  Rows sit on the MFMA column index.  The factors (b^3 elements each) stay
// in L2 and are read as the A operand, 16 bytes per lane, a ring of requests ahead of the products.  bf16 factors meet the
// fp32 values of the tile on the bf16 instruction, the values split into three bf16 parts: 16384 rows of b = 32 through the
// mixer (the two halves of an M2 layer of 16 x 1024 x 1024) 77 and 90 us -> 45 and 50 us with the ring, the pitches, one
// index division per tile instead of one per piece and, for transposed rows, neighbouring tiles on one XCD (277 -> 103 MB
// past L2).  What is left: vector instructions (18 and 26 us, half of them the splitting), LDS (11 us), memory (13 us).
// fp32 (12288 rows, both gates): 89 -> 83 us, all workgroups loading, multiplying and storing at the same time.
#include "half16.h"
#include "kernels.h"

namespace monarch {

namespace inpl {

typedef __attribute__((ext_vector_type(4))) float f32x4;

__device__ __forceinline__ f32x4 mfma(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
__device__ __forceinline__ f32x4 ld4(const float *p) { return *reinterpret_cast<const f32x4 *>(p); }
__device__ __forceinline__ f32x4 ld4(const bf16_t *p)
{
    const uint2 w = *reinterpret_cast<const uint2 *>(p);
    return f32x4{__uint_as_float(w.x << 16), __uint_as_float(w.x & 0xffff0000u), __uint_as_float(w.y << 16),
                 __uint_as_float(w.y & 0xffff0000u)};
}
__device__ __forceinline__ float ld1(const float *p) { return *p; }
__device__ __forceinline__ float ld1(const bf16_t *p) { return __uint_as_float((uint32_t)*reinterpret_cast<const uint16_t *>(p) << 16); }
__device__ __forceinline__ void st4(float *p, f32x4 v) { *reinterpret_cast<f32x4 *>(p) = v; }
// the same for rows that a launch reads or writes once, a wave instruction covering whole cache lines: streaming
// accesses (the plain product: -4.8 % at b = 32, -3.5 % at b = 64 in fp32; the mixer kernel keeps ordinary accesses:
// with the layer's transposed pieces, which take a cache line in several instructions, streaming cost 11 %)
__device__ __forceinline__ f32x4 ld4s(const float *p) { return __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(p)); }
__device__ __forceinline__ f32x4 ld4s(const bf16_t *p)
{
    const uint2 w = load_stream8(p);
    return f32x4{__uint_as_float(w.x << 16), __uint_as_float(w.x & 0xffff0000u), __uint_as_float(w.y << 16),
                 __uint_as_float(w.y & 0xffff0000u)};
}
__device__ __forceinline__ void st4s(float *p, f32x4 v) { __builtin_nontemporal_store(v, reinterpret_cast<f32x4 *>(p)); }
__device__ __forceinline__ void st4(bf16_t *p, f32x4 v)
{
    const bf16_t h[4] = {from_f32<bf16_t>(v[0]), from_f32<bf16_t>(v[1]), from_f32<bf16_t>(v[2]), from_f32<bf16_t>(v[3])};
    *reinterpret_cast<uint2 *>(p) = *reinterpret_cast<const uint2 *>(h);
}
__device__ __forceinline__ void st4s(bf16_t *p, f32x4 v)
{
    const bf16_t h[4] = {from_f32<bf16_t>(v[0]), from_f32<bf16_t>(v[1]), from_f32<bf16_t>(v[2]), from_f32<bf16_t>(v[3])};
    store_stream8(p, *reinterpret_cast<const uint2 *>(h));
}

// b = 32: tiles of 16 rows (78 KB: two workgroups of 8 waves per compute unit); b = 64: tiles of 8 rows (133 KB, one
// workgroup of 16 waves; columns 8..15 of the MFMA repeat the rows).  The pitches SH (of the high digit) and ROWP (of a row)
// have the fewest LDS passes of all pairs up to SH = b + 8 over the accesses below, 64 banks: per tile of the mixer 5632
// at b = 32 (8192 with 36, 1153), 10240 at b = 64 (20480 with 68, 4353).
template <int BS>
struct Geo {
    static constexpr int N = BS * BS, SH = BS == 32 ? 38 : 65, TV = BS == 32 ? 16 : 8, ROWP = BS == 32 ? 1225 : 4169;
    static constexpr int THREADS = BS == 32 ? 512 : 1024, WAVES = THREADS / 64, NBW = BS / WAVES;
    static constexpr int Q = BS / 4, RT = BS / 16;   // contraction indices per lane group; row tiles of a block
    static constexpr size_t LDS_BYTES = sizeof(float) * TV * ROWP;
};

// The blocks' matrices on their way from L2: a wave's items of a stage are (block, row tile) pairs; DEPTH of them (32
// registers) are requested ahead, the first ones of a stage before the barrier in front of it.  One item ahead, every
// stage began and went on by waiting for L2.
//   fp32 (and transposed blocks): 16x16x4 MFMAs, lane (row i, group g) holds columns (b/4) g .. of its row
//   bf16: 16x16x32 MFMAs, lane (row i, group g) holds columns 32 c + 8 g .. of its row for every c < b / 32
template <typename T, bool TRANS> constexpr bool kHalf = sizeof(T) == 2 && !TRANS;
template <typename T, int BS, bool TRANS = false>
struct Ring {
    static constexpr bool HALF = kHalf<T, TRANS>;
    static constexpr int WV = HALF ? BS / 32 : BS / 16, DEPTH = HALF && BS == 64 ? 2 : 8 / WV, ITEMS = Geo<BS>::NBW * Geo<BS>::RT;
    f32x4 w[DEPTH][WV];
};

template <typename T, int BS, bool TRANS>
__device__ __forceinline__ void request_at(const T *__restrict__ src, int blk, int rt, int lane, f32x4 (&dst)[Ring<T, BS, TRANS>::WV])
{
    typedef Geo<BS> G;
    constexpr int WV = Ring<T, BS, TRANS>::WV;
    const int l16 = lane & 15, kg = lane >> 4;
    // (a uniform address per item and one lane offset for all items and matrices: no address registers to keep)
    const T *at = src + ((size_t)blk * BS + (TRANS ? 0 : 16 * rt)) * BS + (TRANS ? 16 * rt : 0);
    if constexpr (TRANS) {   // lane (row i, group g) takes W[blk][(b/4) g + j][i]: loads run along i across a group's lanes
        const uint32_t off = G::Q * kg * BS + l16;
#pragma unroll
        for (int p = 0; p < WV; ++p)
#pragma unroll
            for (int e = 0; e < 4; ++e) dst[p][e] = ld1(at + (4 * p + e) * BS + off);
    } else if constexpr (sizeof(T) == 2) {
        const uint32_t off = l16 * BS + 8 * kg;
#pragma unroll
        for (int p = 0; p < WV; ++p) dst[p] = *reinterpret_cast<const f32x4 *>(at + 32 * p + off);
    } else {
        const uint32_t off = l16 * BS + G::Q * kg;
#pragma unroll
        for (int p = 0; p < WV; ++p) dst[p] = ld4(at + 4 * p + off);
    }
}

template <typename T, int BS, bool TRANS>
__device__ __forceinline__ void request(const T *__restrict__ src, int item, int wave, int lane, f32x4 (&dst)[Ring<T, BS, TRANS>::WV])
{
    typedef Geo<BS> G;
    request_at<T, BS, TRANS>(src, wave * G::NBW + item / G::RT, item % G::RT, lane, dst);
}

template <typename T, int BS, bool TRANS>
__device__ __forceinline__ void preload(Ring<T, BS, TRANS> &ring, const T *__restrict__ W, int wave, int lane)
{
    typedef Ring<T, BS, TRANS> Rg;
    asm volatile("" : "+s"(W));   // (the addresses are formed here, not kept over a persistent workgroup's tiles)
#pragma unroll
    for (int d = 0; d < Rg::DEPTH && d < Rg::ITEMS; ++d) request<T, BS, TRANS>(W, d, wave, lane, ring.w[d]);
}

// The same value, unknown to the compiler: addresses derived from it are formed at their use instead of being kept in
// registers over a persistent workgroup's tiles (with the sums of the gradients there is no room for them: 556 bytes of spills
// a lane).
__device__ __forceinline__ int fresh(int v)
{
    asm volatile("" : "+v"(v));
    return v;
}

// Eight fp32 values as three bf16 operands, x = hi + mid + lo exactly (8 + 8 + 8 significant bits; each part is the
// remainder of the one before cut to its upper 16 bits) for every finite x.  The mid part of an infinity is a NaN, and an
// infinite weight meets parts that are zero: such products come out as NaN and are formed again, see plain_where_nan.
__device__ __forceinline__ uint32_t high_halves(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x07060302u); }
__device__ __forceinline__ void split3(const float (&x)[8], h16::op8 (&p)[3])
{
    uint32_t hi[8], mid[8], lo[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const uint32_t v = __float_as_uint(x[j]);
        hi[j] = v;
        const float r = x[j] - __uint_as_float(v & 0xffff0000u);
        mid[j] = __float_as_uint(r);
        lo[j] = __float_as_uint(r - __uint_as_float(mid[j] & 0xffff0000u));
    }
    p[0] = h16::op8{high_halves(hi[0], hi[1]), high_halves(hi[2], hi[3]), high_halves(hi[4], hi[5]), high_halves(hi[6], hi[7])};
    p[1] = h16::op8{high_halves(mid[0], mid[1]), high_halves(mid[2], mid[3]), high_halves(mid[4], mid[5]), high_halves(mid[6], mid[7])};
    p[2] = h16::op8{high_halves(lo[0], lo[1]), high_halves(lo[2], lo[3]), high_halves(lo[4], lo[5]), high_halves(lo[6], lo[7])};
}

// whether a product of the wave is a NaN (the sum of a lane's products tells it; one of opposite infinities only costs time)
template <int NT>
__device__ __forceinline__ bool any_nan(const f32x4 (&a)[NT])
{
    f32x4 t = a[0];
#pragma unroll
    for (int rt = 1; rt < NT; ++rt) t += a[rt];
    const float sum = (t[0] + t[1]) + (t[2] + t[3]);
    return __builtin_amdgcn_ballot_w64(sum != sum) != 0;
}

// The products of a block of bf16 weights again, its inputs still in place at e: those that are NaN by the three parts as the
// fp32 instruction forms them, so that infinities and NaN of the rows and of the weights come out as plain floating point has
// them, and the others as they were.  A block that holds a NaN takes this way, for rows and weights without them one test per
// block (it replaced a test of every value in split3).
template <int BS, int SK>
__device__ __forceinline__ void plain_where_nan(float *e, const bf16_t *__restrict__ W, int blk, int lane)
{
    typedef Geo<BS> G;
    constexpr int CH = BS / 32;
    const int l16 = lane & 15, kg = lane >> 4;
    float x[CH][8];
    h16::op8 b[CH][3];
#pragma unroll
    for (int c = 0; c < CH; ++c) {
#pragma unroll
        for (int j = 0; j < 8; ++j) x[c][j] = e[(32 * c + 8 * kg + j) * SK];
        split3(x[c], b[c]);
    }
#pragma unroll 1
    for (int rt = 0; rt < G::RT; ++rt) {
        f32x4 w[CH], a = {0, 0, 0, 0}, plain = {0, 0, 0, 0};
        request_at<bf16_t, BS, false>(W, blk, rt, lane, w);
#pragma unroll
        for (int part = 2; part >= 0; --part)
#pragma unroll
            for (int c = 0; c < CH; ++c) a = h16::mfma<bf16_t>(__builtin_bit_cast(h16::op8, w[c]), b[c][part], a);
#pragma unroll
        for (int c = 0; c < CH; ++c)
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const uint32_t pair = __float_as_uint(w[c][j >> 1]);
                plain = mfma(j & 1 ? h16::hi32<bf16_t>(pair) : h16::lo32<bf16_t>(pair), x[c][j], plain);
            }
        if (l16 < G::TV) {
#pragma unroll
            for (int r = 0; r < 4; ++r) e[(16 * rt + 4 * kg + r) * SK] = a[r] != a[r] ? plain[r] : a[r];
        }
    }
}

// One factor in place, its first items in the ring.  Block blk contracts the digit that has stride SK; its other digit
// puts it at at(blk).  bf16 blocks meet the fp32 values of the tile as three bf16 operands (exact, so the products are
// those of the fp32 instruction) on the 16x16x32 MFMA: 96 cycles per block of 32 instead of 512.  EXACT: the tile holds
// bf16 values (the rows as loaded), one operand is enough.
template <typename T, int BS, int SK, bool TRANS, bool EXACT, typename At>
__device__ __forceinline__ void stage_from(Ring<T, BS, TRANS> &ring, float *tile, const T *__restrict__ W, int wave, int lane, At at)
{
    typedef Geo<BS> G;
    typedef Ring<T, BS, TRANS> Rg;
    const int l16 = lane & 15, kg = lane >> 4;
    float *mine = tile + (l16 & (G::TV - 1)) * G::ROWP;
    float anchor = 0.0f;
    uint32_t again = 0;   // the wave's blocks with a NaN among their products: left as they were for plain_where_nan
    // (the pointer passes through an empty asm that names the latest result, so that the compiler keeps each
    // request where it is written instead of hoisting all of a stage's loads to its top)
    auto next = [&](int item) {
        if (item + Rg::DEPTH < Rg::ITEMS) {
            const T *src = W;
            asm volatile("" : "+s"(src) : "v"(anchor));
            request<T, BS, TRANS>(src, item + Rg::DEPTH, wave, lane, ring.w[item % Rg::DEPTH]);
        }
    };
#pragma unroll
    for (int u = 0; u < G::NBW; ++u) {
        float *e = mine + at(wave * G::NBW + u);
        f32x4 acc[G::RT];
        if constexpr (Rg::HALF) {
            constexpr int CH = BS / 32, PARTS = EXACT ? 1 : 3;
            h16::op8 b[CH][3];
#pragma unroll
            for (int c = 0; c < CH; ++c) {
                float x[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) x[j] = e[(32 * c + 8 * kg + j) * SK];
                if constexpr (EXACT) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) b[c][0][j] = high_halves(__float_as_uint(x[2 * j]), __float_as_uint(x[2 * j + 1]));
                } else split3(x, b[c]);
            }
#pragma unroll
            for (int rt = 0; rt < G::RT; ++rt) {
                const int item = u * G::RT + rt;
                f32x4 a = {0, 0, 0, 0};
#pragma unroll
                for (int part = PARTS - 1; part >= 0; --part)
#pragma unroll
                    for (int c = 0; c < CH; ++c)
                        a = h16::mfma<bf16_t>(__builtin_bit_cast(h16::op8, ring.w[item % Rg::DEPTH][c]), b[c][part], a);
                acc[rt] = a;
                anchor = a[0];
                next(item);
            }
        } else {
            float bv[G::Q];
#pragma unroll
            for (int j = 0; j < G::Q; ++j) bv[j] = e[(G::Q * kg + j) * SK];
#pragma unroll
            for (int rt = 0; rt < G::RT; ++rt) {
                const int item = u * G::RT + rt;
                f32x4 a = {0, 0, 0, 0};
#pragma unroll
                for (int j = 0; j < G::Q; ++j) a = mfma(ring.w[item % Rg::DEPTH][j >> 2][j & 3], bv[j], a);
                acc[rt] = a;
                anchor = a[0];
                next(item);
            }
        }
        if constexpr (Rg::HALF && !EXACT) {
            if (__builtin_expect(any_nan(acc), 0)) {
                again |= 1u << u;
                continue;
            }
        }
        // every input of the block has been read: the results take their places
        if (l16 < G::TV) {
#pragma unroll
            for (int rt = 0; rt < G::RT; ++rt)
#pragma unroll
                for (int r = 0; r < 4; ++r) e[(16 * rt + 4 * kg + r) * SK] = acc[rt][r];
        }
    }
    if constexpr (Rg::HALF && !EXACT)
        for (; __builtin_expect(again != 0, 0); again &= again - 1) {
            const int blk = wave * G::NBW + __builtin_ctz(again), ln = fresh(lane);
            plain_where_nan<BS, SK>(tile + (ln & 15 & (G::TV - 1)) * G::ROWP + at(blk), W, blk, ln);
        }
}

template <typename T, int BS, int SK, bool TRANS = false, typename At>
__device__ __forceinline__ void stage(float *tile, const T *__restrict__ W, int wave, int lane, At at)
{
    Ring<T, BS, TRANS> ring;
    preload<T, BS, TRANS>(ring, W, wave, lane);
    stage_from<T, BS, SK, TRANS, false>(ring, tile, W, wave, lane, at);
}

// Tiles are handed out so that neighbouring ones run on one XCD at one time (workgroups go to the eight XCDs in turn):
// tiles of transposed rows share cache lines.  An XCD takes a run of tiles, its workgroups in turn.
struct Tiles {
    int64_t first, end, step;
    __device__ Tiles(int64_t ntiles)
    {
        // workgroups of the XCDs before x, of x: the tiles are divided alike
        const int g = gridDim.x, x = blockIdx.x & 7, before = x * (g / 8) + (x < g % 8 ? x : g % 8);
        step = g / 8 + (x < g % 8 ? 1 : 0);
        first = ntiles * before / g + (blockIdx.x >> 3);
        end = ntiles * (before + step) / g;
    }
};

template <typename T, int BS>
__global__ __launch_bounds__(Geo<BS>::THREADS, 4) void matmul_kernel(const T *__restrict__ x, const T *__restrict__ R,
                                                                                  const T *__restrict__ L, T *__restrict__ y, int64_t batch)
{
    typedef Geo<BS> G;
    extern __shared__ __attribute__((aligned(16))) float tile[];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int64_t ntiles = (batch + G::TV - 1) / G::TV;
    Ring<T, BS> ring;
    for (int64_t t = blockIdx.x; t < ntiles; t += gridDim.x) {
        const int64_t v0 = t * G::TV;
        preload<T, BS, false>(ring, R, wave, lane);
        for (int piece = threadIdx.x; piece < G::TV * G::N / 4; piece += G::THREADS) {
            const int v = piece / (G::N / 4), i = 4 * (piece % (G::N / 4));
            int64_t r = v0 + v;
            if (r >= batch) r = batch - 1;   // (rows past the end: computed, never stored)
            const f32x4 val = ld4s(x + r * G::N + i);
            float *d = tile + v * G::ROWP + (i / BS) * G::SH + i % BS;
            d[0] = val[0]; d[1] = val[1]; d[2] = val[2]; d[3] = val[3];
        }
        __syncthreads();
        stage_from<T, BS, G::SH, false, true>(ring, tile, R, wave, lane, [](int k) { return k; });
        preload<T, BS, false>(ring, L, wave, lane);
        __syncthreads();
        stage_from<T, BS, 1, false, false>(ring, tile, L, wave, lane, [](int r) { return r * G::SH; });
        __syncthreads();
        // y[s b + r] sits at (r, s): a thread stores r = 4 q .. 4 q + 3 of one s
        for (int piece = threadIdx.x; piece < G::TV * G::N / 4; piece += G::THREADS) {
            const int v = piece / (G::N / 4), m = 4 * (piece % (G::N / 4));
            const float *sp = tile + v * G::ROWP + (m % BS) * G::SH + m / BS;
            if (v0 + v < batch) st4s(y + (v0 + v) * G::N + m, f32x4{sp[0], sp[G::SH], sp[2 * G::SH], sp[3 * G::SH]});
        }
        __syncthreads();
    }
}

// NT row tiles of block blk of W from row row0 on (all of them, or with EXACT a part), the block's inputs at e (stride SK), the
// matrices in registers: the products of stage_from, in its order
template <typename T, int BS, int SK, bool EXACT, int NT>
__device__ __forceinline__ void block_products(float *e, const f32x4 (&w)[NT][Ring<T, BS>::WV], const T *__restrict__ W, int blk,
                                               int row0, int lane)
{
    typedef Geo<BS> G;
    static_assert(EXACT || NT == G::RT, "");
    const int l16 = lane & 15, kg = lane >> 4;
    f32x4 acc[NT];
    if constexpr (Ring<T, BS>::HALF) {
        constexpr int CH = BS / 32, PARTS = EXACT ? 1 : 3;
        h16::op8 b[CH][3];
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            float x[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) x[j] = e[(32 * c + 8 * kg + j) * SK];
            if constexpr (EXACT) {
#pragma unroll
                for (int j = 0; j < 4; ++j) b[c][0][j] = high_halves(__float_as_uint(x[2 * j]), __float_as_uint(x[2 * j + 1]));
            } else split3(x, b[c]);
        }
#pragma unroll
        for (int rt = 0; rt < NT; ++rt) {
            acc[rt] = f32x4{0, 0, 0, 0};
#pragma unroll
            for (int part = PARTS - 1; part >= 0; --part)
#pragma unroll
                for (int c = 0; c < CH; ++c) acc[rt] = h16::mfma<bf16_t>(__builtin_bit_cast(h16::op8, w[rt][c]), b[c][part], acc[rt]);
        }
    } else {
        float bv[G::Q];
#pragma unroll
        for (int j = 0; j < G::Q; ++j) bv[j] = e[(G::Q * kg + j) * SK];
#pragma unroll
        for (int rt = 0; rt < NT; ++rt) {
            acc[rt] = f32x4{0, 0, 0, 0};
#pragma unroll
            for (int j = 0; j < G::Q; ++j) acc[rt] = mfma(w[rt][j >> 2][j & 3], bv[j], acc[rt]);
        }
    }
    if constexpr (Ring<T, BS>::HALF && !EXACT) {
        if (__builtin_expect(any_nan(acc), 0)) {
            plain_where_nan<BS, SK>(e, W, blk, lane);
            return;
        }
    }
    if (l16 < G::TV) {
#pragma unroll
        for (int rt = 0; rt < NT; ++rt)
#pragma unroll
            for (int r = 0; r < 4; ++r) e[(row0 + 16 * rt + 4 * kg + r) * SK] = acc[rt][r];
    }
}

// The product for few rows, a tile divided over BS / 16 workgroups: each forms 16 of the middle indices r, rows r of every
// block of R, and takes them through its 16 blocks of L, so that nothing is formed twice and nothing is summed across
// workgroups.  A workgroup of matmul_kernel reads both matrices whole (2 MB in fp32 at b = 64) and that is all of its time
// where the tiles leave compute units idle; here a part of it, requested at once.  Neighbouring workgroups are different
// parts: an XCD fetches one or two of them.  Results are those of matmul_kernel bit for bit.
template <typename T, int BS>
__global__ __launch_bounds__(Geo<BS>::THREADS, Geo<BS>::THREADS / 256) void matmul_few_kernel(const T *__restrict__ x, const T *__restrict__ R,
                                                                                            const T *__restrict__ L, T *__restrict__ y,
                                                                                            int64_t batch)
{
    typedef Geo<BS> G;
    typedef Ring<T, BS> Rg;
    constexpr int NB = 16 / G::WAVES;                        // blocks of L of a wave
    constexpr bool EARLY = BS == 32 || Rg::HALF;             // registers for both matrices
    extern __shared__ __attribute__((aligned(16))) float tile[];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, l16 = lane & 15;
    const int part = blockIdx.x % G::RT;
    const int64_t v0 = (int64_t)(blockIdx.x / G::RT) * G::TV;
    f32x4 wr[G::NBW][1][Rg::WV], wl[NB][G::RT][Rg::WV];
    auto request_l = [&]() {
#pragma unroll
        for (int i = 0; i < NB * G::RT; ++i)
            request_at<T, BS, false>(L, 16 * part + wave * NB + i / G::RT, i % G::RT, lane, wl[i / G::RT][i % G::RT]);
    };
#pragma unroll
    for (int u = 0; u < G::NBW; ++u) request_at<T, BS, false>(R, wave * G::NBW + u, part, lane, wr[u][0]);
    if constexpr (EARLY) request_l();
    for (int piece = threadIdx.x; piece < G::TV * G::N / 4; piece += G::THREADS) {
        const int v = piece / (G::N / 4), i = 4 * (piece % (G::N / 4));
        int64_t r = v0 + v;
        if (r >= batch) r = batch - 1;   // (rows past the end: computed, never stored)
        const f32x4 val = ld4(x + r * G::N + i);
        float *d = tile + v * G::ROWP + (i / BS) * G::SH + i % BS;
        d[0] = val[0]; d[1] = val[1]; d[2] = val[2]; d[3] = val[3];
    }
    __syncthreads();
    float *mine = tile + (l16 & (G::TV - 1)) * G::ROWP;
#pragma unroll
    for (int u = 0; u < G::NBW; ++u) {
        const int blk = wave * G::NBW + u;
        block_products<T, BS, G::SH, true, 1>(mine + blk, wr[u], R, blk, 16 * part, lane);
    }
    if constexpr (!EARLY) request_l();
    __syncthreads();
#pragma unroll
    for (int u = 0; u < NB; ++u) {
        const int blk = 16 * part + wave * NB + u;
        block_products<T, BS, 1, false, G::RT>(mine + blk * G::SH, wl[u], L, blk, 0, lane);
    }
    __syncthreads();
    for (int piece = threadIdx.x; piece < G::TV * BS * 4; piece += G::THREADS) {   // four r of one s
        const int v = piece / (BS * 4), s = piece / 4 % BS, r = 16 * part + 4 * (piece % 4);
        const float *sp = tile + v * G::ROWP + r * G::SH + s;
        if (v0 + v < batch) st4(y + (v0 + v) * G::N + s * BS + r, f32x4{sp[0], sp[G::SH], sp[2 * G::SH], sp[3 * G::SH]});
    }
}

// opt: the options of the basic M2 layer (Sec. 3.2): an activation after the kernel product, rows that run along the
// middle index of a (B, N, H) tensor (transposed: a tile's TV rows are TV neighbouring h of one batch entry, moved in
// pieces of four rows of one position), and the skip connection and layer norm over the row at the store.
template <typename T, int BS, bool GIN, bool GOUT, bool TRANSPOSED>
__global__ __launch_bounds__(Geo<BS>::THREADS, 4) void mixer_kernel(
    const T *__restrict__ u, const T *__restrict__ K, const T *__restrict__ g_in, const T *__restrict__ g_out,
    const T *__restrict__ R1, const T *__restrict__ L1, const T *__restrict__ R2, const T *__restrict__ L2, T *__restrict__ y,
    int64_t rows, int H, const MixOpt opt)
{
    typedef Geo<BS> G;
    extern __shared__ __attribute__((aligned(16))) float tile[];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int64_t ntiles = (rows + G::TV - 1) / G::TV;
    constexpr int PIECES = G::TV * G::N / 4, PIECES_AHEAD = sizeof(T) == 2 ? 4 : 2;
    Ring<T, BS> ring;
    const Tiles mine(ntiles);
    for (int64_t t = mine.first; t < mine.end; t += mine.step) {
        const int64_t v0 = t * G::TV;
        const int64_t bt = v0 / H;           // (one division per tile, not one per piece)
        const int h0 = (int)(v0 - bt * H);
        // piece p of a tile: four elements and where they sit.  Plain rows: elements i .. i + 3 of row v; transposed: element i
        // of rows v .. v + 3 (neighbouring h of one batch entry: contiguous in memory).
        auto where = [&](int p, int &v, int &i) -> int64_t {
            if (TRANSPOSED) {
                i = p / (G::TV / 4);
                v = 4 * (p % (G::TV / 4));
                // (rows is a multiple of TV here and a tile stays inside one batch entry: v0 = bt H + h0)
                return (bt * G::N + i) * H + h0 + v;
            }
            v = p / (G::N / 4);
            i = 4 * (p % (G::N / 4));
            int64_t r = v0 + v;
            if (r >= rows) r = rows - 1;   // (rows past the end: computed, never stored)
            return r * G::N + i;
        };
        // the four tile words of a piece: natural position (hi, lo) = (i / b, i % b)
        constexpr int STEP = TRANSPOSED ? G::ROWP : 1;
        auto put = [&](int v, int i, f32x4 val) {
            float *d = tile + v * G::ROWP + (i / BS) * G::SH + i % BS;
            d[0] = val[0]; d[STEP] = val[1]; d[2 * STEP] = val[2]; d[3 * STEP] = val[3];
        };
        auto get = [&](int v, int i) -> f32x4 {
            const float *d = tile + v * G::ROWP + (i / BS) * G::SH + i % BS;
            return f32x4{d[0], d[STEP], d[2 * STEP], d[3 * STEP]};
        };
        preload<T, BS, false>(ring, R1, wave, lane);
#pragma unroll(PIECES_AHEAD)
        for (int piece = threadIdx.x; piece < PIECES; piece += G::THREADS) {
            int v, i;
            const int64_t at = where(piece, v, i);
            f32x4 val = ld4(u + at);
            if (GIN) val *= ld4(g_in + at);
            put(v, i, val);
        }
        __syncthreads();
        stage_from<T, BS, G::SH, false, !GIN>(ring, tile, R1, wave, lane, [](int k) { return k; });
        preload<T, BS, false>(ring, L1, wave, lane);
        __syncthreads();
        stage_from<T, BS, 1, false, false>(ring, tile, L1, wave, lane, [](int r) { return r * G::SH; });
        preload<T, BS, false>(ring, R2, wave, lane);
        __syncthreads();
        // kernel product: entry m = s b + r of the transform domain sits at (r, s)
#pragma unroll(PIECES_AHEAD)
        for (int piece = threadIdx.x; piece < PIECES; piece += G::THREADS) {
            const int v = piece / (G::N / 4), m = 4 * (piece % (G::N / 4));
            int h = h0 + v;   // of row v0 + v
            if (h >= H) h = H >= G::TV ? h - H : h % H;
            const f32x4 kv = ld4(K + (int64_t)h * G::N + m);
            float *sp = tile + v * G::ROWP + (m % BS) * G::SH + m / BS;
            f32x4 p = {sp[0] * kv[0], sp[G::SH] * kv[1], sp[2 * G::SH] * kv[2], sp[3 * G::SH] * kv[3]};
            if (opt.act) p = f32x4{fmaxf(p[0], 0.0f), fmaxf(p[1], 0.0f), fmaxf(p[2], 0.0f), fmaxf(p[3], 0.0f)};
            sp[0] = p[0]; sp[G::SH] = p[1]; sp[2 * G::SH] = p[2]; sp[3 * G::SH] = p[3];
        }
        __syncthreads();
        stage_from<T, BS, 1, false, false>(ring, tile, R2, wave, lane, [](int k) { return k * G::SH; });
        preload<T, BS, false>(ring, L2, wave, lane);
        __syncthreads();
        stage_from<T, BS, G::SH, false, false>(ring, tile, L2, wave, lane, [](int r) { return r; });
        __syncthreads();
        if (opt.layer_norm) {
            // result (gated) + u back into the tile, then a wave per row: mean, variance, scale and shift
#pragma unroll(PIECES_AHEAD)
            for (int piece = threadIdx.x; piece < PIECES; piece += G::THREADS) {
                int v, i;
                const int64_t at = where(piece, v, i);
                f32x4 val = get(v, i);
                if (GOUT) val *= ld4(g_out + at);
                put(v, i, val + ld4(u + at));
            }
            __syncthreads();
            for (int v = wave; v < G::TV; v += G::WAVES) {
                const float *row = tile + v * G::ROWP;
                auto four = [&](int q) -> f32x4 {   // four neighbouring elements of the row
                    const float *d = row + ((256 * q + 4 * lane) / BS) * G::SH + (4 * lane) % BS;
                    return f32x4{d[0], d[1], d[2], d[3]};
                };
                float sum = 0.0f;
#pragma unroll 4
                for (int q = 0; q < G::N / 256; ++q) {
                    const f32x4 x = four(q);
                    sum += (x[0] + x[1]) + (x[2] + x[3]);
                }
                for (int m = 32; m; m >>= 1) sum += __shfl_xor(sum, m);
                const float mean = sum / G::N;
                float sq = 0.0f;
#pragma unroll 4
                for (int q = 0; q < G::N / 256; ++q) {
                    const f32x4 x = four(q) - mean;
                    sq += (x[0] * x[0] + x[1] * x[1]) + (x[2] * x[2] + x[3] * x[3]);
                }
                for (int m = 32; m; m >>= 1) sq += __shfl_xor(sq, m);
                const float rstd = rsqrtf(sq / G::N + opt.eps);
                const int64_t r = v0 + v;
                if (r < rows) {
#pragma unroll 4
                    for (int q = 0; q < G::N / 256; ++q) {
                        const int j = 256 * q + 4 * lane;
                        const f32x4 gm = ld4((const T *)opt.gamma + j), bb = ld4((const T *)opt.beta + j);
                        const f32x4 res = (four(q) - mean) * rstd * gm + bb;
                        if (TRANSPOSED) {
#pragma unroll
                            for (int e = 0; e < 4; ++e) y[(bt * G::N + j + e) * H + h0 + v] = from_f32<T>(res[e]);
                        } else st4(y + r * G::N + j, res);
                    }
                }
            }
        } else {
#pragma unroll(PIECES_AHEAD)
            for (int piece = threadIdx.x; piece < PIECES; piece += G::THREADS) {
                int v, i;
                const int64_t at = where(piece, v, i);
                if (v0 + v < rows) {
                    f32x4 val = get(v, i);
                    if (GOUT) val *= ld4(g_out + at);
                    st4(y + at, val);
                }
            }
        }
        __syncthreads();
    }
}

// ---- gradients (blocks of 32) ----------------------------------------------------------------------------------
// With S = sum_v <dy_v, M x_v>, mid = R-stage of x at (r, k) and dy loaded at (r, s):
//   dmid(r, k) = sum_s L[r][s][k] dy(r, s)    (block r of L transposed contracts s, stride 1)
//   dx(c, k)   = sum_r R[k][r][c] dmid(r, k)  (block k of R transposed contracts r, stride SH)
//   dL[r][s][k] = sum_v dy_v(r, s) mid_v(r, k),   dR[k][r][c] = sum_v dmid_v(r, k) x_v(c, k).
// Two tiles of 16 rows (forward values and gradients, 157 KB, one workgroup per compute unit): a factor's gradient is, per
// block and 16 x 16 piece of it, four MFMAs whose contraction index is the row of the tile; the sums of a wave's four
// blocks (64 registers a factor) stay in registers over all tiles of the workgroup and are added to the cleared buffer once.

// sum[u][it][jt] += (rows 16 it .. of side A)^T (rows 16 jt .. of side B) of block wave NBW + u, over the tile's rows
template <int BS, int SK, typename At>
__device__ __forceinline__ void outer(const float *ta, const float *tb, int wave, int lane, At at,
                                      f32x4 (&sum)[Geo<BS>::NBW][Geo<BS>::RT][Geo<BS>::RT])
{
    typedef Geo<BS> G;
    const int l16 = lane & 15, kg = lane >> 4;
#pragma unroll
    for (int u = 0; u < G::NBW; ++u) {
        const int off = at(wave * G::NBW + u);
#pragma unroll
        for (int q = 0; q < G::TV / 4; ++q) {   // the MFMA's contraction index kg is row 4 q + kg of the tile
            const float *ra = ta + (4 * q + kg) * G::ROWP + off, *rb = tb + (4 * q + kg) * G::ROWP + off;
            float a[G::RT], b[G::RT];
#pragma unroll
            for (int it = 0; it < G::RT; ++it) {
                a[it] = ra[(16 * it + l16) * SK];
                b[it] = rb[(16 * it + l16) * SK];
            }
#pragma unroll
            for (int it = 0; it < G::RT; ++it)
#pragma unroll
                for (int jt = 0; jt < G::RT; ++jt) sum[u][it][jt] = mfma(a[it], b[jt], sum[u][it][jt]);
        }
    }
}

template <int BS>
__device__ __forceinline__ void flush(float *dW, int wave, int lane, const f32x4 (&sum)[Geo<BS>::NBW][Geo<BS>::RT][Geo<BS>::RT])
{
    typedef Geo<BS> G;
    const int l16 = lane & 15, kg = lane >> 4;
#pragma unroll
    for (int u = 0; u < G::NBW; ++u)
#pragma unroll
        for (int it = 0; it < G::RT; ++it)
#pragma unroll
            for (int jt = 0; jt < G::RT; ++jt)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    atomicAdd(dW + ((size_t)(wave * G::NBW + u) * BS + 16 * it + 4 * kg + r) * BS + 16 * jt + l16, sum[u][it][jt][r]);
}

// A transposed factor on its way from L2, by block: lane (i, group g) takes columns 2 i, 2 i + 1 of the block's rows 8 g ..
// 8 g + 7, which serve both row tiles of the result (row tile rt holds outputs 2 i + rt): 8 loads of a pair where one per
// row and row tile took 16.  DEPTH blocks are requested ahead.
template <typename T> struct Pair;
template <> struct Pair<float> { typedef float2 type; };
template <> struct Pair<bf16_t> { typedef uint32_t type; };
template <typename T>
struct TRing {
    static constexpr int DEPTH = 2;
    typename Pair<T>::type w[DEPTH][8];
};

template <typename T>
__device__ __forceinline__ void request_t(const T *__restrict__ src, int blk, int lane, typename Pair<T>::type (&dst)[8])
{
    const T *at = src + (size_t)blk * 32 * 32;
    const uint32_t off = 8 * (lane >> 4) * 32 + 2 * (lane & 15);
#pragma unroll
    for (int j = 0; j < 8; ++j) dst[j] = *reinterpret_cast<const typename Pair<T>::type *>(at + 32 * j + off);
}

template <typename T>
__device__ __forceinline__ void preload_t(TRing<T> &ring, const T *__restrict__ W, int wave, int lane)
{
    asm volatile("" : "+s"(W));
#pragma unroll
    for (int d = 0; d < TRing<T>::DEPTH; ++d) request_t<T>(W, wave * Geo<32>::NBW + d, lane, ring.w[d]);
}

// A block's two operands of row tiles 0 and 1 from its requested pairs
__device__ __forceinline__ void transposed_operands(const uint32_t (&w)[8], h16::op8 (&a)[2])
{
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        a[0][j] = __builtin_amdgcn_perm(w[2 * j + 1], w[2 * j], 0x05040100u);
        a[1][j] = __builtin_amdgcn_perm(w[2 * j + 1], w[2 * j], 0x07060302u);
    }
}

// plain_where_nan for a transposed block
template <int SK>
__device__ __forceinline__ void plain_where_nan_t(float *e, const bf16_t *__restrict__ W, int blk, int lane)
{
    const int kg = lane >> 4;
    uint32_t w[8];
    request_t<bf16_t>(W, blk, lane, w);
    float x[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) x[j] = e[(8 * kg + j) * SK];
    h16::op8 b[3], a[2];
    split3(x, b);
    transposed_operands(w, a);
    f32x4 acc[2] = {{0, 0, 0, 0}, {0, 0, 0, 0}}, plain[2] = {{0, 0, 0, 0}, {0, 0, 0, 0}};
#pragma unroll
    for (int part = 2; part >= 0; --part)
#pragma unroll
        for (int rt = 0; rt < 2; ++rt) acc[rt] = h16::mfma<bf16_t>(a[rt], b[part], acc[rt]);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        plain[0] = mfma(h16::lo32<bf16_t>(w[j]), x[j], plain[0]);
        plain[1] = mfma(h16::hi32<bf16_t>(w[j]), x[j], plain[1]);
    }
#pragma unroll
    for (int rt = 0; rt < 2; ++rt)
#pragma unroll
        for (int r = 0; r < 4; ++r) e[(8 * kg + 2 * r + rt) * SK] = acc[rt][r] != acc[rt][r] ? plain[rt][r] : acc[rt][r];
}

// One transposed factor in place, its first blocks in the ring.
template <typename T, int SK, typename At>
__device__ __forceinline__ void stage_t(TRing<T> &ring, float *tile, const T *__restrict__ W, int wave, int lane, At at)
{
    typedef Geo<32> G;
    constexpr int DEPTH = TRing<T>::DEPTH;
    const int l16 = lane & 15, kg = lane >> 4;
    float *mine = tile + l16 * G::ROWP;
    uint32_t again = 0;   // as in stage_from
#pragma unroll
    for (int u = 0; u < G::NBW; ++u) {
        float *e = mine + at(wave * G::NBW + u);
        const auto &w = ring.w[u % DEPTH];
        float x[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) x[j] = e[(8 * kg + j) * SK];
        f32x4 acc[2] = {{0, 0, 0, 0}, {0, 0, 0, 0}};
        if constexpr (sizeof(T) == 2) {
            h16::op8 b[3], a[2];
            split3(x, b);
            transposed_operands(w, a);
#pragma unroll
            for (int part = 2; part >= 0; --part)
#pragma unroll
                for (int rt = 0; rt < 2; ++rt) acc[rt] = h16::mfma<bf16_t>(a[rt], b[part], acc[rt]);
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                acc[0] = mfma(w[j].x, x[j], acc[0]);
                acc[1] = mfma(w[j].y, x[j], acc[1]);
            }
        }
        if (u + DEPTH < G::NBW) {
            const T *src = W;
            asm volatile("" : "+s"(src) : "v"(acc[1][0]));   // (the request stays behind these products)
            request_t<T>(src, wave * G::NBW + u + DEPTH, lane, ring.w[u % DEPTH]);
        }
        if constexpr (sizeof(T) == 2) {
            if (__builtin_expect(any_nan(acc), 0)) {
                again |= 1u << u;
                continue;
            }
        }
        // every input of the block has been read: the results take their places
#pragma unroll
        for (int rt = 0; rt < 2; ++rt)
#pragma unroll
            for (int r = 0; r < 4; ++r) e[(8 * kg + 2 * r + rt) * SK] = acc[rt][r];
    }
    if constexpr (sizeof(T) == 2)
        for (; __builtin_expect(again != 0, 0); again &= again - 1) {
            const int blk = wave * G::NBW + __builtin_ctz(again), ln = fresh(lane);
            plain_where_nan_t<SK>(tile + (ln & 15) * G::ROWP + at(blk), W, blk, ln);
        }
}

// A thread's share of a 16 x 1024 tile: piece p holds elements i .. i + 3 of row v(p).
struct Share {
    static constexpr int PIECES = Geo<32>::TV * Geo<32>::N / 4 / Geo<32>::THREADS;
    const int v0, i;
    explicit __device__ Share(int thread) : v0(thread >> 8), i(4 * (thread & 255)) {}
    __device__ int v(int p) const { return v0 + 2 * p; }
    __device__ int natural(int p) const { return v(p) * Geo<32>::ROWP + (i / 32) * Geo<32>::SH + i % 32; }   // elements 1 apart
    __device__ int swapped(int p) const { return v(p) * Geo<32>::ROWP + (i % 32) * Geo<32>::SH + i / 32; }   // SH apart
};
template <int STEP> __device__ __forceinline__ void put(float *d, f32x4 v) { d[0] = v[0]; d[STEP] = v[1]; d[2 * STEP] = v[2]; d[3 * STEP] = v[3]; }
template <int STEP> __device__ __forceinline__ f32x4 get(const float *d) { return f32x4{d[0], d[STEP], d[2 * STEP], d[3 * STEP]}; }

typedef f32x4 Sums[Geo<32>::NBW][Geo<32>::RT][Geo<32>::RT];
__device__ __forceinline__ void zero(Sums &sum)
{
    for (auto &u : sum)
        for (auto &it : u)
            for (auto &jt : it) jt = f32x4{0, 0, 0, 0};
}

// Gradients of y = M (g_in o u) (g_in null: of M u) for rows of 1024: dx and dg_in (DX), dR (DR) and dL (DL), each may be null.
// The values that dR needs again after mid took their places wait in registers.  One gradient alone takes an instance of
// its own: told by the pointers only, the kernel read u and R and went through stages for gradients that nobody asked for (fp32,
// 4096 rows, us: dx 16.8 -> 13.0, dR 52.2 -> 49.5, dL 56.0 -> 50.6).  Two or three take the instance of all (with the sets
// told apart at compile time it spilled 26 registers).
template <typename T, bool DX, bool DR, bool DL>
__global__ __launch_bounds__(512, 2) void backward_kernel(const T *__restrict__ u, const T *__restrict__ g_in, const T *__restrict__ R,
                                                          const T *__restrict__ L, const T *__restrict__ dy, T *__restrict__ dx,
                                                          T *__restrict__ dg_in, float *__restrict__ dR, float *__restrict__ dL, int64_t batch)
{
    typedef Geo<32> G;
    extern __shared__ __attribute__((aligned(16))) float tile[];
    float *fw = tile, *gr = tile + G::TV * G::ROWP;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const bool want_dx = DX && (dx || dg_in), want_dR = DR && dR, want_dL = DL && dL;
    Sums sumR, sumL;
    if (DR) zero(sumR);
    if (DL) zero(sumL);
    const int64_t ntiles = (batch + G::TV - 1) / G::TV;
    for (int64_t t = blockIdx.x; t < ntiles; t += gridDim.x) {
        const int64_t v0 = t * G::TV;
        f32x4 x[Share::PIECES];
        Ring<T, 32> ring;
        TRing<T> tring;
        // rows past the batch: their gradients are zero, their values a copy of the last row
        float last = 0.0f;
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            int thread = threadIdx.x;
            asm volatile("" : "+v"(thread) : "v"(last));   // (half of the requests at a time: registers)
            const Share mine(thread);
#pragma unroll
            for (int p = 4 * half; p < 4 * half + 4; ++p) {
                const bool live = v0 + mine.v(p) < batch;
                const int64_t at = (live ? v0 + mine.v(p) : batch - 1) * G::N + mine.i;
                if (DR || DL) {
                    x[p] = ld4(u + at);
                    if (g_in) x[p] *= ld4(g_in + at);
                }
                f32x4 g = ld4(dy + at);
                if (!live) g = f32x4{0, 0, 0, 0};
                if (DR || DL) put<1>(fw + mine.natural(p), x[p]);
                put<G::SH>(gr + mine.swapped(p), g);   // dy[s b + r] at (r, s)
                last = g[0];
            }
        }
        if (DL) preload<T, 32, false>(ring, R, wave, fresh(lane));
        __syncthreads();
        if (want_dL) {
            stage_from<T, 32, G::SH, false, false>(ring, fw, R, wave, fresh(lane), [](int k) { return k; });   // x -> mid
            __syncthreads();
            outer<32, 1>(gr, fw, wave, fresh(lane), [](int r) { return r * G::SH; }, sumL);   // dL[r][s][k]: dy(r, s) x mid(r, k)
        }
        if (DX || DR) {
            preload_t<T>(tring, L, wave, fresh(lane));
            // (a wave's blocks of the gradient tile are its own in both: no barrier)
            stage_t<T, 1>(tring, gr, L, wave, fresh(lane), [](int r) { return r * G::SH; });   // dy -> dmid
            if (DX) preload_t<T>(tring, R, wave, fresh(lane));
            __syncthreads();
        }
        if (want_dR) {
            if (want_dL) {
                const Share mine(fresh(threadIdx.x));
#pragma unroll
                for (int p = 0; p < Share::PIECES; ++p) put<1>(fw + mine.natural(p), x[p]);
                __syncthreads();
            }
            outer<32, G::SH>(gr, fw, wave, fresh(lane), [](int k) { return k; }, sumR);   // dR[k][r][c]: dmid(r, k) x x(c, k)
        }
        if (want_dx) {
            stage_t<T, G::SH>(tring, gr, R, wave, fresh(lane), [](int k) { return k; });   // dmid -> dx at (c, k)
            __syncthreads();
            const Share mine(fresh(threadIdx.x));
#pragma unroll 4
            for (int p = 0; p < Share::PIECES; ++p) {
                const int64_t at = (v0 + mine.v(p)) * G::N + mine.i;
                if (v0 + mine.v(p) >= batch) break;
                const f32x4 d = get<1>(gr + mine.natural(p));
                if (dx) st4(dx + at, g_in ? d * ld4(g_in + at) : d);
                if (dg_in) st4(dg_in + at, d * ld4(u + at));
            }
        }
        __syncthreads();
    }
    if (want_dL) flush<32>(dL, wave, fresh(lane), sumL);
    if (want_dR) flush<32>(dR, wave, fresh(lane), sumR);
}

// The rows that a workgroup of the next kernel takes: whole tiles, all but the last of the call
struct TileRun {
    int64_t begin, end;
    __host__ __device__ TileRun(int64_t rows, int64_t wg, int64_t grid)
    {
        constexpr int TV = Geo<32>::TV;
        const int64_t ntiles = (rows + TV - 1) / TV;
        begin = ntiles * wg / grid * TV;
        end = ntiles * (wg + 1) / grid * TV;
        if (end > rows) end = rows;
    }
};

// The first half of the mixer's gradients, y = g_out o M2 (K o s), s = M1 (g_in o u): s again, dg_out, dR2, dL2, dK and
// ds = dt o K (dt = M2^T (dy o g_out)); backward_kernel takes ds through M1.  Everything between stays in the two tiles, s
// in registers.  Tiles take their rows channel by channel (row q is sequence q % B of channel q / B) and a workgroup's
// tiles follow each other, so K is read once per channel and a channel's dK is summed in registers, sequence after sequence
// (the products change hands in the free tile: two whole columns to a thread).
// Parts of a channel that workgroups share go to dK_parts (two rows of 1024 per workgroup) and are joined in order, so the
// same call gives the same dK.  (Sums by parity of the row, joined by atomic adds into a cleared dK, were slower too: training
// step of 12288 rows in fp32 438 -> 428 us, in bf16 327 -> 313.)
// M2 works on M1's transposed result as it lies, t(s, r) at (r, s): block k' of R2 contracts its own row k' SH of the tile,
// block r' of L2 the stride SH; dy enters in natural order.
template <typename T>
__global__ __launch_bounds__(512, 2) void mixer_backward_kernel(
    const T *__restrict__ u, const T *__restrict__ K, const T *__restrict__ g_in, const T *__restrict__ g_out, const T *__restrict__ R1,
    const T *__restrict__ L1, const T *__restrict__ R2, const T *__restrict__ L2, const T *__restrict__ dy, T *__restrict__ ds,
    float *__restrict__ dK, float *__restrict__ dK_parts, T *__restrict__ dg_out, float *__restrict__ dR2, float *__restrict__ dL2, int B,
    int H)
{
    typedef Geo<32> G;
    extern __shared__ __attribute__((aligned(16))) float tile[];
    float *fw = tile, *gr = tile + G::TV * G::ROWP;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    Sums sumR, sumL;
    zero(sumR);
    zero(sumL);
    const int64_t rows = (int64_t)B * H;
    const TileRun run(rows, blockIdx.x, gridDim.x);
    float2 dk = make_float2(0.0f, 0.0f);   // of this thread's two columns, over the rows of the channel so far
    auto store_dk = [&](int h) {
        const int64_t first = (int64_t)h * B;
        float *dst = first < run.begin ? dK_parts + 2 * blockIdx.x * G::N
                   : first + B > run.end ? dK_parts + (2 * blockIdx.x + 1) * G::N : dK + (int64_t)h * G::N;
        *reinterpret_cast<float2 *>(dst + 2 * fresh(threadIdx.x)) = dk;
        dk = make_float2(0.0f, 0.0f);
    };
    for (int64_t q0 = run.begin; q0 < run.end; q0 += G::TV) {
        const int h0 = (int)(q0 / B), b0 = (int)(q0 - (int64_t)h0 * B);
        // channel and element offset of piece p; rows past the end: gradients zero, values a copy of the last row
        auto live = [&](const Share &mine, int p) { return q0 + mine.v(p) < rows; };
        auto where = [&](const Share &mine, int p, int &h) -> int64_t {
            const uint32_t v = live(mine, p) ? mine.v(p) : (uint32_t)(rows - 1 - q0), b = b0 + v, over = b / (uint32_t)B;
            h = h0 + over;
            return ((int64_t)(b - over * B) * H + h) * G::N + mine.i;
        };
        Ring<T, 32> ring;
        TRing<T> tring;
        preload<T, 32, false>(ring, R1, wave, fresh(lane));
        {
            const Share mine(fresh(threadIdx.x));
#pragma unroll 4
            for (int p = 0; p < Share::PIECES; ++p) {
                int h;
                const int64_t at = where(mine, p, h);
                f32x4 a = ld4(u + at), g = ld4(dy + at);
                if (g_in) a *= ld4(g_in + at);
                if (g_out) g *= ld4(g_out + at);
                if (!live(mine, p)) g = f32x4{0, 0, 0, 0};
                put<1>(fw + mine.natural(p), a);
                put<1>(gr + mine.natural(p), g);
            }
        }
        __syncthreads();
        stage_from<T, 32, G::SH, false, false>(ring, fw, R1, wave, fresh(lane), [](int k) { return k; });
        preload<T, 32, false>(ring, L1, wave, fresh(lane));
        __syncthreads();
        stage_from<T, 32, 1, false, false>(ring, fw, L1, wave, fresh(lane), [](int r) { return r * G::SH; });
        preload<T, 32, false>(ring, R2, wave, fresh(lane));
        __syncthreads();
        f32x4 s[Share::PIECES];
        {
            const Share mine(fresh(threadIdx.x));
#pragma unroll
            for (int p = 0; p < Share::PIECES; ++p) {
                int h;
                where(mine, p, h);
                s[p] = get<G::SH>(fw + mine.swapped(p));
                put<G::SH>(fw + mine.swapped(p), s[p] * ld4(K + (int64_t)h * G::N + mine.i));
            }
        }
        __syncthreads();
        if (dL2 || dg_out) {
            stage_from<T, 32, 1, false, false>(ring, fw, R2, wave, fresh(lane), [](int k) { return k * G::SH; });   // t -> mid
            preload<T, 32, false>(ring, L2, wave, fresh(lane));
            __syncthreads();
            if (dL2) outer<32, G::SH>(gr, fw, wave, fresh(lane), [](int r) { return r; }, sumL);
            // (a wave's blocks of either tile are its own in these three: no barrier)
            if (dg_out) stage_from<T, 32, G::SH, false, false>(ring, fw, L2, wave, fresh(lane), [](int r) { return r; });   // mid -> w
        }
        preload_t<T>(tring, L2, wave, fresh(lane));
        stage_t<T, G::SH>(tring, gr, L2, wave, fresh(lane), [](int r) { return r; });   // dw -> dmid
        preload_t<T>(tring, R2, wave, fresh(lane));
        __syncthreads();
        if (dL2 || dg_out) {
            if (dg_out) {
                const Share mine(fresh(threadIdx.x));
#pragma unroll 4
                for (int p = 0; p < Share::PIECES; ++p) {
                    int h;
                    const int64_t at = where(mine, p, h);
                    if (live(mine, p)) st4(dg_out + at, get<1>(fw + mine.natural(p)) * ld4(dy + at));
                }
                __syncthreads();
            }
            if (dR2) {
                const Share mine(fresh(threadIdx.x));
#pragma unroll
                for (int p = 0; p < Share::PIECES; ++p) {
                    int h;
                    where(mine, p, h);
                    put<G::SH>(fw + mine.swapped(p), s[p] * ld4(K + (int64_t)h * G::N + mine.i));
                }
                __syncthreads();
            }
        }
        if (dR2) outer<32, 1>(gr, fw, wave, fresh(lane), [](int k) { return k * G::SH; }, sumR);
        stage_t<T, 1>(tring, gr, R2, wave, fresh(lane), [](int k) { return k * G::SH; });   // dmid -> dt, where t was
        __syncthreads();
        {
            const Share mine(fresh(threadIdx.x));
#pragma unroll
            for (int p = 0; p < Share::PIECES; ++p) {
                int h;
                const int64_t at = where(mine, p, h);
                if (!live(mine, p)) break;
                const f32x4 d = get<G::SH>(gr + mine.swapped(p));
                st4(ds + at, d * ld4(K + (int64_t)h * G::N + mine.i));
                s[p] *= d;
            }
        }
        if (dK) {
            {
                const int thread = fresh(threadIdx.x);
#pragma unroll
                for (int p = 0; p < Share::PIECES; ++p) *reinterpret_cast<f32x4 *>(fw + 2048 * p + 4 * thread) = s[p];   // row after row
            }
            __syncthreads();
            const float2 *column = reinterpret_cast<const float2 *>(fw) + fresh(threadIdx.x);
            const int live_rows = run.end - q0 < G::TV ? (int)(run.end - q0) : G::TV;
            int h = h0, b = b0;
#pragma unroll 1
            for (int v4 = 0; v4 < G::TV; v4 += 4) {
                float2 x[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) x[e] = column[512 * (v4 + e)];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (v4 + e >= live_rows) break;
                    dk.x += x[e].x;
                    dk.y += x[e].y;
                    if (++b == B) {
                        store_dk(h++);
                        b = 0;
                    }
                }
            }
            if (b && q0 + G::TV >= run.end) store_dk(h);
        }
        __syncthreads();
    }
    if (dL2) flush<32>(dL2, wave, fresh(lane), sumL);
    if (dR2) flush<32>(dR2, wave, fresh(lane), sumR);
}

// dK of the channels that several workgroups share: workgroup w joins the channel that begins among its rows and goes on after
// them, parts in the order of the workgroups
__global__ __launch_bounds__(256) void join_dk_kernel(const float *__restrict__ parts, float *__restrict__ dK, int B, int64_t rows, int grid)
{
    const int w = blockIdx.x;
    const TileRun run(rows, w, grid);
    const int64_t h = run.end / B, next = (h + 1) * B;   // the channel at the end of the run
    if (run.end % B == 0 || h * B < run.begin) return;
    const float *at = parts + 4 * threadIdx.x;
    f32x4 sum = ld4(at + (2 * (int64_t)w + 1) * Geo<32>::N);
    for (int q = w + 1; q < grid; ++q) {
        const TileRun other(rows, q, grid);
        sum += ld4(at + 2 * (int64_t)q * Geo<32>::N);
        if (other.end >= next) break;
    }
    st4(dK + h * Geo<32>::N + 4 * threadIdx.x, sum);
}

// ---- gradients (blocks of 64) ----------------------------------------------------------------------------------
// The factor gradients (b^3 = 262144 floats each) do not fit in a workgroup's registers, and two tiles of eight rows
// do not fit in LDS.  Three launches:
//   dx: one tile of eight rows, the transposed stages of L and R (as the forward product, reversed);
//   dL: workgroup (group g, slice) sums the 16 blocks r = 16 g .. 16 g + 15, one per wave, over the tiles of its
//       slice of the rows: x whole (tile of four rows), the R stage restricted to the output rows r of the group
//       (one row tile per block k), dy only at (r, s) with r in the group (a compact tile);
//   dR: the same with the 16 blocks k of a group: dy whole, the transposed L stage restricted to the outputs k of
//       the group, x only at (c, k) with k in the group.
// A factor's gradient is then one MFMA per block and 16 x 16 piece (contraction index = the tile's four rows).
constexpr int TV64 = 4;                 // rows of a gradient tile at b = 64
constexpr int CP64 = 16 * 68 + 1;       // floats per row of the compact tile holding (r, s), r in a group of 16: r' 68 + s
constexpr int CX64 = 64 * 20 + 1;       // floats per row of the compact tile holding (c, k), k in a group of 16: c 20 + k'

// One factor in place, restricted to row tile rt0 of every block's outputs (the other positions keep their inputs).
template <typename T, int BS, int SK, bool TRANS, typename At>
__device__ __forceinline__ void stage_one(float *tile, const T *__restrict__ W, int wave, int lane, At at, int rt0, int tv)
{
    typedef Geo<BS> G;
    const int l16 = lane & 15, kg = lane >> 4;
    float *mine = tile + (l16 & (tv - 1)) * G::ROWP;
    constexpr int WV = G::Q / 4;
    f32x4 w[2][WV];
    float anchor = 0.0f;
    auto request = [&](int u, f32x4 (&dst)[WV]) {
        const T *src = W;
        asm volatile("" : "+s"(src) : "v"(anchor));
        const int blk = wave * G::NBW + u;
        if constexpr (TRANS) {
            const T *col = src + ((size_t)blk * BS + G::Q * kg) * BS + 16 * rt0 + l16;
#pragma unroll
            for (int p = 0; p < WV; ++p)
#pragma unroll
                for (int e = 0; e < 4; ++e) dst[p][e] = ld1(col + (size_t)(4 * p + e) * BS);
        } else {
            const T *row = src + ((size_t)blk * BS + 16 * rt0 + l16) * BS + G::Q * kg;
#pragma unroll
            for (int p = 0; p < WV; ++p) dst[p] = ld4(row + 4 * p);
        }
    };
    request(0, w[0]);
#pragma unroll
    for (int u = 0; u < G::NBW; ++u) {
        float *e = mine + at(wave * G::NBW + u);
        float bv[G::Q];
#pragma unroll
        for (int j = 0; j < G::Q; ++j) bv[j] = e[(G::Q * kg + j) * SK];
        if (u + 1 < G::NBW) request(u + 1, w[(u + 1) & 1]);
        f32x4 a = {0, 0, 0, 0};
#pragma unroll
        for (int j = 0; j < G::Q; ++j) a = mfma(w[u & 1][j >> 2][j & 3], bv[j], a);
        anchor = a[0];
        if (l16 < tv) {
#pragma unroll
            for (int r = 0; r < 4; ++r) e[(16 * rt0 + 4 * kg + r) * SK] = a[r];
        }
    }
}

template <typename T>
__global__ __launch_bounds__(1024, 1) void backward64_dx_kernel(const T *__restrict__ R, const T *__restrict__ L, const T *__restrict__ dy,
                                                                  T *__restrict__ dx, int64_t batch)
{
    typedef Geo<64> G;
    constexpr int BS = 64;
    extern __shared__ __attribute__((aligned(16))) float tile[];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int64_t ntiles = (batch + G::TV - 1) / G::TV;
    for (int64_t t = blockIdx.x; t < ntiles; t += gridDim.x) {
        const int64_t v0 = t * G::TV;
        for (int piece = threadIdx.x; piece < G::TV * G::N / 4; piece += G::THREADS) {
            const int v = piece / (G::N / 4), i = 4 * (piece % (G::N / 4));
            int64_t r = v0 + v;
            if (r >= batch) r = batch - 1;   // (rows past the end: computed, never stored)
            const f32x4 g = ld4(dy + r * G::N + i);
            float *sp = tile + v * G::ROWP + (i % BS) * G::SH + i / BS;   // dy[s b + r] at (r, s)
            sp[0] = g[0]; sp[G::SH] = g[1]; sp[2 * G::SH] = g[2]; sp[3 * G::SH] = g[3];
        }
        __syncthreads();
        stage<T, BS, 1, true>(tile, L, wave, lane, [](int r) { return r * G::SH; });   // dy -> dmid at (r, k)
        __syncthreads();
        stage<T, BS, G::SH, true>(tile, R, wave, lane, [](int k) { return k; });       // dmid -> dx at (c, k)
        __syncthreads();
        for (int piece = threadIdx.x; piece < G::TV * G::N / 4; piece += G::THREADS) {
            const int v = piece / (G::N / 4), i = 4 * (piece % (G::N / 4));
            const float *sp = tile + v * G::ROWP + (i / BS) * G::SH + i % BS;
            if (v0 + v < batch) st4(dx + (v0 + v) * G::N + i, f32x4{sp[0], sp[1], sp[2], sp[3]});
        }
        __syncthreads();
    }
}

// WHICH = 0: dL (group of blocks r), 1: dR (group of blocks k).  blockIdx.x = 4 slice + group.
template <typename T, int WHICH>
__global__ __launch_bounds__(1024, 1) void backward64_factor_kernel(const T *__restrict__ x, const T *__restrict__ W,
                                                                      const T *__restrict__ dy, float *__restrict__ dW, int64_t batch)
{
    typedef Geo<64> G;
    constexpr int BS = 64, TV = TV64, CP = WHICH == 0 ? CP64 : CX64;
    extern __shared__ __attribute__((aligned(16))) float tile[];
    float *full = tile, *part = tile + TV * G::ROWP;   // dL: full = x -> mid, part = dy(r in group, s); dR: full = dy -> dmid, part = x(c, k in group)
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int l16 = lane & 15, kg = lane >> 4;
    const int group = blockIdx.x & 3, slice = blockIdx.x >> 2, nslices = gridDim.x >> 2;
    f32x4 sum[4][4];
#pragma unroll
    for (int it = 0; it < 4; ++it)
#pragma unroll
        for (int jt = 0; jt < 4; ++jt) sum[it][jt] = f32x4{0, 0, 0, 0};
    const int64_t ntiles = (batch + TV - 1) / TV;
    for (int64_t t = slice; t < ntiles; t += nslices) {
        const int64_t v0 = t * TV;
        // the whole rows of one operand, 16 elements (64 bytes) per 64 of the other
        for (int piece = threadIdx.x; piece < TV * G::N / 4; piece += G::THREADS) {
            const int v = piece / (G::N / 4), i = 4 * (piece % (G::N / 4));
            const bool live = v0 + v < batch;
            const int64_t r = live ? v0 + v : batch - 1;
            if (WHICH == 0) {
                const f32x4 val = ld4(x + r * G::N + i);
                float *d = full + v * G::ROWP + (i / BS) * G::SH + i % BS;
                d[0] = val[0]; d[1] = val[1]; d[2] = val[2]; d[3] = val[3];
            } else {
                f32x4 g = ld4(dy + r * G::N + i);
                if (!live) g = f32x4{0, 0, 0, 0};
                float *sp = full + v * G::ROWP + (i % BS) * G::SH + i / BS;
                sp[0] = g[0]; sp[G::SH] = g[1]; sp[2 * G::SH] = g[2]; sp[3 * G::SH] = g[3];
            }
        }
        for (int piece = threadIdx.x; piece < TV * 64 * 4; piece += G::THREADS) {   // (one piece per thread)
            const int v = piece >> 8, hi = (piece >> 2) & 63, q = piece & 3;   // element hi b + 16 group + 4 q ..
            const bool live = v0 + v < batch;
            const int64_t r = live ? v0 + v : batch - 1;
            const int i = hi * BS + 16 * group + 4 * q;
            if (WHICH == 0) {   // dy[s b + r], s = hi, r = 16 group + 4 q + e  ->  (r', s) at r' 68 + s
                f32x4 g = ld4(dy + r * G::N + i);
                if (!live) g = f32x4{0, 0, 0, 0};
                float *sp = part + v * CP + (4 * q) * 68 + hi;
                sp[0] = g[0]; sp[68] = g[1]; sp[2 * 68] = g[2]; sp[3 * 68] = g[3];
            } else {            // x[c b + k], c = hi, k = 16 group + 4 q + e  ->  (c, k') at c 20 + k'
                const f32x4 val = ld4(x + r * G::N + i);
                float *d = part + v * CP + hi * 20 + 4 * q;
                d[0] = val[0]; d[1] = val[1]; d[2] = val[2]; d[3] = val[3];
            }
        }
        __syncthreads();
        if (WHICH == 0) stage_one<T, BS, G::SH, false>(full, W, wave, lane, [](int k) { return k; }, group, TV);        // mid(r, k), r in the group
        else stage_one<T, BS, 1, true>(full, W, wave, lane, [](int r) { return r * G::SH; }, group, TV);                // dmid(r, k), k in the group
        __syncthreads();
        // this wave's block: the MFMA's contraction index kg is row kg of the tiles
        {
            const int blk = 16 * group + wave;
            float a[4], b[4];
#pragma unroll
            for (int it = 0; it < 4; ++it) {
                if (WHICH == 0) {   // dL[r][s][k]: dy(r, s) from the compact tile, mid(r, k) from the full one
                    a[it] = part[kg * CP + wave * 68 + 16 * it + l16];
                    b[it] = full[kg * G::ROWP + blk * G::SH + 16 * it + l16];
                } else {            // dR[k][r][c]: dmid(r, k) from the full tile, x(c, k) from the compact one
                    a[it] = full[kg * G::ROWP + (16 * it + l16) * G::SH + blk];
                    b[it] = part[kg * CP + (16 * it + l16) * 20 + wave];
                }
            }
#pragma unroll
            for (int it = 0; it < 4; ++it)
#pragma unroll
                for (int jt = 0; jt < 4; ++jt) sum[it][jt] = mfma(a[it], b[jt], sum[it][jt]);
        }
        __syncthreads();
    }
    const int blk = 16 * group + wave;
#pragma unroll
    for (int it = 0; it < 4; ++it)
#pragma unroll
        for (int jt = 0; jt < 4; ++jt)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                atomicAdd(dW + ((size_t)blk * BS + 16 * it + 4 * kg + r) * BS + 16 * jt + l16, sum[it][jt][r]);
}

// ---- the polynomial-parameterised Monarch convolution (blocks of 32 and 64) --------------------------------------
// y = g_out o Re( M2 ( Kf o M1 (g_in o u, 0) ) )[0:n] with complex block-diagonal factors (appendix: the blocky
// Monarch convolution): the mixer's four stages on two planes of the tile (real and imaginary parts), a complex
// product being four real MFMA chains, two when the input is real (first stage) or only the real part is kept (last
// stage, which also skips the row tiles of its outputs past n).  The factors are complex float32 [block][row][column]:
// a lane reads the (b/4) complex columns of its row as (b/2) consecutive floats.
template <int BS>
struct CGeo {   // rows of a tile: two planes of TV rows fit in LDS
    static constexpr int TV = BS == 32 ? 16 : 4;
    static constexpr size_t LDS_BYTES = 2 * sizeof(float) * TV * Geo<BS>::ROWP;
};

// RTMAX: row tiles of every block's outputs that are computed (the others keep their inputs).
template <int BS, int SK, bool REAL_IN, bool REAL_OUT, int RTMAX, typename At>
__device__ __forceinline__ void cstage(float *tre, float *tim, const float2 *__restrict__ W, int wave, int lane, At at)
{
    typedef Geo<BS> G;
    constexpr int TV = CGeo<BS>::TV;
    const int l16 = lane & 15, kg = lane >> 4;
    float *mre = tre + (l16 & (TV - 1)) * G::ROWP, *mim = tim + (l16 & (TV - 1)) * G::ROWP;
    // a lane's Q complex columns of a row come in halves of 8 (4 pieces of 16 bytes), the next half requested while the
    // current one is multiplied
    constexpr int HALVES = G::Q / 8, WV = 4;
    f32x4 w[2][WV];
    float anchor = 0.0f;
    constexpr int ITEMS = G::NBW * RTMAX * HALVES;
    auto request = [&](int item, f32x4 (&dst)[WV]) {
        const float2 *src = W;
        asm volatile("" : "+s"(src) : "v"(anchor));
        const int half = item % HALVES, rt = (item / HALVES) % RTMAX, blk = wave * G::NBW + item / (HALVES * RTMAX);
        const float *row = reinterpret_cast<const float *>(src + ((size_t)blk * BS + 16 * rt + l16) * BS + G::Q * kg + 8 * half);
#pragma unroll
        for (int p = 0; p < WV; ++p) dst[p] = ld4(row + 4 * p);
    };
    request(0, w[0]);
#pragma unroll
    for (int u = 0; u < G::NBW; ++u) {
        const int off = at(wave * G::NBW + u);
        float *ere = mre + off, *eim = mim + off;
        float bre[G::Q], bim[G::Q];
#pragma unroll
        for (int j = 0; j < G::Q; ++j) {
            bre[j] = ere[(G::Q * kg + j) * SK];
            if constexpr (!REAL_IN) bim[j] = eim[(G::Q * kg + j) * SK];
        }
        // (every input of the block is in registers by now: a row tile's results take their places at once)
#pragma unroll
        for (int rt = 0; rt < RTMAX; ++rt) {
            f32x4 ar = {0, 0, 0, 0}, ai = {0, 0, 0, 0}, sub = {0, 0, 0, 0};   // real part = ar - sub
#pragma unroll
            for (int half = 0; half < HALVES; ++half) {
                const int item = (u * RTMAX + rt) * HALVES + half;
                if (item + 1 < ITEMS) request(item + 1, w[(item + 1) & 1]);
                const f32x4 (&wc)[WV] = w[item & 1];
#pragma unroll
                for (int jj = 0; jj < 8; ++jj) {
                    const int j = 8 * half + jj;
                    const float wre = wc[jj >> 1][2 * (jj & 1)], wim = wc[jj >> 1][2 * (jj & 1) + 1];
                    ar = mfma(wre, bre[j], ar);
                    if constexpr (!REAL_IN) sub = mfma(wim, bim[j], sub);
                    if constexpr (!REAL_OUT) {
                        ai = mfma(wim, bre[j], ai);
                        if constexpr (!REAL_IN) ai = mfma(wre, bim[j], ai);
                    }
                }
            }
            ar -= sub;
            anchor = ar[0];
            if (l16 < TV) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    ere[(16 * rt + 4 * kg + r) * SK] = ar[r];
                    if constexpr (!REAL_OUT) eim[(16 * rt + 4 * kg + r) * SK] = ai[r];
                }
            }
        }
    }
}

template <typename T, int BS, bool GIN, bool GOUT>
__global__ __launch_bounds__(Geo<BS>::THREADS, 1) void blocky_kernel(
    const T *__restrict__ u, const T *__restrict__ g_in, const T *__restrict__ g_out, const float2 *__restrict__ R1,
    const float2 *__restrict__ L1, const float2 *__restrict__ R2, const float2 *__restrict__ L2, const float2 *__restrict__ Kf,
    T *__restrict__ y, int64_t rows, int H, int n)
{
    typedef Geo<BS> G;
    constexpr int TV = CGeo<BS>::TV;
    extern __shared__ __attribute__((aligned(16))) float tile[];
    float *tre = tile, *tim = tile + TV * G::ROWP;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int64_t ntiles = (rows + TV - 1) / TV;
    const int live_rt = ((n + BS - 1) / BS + 15) / 16;   // row tiles of the last stage that hold outputs below n
    for (int64_t t = blockIdx.x; t < ntiles; t += gridDim.x) {
        const int64_t v0 = t * TV;
        for (int piece = threadIdx.x; piece < TV * G::N / 4; piece += G::THREADS) {
            const int v = piece / (G::N / 4), i = 4 * (piece % (G::N / 4));
            int64_t r = v0 + v;
            if (r >= rows) r = rows - 1;   // (rows past the end: computed, never stored)
            f32x4 val = {0, 0, 0, 0};      // (n is a multiple of 4: a piece is inside the row or past it)
            if (i < n) {
                val = ld4(u + r * n + i);
                if (GIN) val *= ld4(g_in + r * n + i);
            }
            float *d = tre + v * G::ROWP + (i / BS) * G::SH + i % BS;
            d[0] = val[0]; d[1] = val[1]; d[2] = val[2]; d[3] = val[3];
        }
        __syncthreads();
        cstage<BS, G::SH, true, false, G::RT>(tre, tim, R1, wave, lane, [](int k) { return k; });
        __syncthreads();
        cstage<BS, 1, false, false, G::RT>(tre, tim, L1, wave, lane, [](int r) { return r * G::SH; });
        __syncthreads();
        // kernel product: entry m = s b + r of the transform domain sits at (r, s)
        for (int piece = threadIdx.x; piece < TV * G::N / 4; piece += G::THREADS) {
            const int v = piece / (G::N / 4), m = 4 * (piece % (G::N / 4));
            int64_t r = v0 + v;
            if (r >= rows) r = rows - 1;
            const float *kp = reinterpret_cast<const float *>(Kf + (r % H) * (int64_t)G::N + m);
            const f32x4 k01 = ld4(kp), k23 = ld4(kp + 4);
            const float kre[4] = {k01[0], k01[2], k23[0], k23[2]}, kim[4] = {k01[1], k01[3], k23[1], k23[3]};
            const int at = v * G::ROWP + (m % BS) * G::SH + m / BS;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float xr = tre[at + e * G::SH], xi = tim[at + e * G::SH];
                tre[at + e * G::SH] = xr * kre[e] - xi * kim[e];
                tim[at + e * G::SH] = xr * kim[e] + xi * kre[e];
            }
        }
        __syncthreads();
        cstage<BS, 1, false, false, G::RT>(tre, tim, R2, wave, lane, [](int k) { return k * G::SH; });
        __syncthreads();
        // (only the row tiles of the outputs below n)
        if (live_rt == 1) cstage<BS, G::SH, false, true, 1>(tre, tim, L2, wave, lane, [](int r) { return r; });
        else if (live_rt == 2 || G::RT == 2) cstage<BS, G::SH, false, true, 2>(tre, tim, L2, wave, lane, [](int r) { return r; });
        else if (live_rt == 3) cstage<BS, G::SH, false, true, (G::RT > 2 ? 3 : 2)>(tre, tim, L2, wave, lane, [](int r) { return r; });
        else cstage<BS, G::SH, false, true, G::RT>(tre, tim, L2, wave, lane, [](int r) { return r; });
        __syncthreads();
        for (int piece = threadIdx.x; piece < TV * G::N / 4; piece += G::THREADS) {
            const int v = piece / (G::N / 4), i = 4 * (piece % (G::N / 4));
            if (v0 + v < rows && i < n) {
                const float *sp = tre + v * G::ROWP + (i / BS) * G::SH + i % BS;
                f32x4 val = {sp[0], sp[1], sp[2], sp[3]};
                if (GOUT) val *= ld4(g_out + (v0 + v) * n + i);
                st4(y + (v0 + v) * n + i, val);
            }
        }
        __syncthreads();
    }
}

template <int BS>
static int grid_for(int64_t ntiles, int64_t *grid)
{
    int dev = 0, ncu = 0;
    MONARCH_HIP_CHECK(hipGetDevice(&dev));
    MONARCH_HIP_CHECK(hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev));
    *grid = (int64_t)ncu * (BS == 32 ? 2 : 1);
    if (*grid > ntiles) *grid = ntiles;
    return MONARCH_OK;
}

template <typename T, int BS>
static int launch_matmul(const void *x, const void *R, const void *L, void *y, int64_t batch, hipStream_t s)
{
    typedef Geo<BS> G;
    const int64_t ntiles = (batch + G::TV - 1) / G::TV;
    int64_t grid = 0;
    if (int rc = grid_for<BS>(ntiles, &grid)) return rc;
    // a compute unit for every part; matmul_kernel : matmul_few_kernel, us, at that line and past it: b = 64, 512 rows, fp32
    // 68.3 : 25.3, bf16 35.5 : 16.1 (one row 64.8 : 21.6, 31.1 : 12.3); b = 32, 2048 rows, fp32
    // 14.9 : 11.3, bf16 9.4 : 9.2, 4096 rows 15.8 : 17.6, 10.0 : 11.5
    const bool few = grid == ntiles && ntiles * G::RT <= 256;
    if (few) grid = ntiles * G::RT;
    auto kern = few ? matmul_few_kernel<T, BS> : matmul_kernel<T, BS>;
    MONARCH_HIP_CHECK(hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)G::LDS_BYTES));
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(G::THREADS), G::LDS_BYTES, s, (const T *)x, (const T *)R, (const T *)L, (T *)y, batch);
    MONARCH_HIP_CHECK(hipGetLastError());
    return MONARCH_OK;
}

template <typename T, int BS, bool GIN, bool GOUT>
static int launch_mixer_g(const void *u, const void *K, const void *g_in, const void *g_out, const void *R1, const void *L1,
                          const void *R2, const void *L2, void *y, int64_t rows, int H, const MixOpt &opt, hipStream_t s)
{
    typedef Geo<BS> G;
    int64_t grid = 0;
    if (int rc = grid_for<BS>((rows + G::TV - 1) / G::TV, &grid)) return rc;
    auto kern = opt.transposed ? mixer_kernel<T, BS, GIN, GOUT, true> : mixer_kernel<T, BS, GIN, GOUT, false>;
    MONARCH_HIP_CHECK(hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)G::LDS_BYTES));
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(G::THREADS), G::LDS_BYTES, s, (const T *)u, (const T *)K, (const T *)g_in,
                       (const T *)g_out, (const T *)R1, (const T *)L1, (const T *)R2, (const T *)L2, (T *)y, rows, H, opt);
    MONARCH_HIP_CHECK(hipGetLastError());
    return MONARCH_OK;
}

template <typename T, int BS>
static int launch_mixer_t(const void *u, const void *K, const void *g_in, const void *g_out, const void *R1, const void *L1,
                          const void *R2, const void *L2, void *y, int64_t rows, int H, const MixOpt &opt, hipStream_t s)
{
    if (g_in && g_out) return launch_mixer_g<T, BS, true, true>(u, K, g_in, g_out, R1, L1, R2, L2, y, rows, H, opt, s);
    if (g_in) return launch_mixer_g<T, BS, true, false>(u, K, g_in, g_out, R1, L1, R2, L2, y, rows, H, opt, s);
    if (g_out) return launch_mixer_g<T, BS, false, true>(u, K, g_in, g_out, R1, L1, R2, L2, y, rows, H, opt, s);
    return launch_mixer_g<T, BS, false, false>(u, K, g_in, g_out, R1, L1, R2, L2, y, rows, H, opt, s);
}


// a persistent workgroup per compute unit with both tiles
template <typename Kern>
static int gradient_grid(Kern kern, int64_t rows, unsigned *grid)
{
    typedef Geo<32> G;
    int dev = 0, ncu = 0;
    MONARCH_HIP_CHECK(hipGetDevice(&dev));
    MONARCH_HIP_CHECK(hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev));
    MONARCH_HIP_CHECK(hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)(2 * G::LDS_BYTES)));
    const int64_t ntiles = (rows + G::TV - 1) / G::TV;
    *grid = (unsigned)(ntiles < ncu ? ntiles : ncu);
    return MONARCH_OK;
}

template <typename T>
static int launch_backward32(const void *x, const void *g_in, const void *R, const void *L, const void *dy, void *dx, void *dg_in,
                             float *dR, float *dL, int64_t batch, hipStream_t s)
{
    const int set = (dx || dg_in ? 4 : 0) | (dR ? 2 : 0) | (dL ? 1 : 0);
    if (!set) return MONARCH_OK;
    auto kern = set == 4   ? backward_kernel<T, true, false, false>
                : set == 2 ? backward_kernel<T, false, true, false>
                : set == 1 ? backward_kernel<T, false, false, true>
                           : backward_kernel<T, true, true, true>;
    unsigned grid = 0;
    if (int rc = gradient_grid(kern, batch, &grid)) return rc;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(512), 2 * Geo<32>::LDS_BYTES, s, (const T *)x, (const T *)g_in, (const T *)R,
                       (const T *)L, (const T *)dy, (T *)dx, (T *)dg_in, dR, dL, batch);
    MONARCH_HIP_CHECK(hipGetLastError());
    return MONARCH_OK;
}

template <typename T>
static int launch_mixer_backward32(const void *u, const void *K, const void *g_in, const void *g_out, const void *R1, const void *L1,
                                   const void *R2, const void *L2, const void *dy, void *ds, void *du, float *dK, void *dg_in,
                                   void *dg_out, float *dR1, float *dL1, float *dR2, float *dL2, int64_t B, int H, hipStream_t s)
{
    unsigned grid = 0;
    const int64_t rows = B * H;
    if (int rc = gradient_grid(mixer_backward_kernel<T>, rows, &grid)) return rc;
    float *parts = (float *)((char *)ds + align_up(sizeof(T) * rows * Geo<32>::N, 256));
    hipLaunchKernelGGL((mixer_backward_kernel<T>), dim3(grid), dim3(512), 2 * Geo<32>::LDS_BYTES, s, (const T *)u, (const T *)K,
                       (const T *)g_in, (const T *)g_out, (const T *)R1, (const T *)L1, (const T *)R2, (const T *)L2, (const T *)dy,
                       (T *)ds, dK, parts, (T *)dg_out, dR2, dL2, (int)B, H);
    MONARCH_HIP_CHECK(hipGetLastError());
    bool shared = false;
    for (unsigned w = 0; dK && w < grid; ++w) shared = shared || TileRun(rows, w, grid).end % B != 0;
    if (shared) {
        hipLaunchKernelGGL(join_dk_kernel, dim3(grid), dim3(256), 0, s, parts, dK, (int)B, rows, (int)grid);
        MONARCH_HIP_CHECK(hipGetLastError());
    }
    return launch_backward32<T>(u, g_in, R1, L1, ds, du, dg_in, dR1, dL1, rows, s);
}

template <typename T>
static int launch_backward64(const void *x, const void *R, const void *L, const void *dy, void *dx, float *dR, float *dL, int64_t batch,
                             hipStream_t s)
{
    typedef Geo<64> G;
    int dev = 0, ncu = 0;
    MONARCH_HIP_CHECK(hipGetDevice(&dev));
    MONARCH_HIP_CHECK(hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev));
    if (dx) {
        const int64_t ntiles = (batch + G::TV - 1) / G::TV;
        const unsigned grid = (unsigned)(ntiles < ncu ? ntiles : ncu);
        auto kern = backward64_dx_kernel<T>;
        MONARCH_HIP_CHECK(hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)G::LDS_BYTES));
        hipLaunchKernelGGL(kern, dim3(grid), dim3(1024), G::LDS_BYTES, s, (const T *)R, (const T *)L, (const T *)dy, (T *)dx, batch);
        MONARCH_HIP_CHECK(hipGetLastError());
    }
    const int64_t ntiles = (batch + TV64 - 1) / TV64;
    int64_t slices = ncu / 4 > 0 ? ncu / 4 : 1;   // four groups of blocks per slice of the rows: one workgroup per compute unit
    if (slices > ntiles) slices = ntiles;
    if (dL) {
        const size_t lds = sizeof(float) * TV64 * (G::ROWP + CP64);
        auto kern = backward64_factor_kernel<T, 0>;
        MONARCH_HIP_CHECK(hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
        hipLaunchKernelGGL(kern, dim3((unsigned)(4 * slices)), dim3(1024), lds, s, (const T *)x, (const T *)R, (const T *)dy, dL, batch);
        MONARCH_HIP_CHECK(hipGetLastError());
    }
    if (dR) {
        const size_t lds = sizeof(float) * TV64 * (G::ROWP + CX64);
        auto kern = backward64_factor_kernel<T, 1>;
        MONARCH_HIP_CHECK(hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
        hipLaunchKernelGGL(kern, dim3((unsigned)(4 * slices)), dim3(1024), lds, s, (const T *)x, (const T *)L, (const T *)dy, dR, batch);
        MONARCH_HIP_CHECK(hipGetLastError());
    }
    return MONARCH_OK;
}


template <typename T, int BS>
static int launch_blocky_t(const void *u, const void *g_in, const void *g_out, const float2 *R1, const float2 *L1, const float2 *R2,
                           const float2 *L2, const float2 *Kf, void *y, int64_t rows, int H, int n, hipStream_t s)
{
    typedef Geo<BS> G;
    int dev = 0, ncu = 0;
    MONARCH_HIP_CHECK(hipGetDevice(&dev));
    MONARCH_HIP_CHECK(hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev));
    const int64_t ntiles = (rows + CGeo<BS>::TV - 1) / CGeo<BS>::TV;
    const unsigned grid = (unsigned)(ntiles < ncu ? ntiles : ncu);   // one workgroup per compute unit
#define MONARCH_INPL_BLOCKY(GI, GO)                                                                                        \
    do {                                                                                                                   \
        auto kern = blocky_kernel<T, BS, GI, GO>;                                                                          \
        MONARCH_HIP_CHECK(hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)CGeo<BS>::LDS_BYTES)); \
        hipLaunchKernelGGL(kern, dim3(grid), dim3(G::THREADS), CGeo<BS>::LDS_BYTES, s, (const T *)u, (const T *)g_in, (const T *)g_out, \
                           R1, L1, R2, L2, Kf, (T *)y, rows, H, n);                                                        \
    } while (0)
    if (g_in && g_out) MONARCH_INPL_BLOCKY(true, true);
    else if (g_in) MONARCH_INPL_BLOCKY(true, false);
    else if (g_out) MONARCH_INPL_BLOCKY(false, true);
    else MONARCH_INPL_BLOCKY(false, false);
#undef MONARCH_INPL_BLOCKY
    MONARCH_HIP_CHECK(hipGetLastError());
    return MONARCH_OK;
}

}  // namespace inpl

bool monarch_inplace_supported(int bs, monarch_dtype dt) { return (bs == 32 || bs == 64) && (dt == MONARCH_F32 || dt == MONARCH_BF16); }

int launch_matmul_inplace(const void *x, const void *R, const void *L, void *y, int64_t batch, int bs, monarch_dtype dt, hipStream_t s)
{
    if (batch == 0) return MONARCH_OK;
    if (bs == 32) return dt == MONARCH_F32 ? inpl::launch_matmul<float, 32>(x, R, L, y, batch, s) : inpl::launch_matmul<bf16_t, 32>(x, R, L, y, batch, s);
    return dt == MONARCH_F32 ? inpl::launch_matmul<float, 64>(x, R, L, y, batch, s) : inpl::launch_matmul<bf16_t, 64>(x, R, L, y, batch, s);
}

// transposed access needs whole tiles inside a batch entry
bool mixer_inplace_takes(int bs, int H, monarch_dtype dt, const MixOpt &opt)
{
    if (!monarch_inplace_supported(bs, dt) || opt.act > 1) return false;
    return !opt.transposed || H % (bs == 32 ? inpl::Geo<32>::TV : inpl::Geo<64>::TV) == 0;
}

int launch_mixer_inplace(const void *u, const void *K, const void *g_in, const void *g_out, const void *R1, const void *L1,
                         const void *R2, const void *L2, void *y, int64_t rows, int H, int bs, monarch_dtype dt, const MixOpt &opt,
                         hipStream_t s)
{
    if (rows == 0) return MONARCH_OK;
    if (bs == 32)
        return dt == MONARCH_F32 ? inpl::launch_mixer_t<float, 32>(u, K, g_in, g_out, R1, L1, R2, L2, y, rows, H, opt, s)
                                 : inpl::launch_mixer_t<bf16_t, 32>(u, K, g_in, g_out, R1, L1, R2, L2, y, rows, H, opt, s);
    return dt == MONARCH_F32 ? inpl::launch_mixer_t<float, 64>(u, K, g_in, g_out, R1, L1, R2, L2, y, rows, H, opt, s)
                             : inpl::launch_mixer_t<bf16_t, 64>(u, K, g_in, g_out, R1, L1, R2, L2, y, rows, H, opt, s);
}

bool monarch_inplace_backward_supported(int bs, monarch_dtype dt) { return (bs == 32 || bs == 64) && (dt == MONARCH_F32 || dt == MONARCH_BF16); }

// dR and dL must have been cleared; batch > 0.
int launch_matmul_backward_inplace(const void *x, const void *R, const void *L, const void *dy, void *dx, float *dR, float *dL,
                                   int64_t batch, int bs, monarch_dtype dt, hipStream_t s)
{
    if (bs == 64)
        return dt == MONARCH_F32 ? inpl::launch_backward64<float>(x, R, L, dy, dx, dR, dL, batch, s)
                                 : inpl::launch_backward64<bf16_t>(x, R, L, dy, dx, dR, dL, batch, s);
    return dt == MONARCH_F32 ? inpl::launch_backward32<float>(x, nullptr, R, L, dy, dx, nullptr, dR, dL, batch, s)
                             : inpl::launch_backward32<bf16_t>(x, nullptr, R, L, dy, dx, nullptr, dR, dL, batch, s);
}

// (the kernel counts the rows of a channel in 32 bits)
bool mixer_backward_inplace_takes(int64_t B, int bs, monarch_dtype dt)
{
    return bs == 32 && B > 0 && B < (1 << 30) && (dt == MONARCH_F32 || dt == MONARCH_BF16);
}

// The factor gradients must have been cleared; scratch: mixer_backward_workspace_bytes, of it ds takes the size of u and the
// parts of dK two rows of fp32 per workgroup (at most 8 KB per tile of 16 rows, against 8 KB per row).
int launch_mixer_backward_inplace(const void *u, const void *K, const void *g_in, const void *g_out, const void *R1, const void *L1,
                                  const void *R2, const void *L2, const void *dy, void *scratch, void *du, float *dK, void *dg_in,
                                  void *dg_out, float *dR1, float *dL1, float *dR2, float *dL2, int64_t B, int H, monarch_dtype dt,
                                  hipStream_t s)
{
    return dt == MONARCH_F32 ? inpl::launch_mixer_backward32<float>(u, K, g_in, g_out, R1, L1, R2, L2, dy, scratch, du, dK, dg_in, dg_out,
                                                                    dR1, dL1, dR2, dL2, B, H, s)
                             : inpl::launch_mixer_backward32<bf16_t>(u, K, g_in, g_out, R1, L1, R2, L2, dy, scratch, du, dK, dg_in, dg_out,
                                                                     dR1, dL1, dR2, dL2, B, H, s);
}

// rows of a multiple of 4 elements (16-byte pieces of fp32 rows, 8-byte pieces of bf16 rows)
bool blocky_inplace_takes(int bs, int n, monarch_dtype dt) { return monarch_inplace_supported(bs, dt) && n >= 4 && n % 4 == 0; }

int launch_blocky_inplace(const void *u, const void *g_in, const void *g_out, const float2 *R1, const float2 *L1, const float2 *R2,
                          const float2 *L2, const float2 *Kf, void *y, int64_t rows, int H, int n, int bs, monarch_dtype dt, hipStream_t s)
{
    if (bs == 32)
        return dt == MONARCH_F32 ? inpl::launch_blocky_t<float, 32>(u, g_in, g_out, R1, L1, R2, L2, Kf, y, rows, H, n, s)
                                 : inpl::launch_blocky_t<bf16_t, 32>(u, g_in, g_out, R1, L1, R2, L2, Kf, y, rows, H, n, s);
    return dt == MONARCH_F32 ? inpl::launch_blocky_t<float, 64>(u, g_in, g_out, R1, L1, R2, L2, Kf, y, rows, H, n, s)
                             : inpl::launch_blocky_t<bf16_t, 64>(u, g_in, g_out, R1, L1, R2, L2, Kf, y, rows, H, n, s);
}

}  // namespace monarch
