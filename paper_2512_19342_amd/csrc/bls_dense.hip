// bls_mlp_layer and bls_interact: the dense part of the model around the lookup (apply_mlp and
// interact_features of Listings 1 and 2), fp32 in and out, on the matrix cores.
//
// Operand layouts.  v_mfma_f32_32x32x2_f32: lane l supplies A[l % 32][l / 32] and B[l / 32][l % 32].
// v_mfma_f32_32x32x16_bf16: lane l supplies the eight k from 8 * (l / 32) of row (column) l % 32.  Both:
// accumulator register v of lane l is element (8 * (v / 4) + 4 * (l / 32) + v % 4, l % 32).
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "bls_internal.h"

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef f32x4 f32x4_a4 __attribute__((aligned(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kThreads = 256;
constexpr int kAllK = 16;                                     // layers of up to 16 k: all nine products

template <int ACT>
__device__ __forceinline__ float activate(float v)
{
    if constexpr (ACT == BLS_ACT_RELU) return v > 0.f ? v : 0.f;
    else if constexpr (ACT == BLS_ACT_SIGMOID) return 1.f / (1.f + expf(-v));
    else return v;
}

// ---- one layer: Y[M][N] = act(X[M][K] * W[N][K]^T + bias[N]) ---------------------------------
//
// fp32 operands on the bf16 matrix instructions.  A float times 2^16 is the sum of three bf16 numbers,
// exactly (24 significant bits, eight in each, the second and third being what rounding to nearest left;
// bf16 ends at 2^-133, floats at 2^-149), and of the nine products of two such sums the six largest are
// added up in fp32; what is left out is at most 2^-24 of the product, as much as the rounding of one fp32
// multiply-add.  Up to 16 k, one step, all nine are taken: with one or two products that are not zero the six
// would be further off than the fp32 instruction (K = 1: 1.7 units of 2^-24 instead of 1).  A longer row with
// a single value that is not zero still is.
// v_mfma_f32_32x32x16_bf16 takes 32 cycles for 16 k, v_mfma_f32_32x32x2_f32 64 for 2: six of the
// former against eight of the latter are 192 cycles against 512.  The products of the first parts and
// the five small ones have an accumulator each: one rounding of the large sum per 16 k.  Against 64
// bits the error is a third of the fp32 instruction's (2-norm, K = 1024: 1.5e-7 and 4.1e-7; K = 2208:
// 2.2e-7 and 5.9e-7; K = 13: 3.9e-8 and 6.7e-8); with one accumulator for all six it is larger
// (K = 1024: 4.7e-7).
//
// Conversion and instruction keep subnormal numbers, so small operands lose nothing, and sums that are
// 2^32 times the result lose nothing below 2^-126 (unscaled, operands of 2^-116 were 15 times over the
// error bound; the eight multiplications a chunk cost up to 5 % of a layer's time).
//
// A result that is not finite says nothing (an infinity has no three parts, and a float of 2^112 and more
// or a sum of 2^96 and more neither): it is taken again on the fp32 matrix instructions.  A finite one
// had finite operands: no product of an infinity or a NaN is finite.
//
// A workgroup of four wavefronts, two by two, owns a tile of 64 TI x 64 TJ; each wavefront multiplies
// 32 TI x 32 TJ.  Every element is summed over k in the same order whatever the tile, so that a
// sample's result does not depend on how many others are in the call.
// Tiles are staged already split, in planes of eight k: what a lane needs of a row is one 16-byte
// read, rows consecutive; two buffers, and the loads of two further steps in flight while one is
// multiplied.  Whole steps are loaded without a branch and the splitting is spread behind the multiplies
// (a branch per chunk made the compiler wait for the loads before the first multiply: 394 us for
// 16384 x 2208 -> 1024 instead of 375, 28 for 512 x 1024 -> 1024 instead of 21).  Workgroups are numbered so
// that those that share rows of X follow each other on one XCD (one L2), N-tile fastest.
//
// M = 16384, us, fp32 instructions / this: 2208 -> 1024 594 / 398 (186 TFLOP/s; 377 to 425 from card to card),
// 1024 -> 1024 284 / 186, 1024 -> 512 155 / 96, 512 -> 256 55 / 33, 256 -> 128 33 / 13.3.  M = 2048 (mlp_split): 415 -> 1024
// 52 / 17, 1024 -> 1024 96 / 33, 512 -> 256 52 / 11.  Counted for the first (413 us under the profiler, 672000
// cycles, i.e. 1.63 GHz: the card lowers its clock under these products): matrix pipe busy 63 % of the cycles,
// vector operations issued 45 %, LDS 32 %, no bank conflicts; a wavefront waits 43 % of its time for its turn to
// issue and 19 % for data or a barrier.
__device__ __forceinline__ bool finite(float v) { return __builtin_fabsf(v) <= 3.402823466e38f; }

struct Chunk { float v[8]; };                                 // eight consecutive k of one row

// A chunk asked for at k that was loaded as the last eight of a row of K: zeros for what comes before k.
__device__ __forceinline__ void clear_before(Chunk &c, int k, int K)
{
    const int gone = K < 8 ? 0 : k - std::min(k, K - 8);
#pragma unroll
    for (int j = 0; j < 8; ++j) c.v[j] = j < gone ? 0.f : c.v[j];
}

// Eight floats from k of a row of K; rows need no alignment beyond the float's.  WHOLE: all eight are there.
// Otherwise zeros stand for what is not: a row's last eight are loaded, without a branch, and those before k cleared
// (rows of fewer than eight: from K on).  us, a branch per chunk and float / this: 10^6 x 13 -> 16 49 / 39, 10^5 x 5 -> 50
// 14.5 / 12.3, 300000 x 64 -> 64 62 / 61.
template <bool WHOLE>
__device__ __forceinline__ Chunk load_chunk(const float *__restrict__ row, int k, int K)
{
    Chunk c;
    f32x4 lo = 0.f, hi = 0.f;
    if (WHOLE || K >= 8) {
        const int at = WHOLE ? k : std::min(k, K - 8);
        lo = *reinterpret_cast<const f32x4_a4 *>(row + at);
        hi = *reinterpret_cast<const f32x4_a4 *>(row + at + 4);
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (k + j < K) lo[j] = row[k + j];
            if (k + 4 + j < K) hi[j] = row[k + 4 + j];
        }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) { c.v[j] = lo[j]; c.v[4 + j] = hi[j]; }
    if (!WHOLE && K >= 8) clear_before(c, k, K);
    return c;
}

// Two floats as bf16 (to nearest), the first in the low half; what they leave is returned in place.
__device__ __forceinline__ uint32_t take_bf16(float &a, float &b)
{
    const f32x2 v = {a, b};
    const uint32_t p = __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
    a -= __uint_as_float(p << 16);                            // exact
    b -= __uint_as_float(p & 0xffff0000u);
    return p;
}

// The three parts of a chunk times 2^16.
__device__ __forceinline__ void split(Chunk c, u32x4 (&part)[3])
{
#pragma unroll
    for (int j = 0; j < 8; ++j) c.v[j] *= 0x1p16f;
#pragma unroll
    for (int p = 0; p < 3; ++p)
#pragma unroll
        for (int j = 0; j < 4; ++j) part[p][j] = take_bf16(c.v[2 * j], c.v[2 * j + 1]);
}

// 32 rows of X from `row` times 32 TJ rows of W from `col` on the fp32 instruction: 16 bytes a lane at a time,
// lanes 0 to 31 hold k to k + 3 and the others k + 4 to k + 7.
template <int TJ>
__device__ __forceinline__ void multiply_fp32(f32x16 (&s)[TJ], const float *__restrict__ X, const float *__restrict__ W,
                                              int64_t M, int N, int K, int64_t row, int col)
{
    const int half = (threadIdx.x & 63) >> 5, l32 = threadIdx.x & 31;
    const float *x = X + std::min<int64_t>(row + l32, M - 1) * K, *w[TJ];
#pragma unroll
    for (int j = 0; j < TJ; ++j) {
        w[j] = W + (int64_t)std::min(col + 32 * j + l32, N - 1) * K;
        s[j] = 0.f;
    }
    auto step = [&](f32x4 a, const f32x4 (&b)[TJ]) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < TJ; ++j) s[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i], b[j][i], s[j], 0, 0, 0);
    };
    int k = 4 * half;
    const int whole = K / 8;
#pragma unroll 4
    for (int n = 0; n < whole; ++n, k += 8) {
        f32x4 b[TJ];
#pragma unroll
        for (int j = 0; j < TJ; ++j) b[j] = *reinterpret_cast<const f32x4_a4 *>(w[j] + k);
        step(*reinterpret_cast<const f32x4_a4 *>(x + k), b);
    }
    if (8 * whole < K) {
        f32x4 a = 0.f, b[TJ];
#pragma unroll
        for (int j = 0; j < TJ; ++j) b[j] = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (k + i < K) {
                a[i] = x[k + i];
#pragma unroll
                for (int j = 0; j < TJ; ++j) b[j][i] = w[j][k + i];
            }
        step(a, b);
    }
}

// Results of 128 MB and more are stored with the streaming hint: the next layer would not find them in the
// memory-side cache, and with few k the stores are the bound.  us, fp32 instruction / without the hint / with it,
// M K N: 1000000 13 128 (512 MB) 178 / 206 / 180, 131072 128 512 180 / 179 / 154, 65536 13 512 (128 MB) 48 / 54 / 49;
// 64 MB cost the layer that reads them next as much as they gain.
constexpr int64_t kStreamFloats = (int64_t)32 << 20;

// Sums r (2^32 times the result) of 32 rows from `row` and 32 TJ columns from `col`: scaled, those that are not
// finite taken again, bias and activation, stored.  The repeat is one pass of the wavefront over the rows' k for
// all its columns: a layer of 16384 x 2208 -> 1024 with one NaN among its samples takes 433 us (a sub-tile of 32 x 32
// after another with 4-byte loads: 662), with one in every sample 1134 (4165; the fp32 instruction alone: 594).
template <int ACT, int TJ>
__device__ __forceinline__ void finish(f32x16 (&r)[TJ], const float *__restrict__ X, const float *__restrict__ W,
                                       const float *__restrict__ bias, float *__restrict__ Y, int64_t M, int N, int K,
                                       int64_t row, int col)
{
    const int half = (threadIdx.x & 63) >> 5, l32 = threadIdx.x & 31;
    bool redo = false;
#pragma unroll
    for (int j = 0; j < TJ; ++j) {
#pragma unroll
        for (int v = 0; v < 16; ++v) redo = redo || !finite(r[j][v]);
#pragma unroll
        for (int v = 0; v < 16; ++v) r[j][v] *= 0x1p-32f;      // what is not finite stays so
    }
    if (__any(redo)) {
        f32x16 s[TJ];
        multiply_fp32<TJ>(s, X, W, M, N, K, row, col);
#pragma unroll
        for (int j = 0; j < TJ; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v)
                if (!finite(r[j][v])) r[j][v] = s[j][v];
    }
    auto store = [&](auto streaming) {
#pragma unroll
        for (int j = 0; j < TJ; ++j) {
            const int c = col + 32 * j + l32;
            if (c >= N) continue;
            const float bv = bias ? bias[c] : 0.f;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int64_t at = row + 8 * (v >> 2) + 4 * half + (v & 3);
                if (at >= M) continue;
                if constexpr (decltype(streaming)::value) __builtin_nontemporal_store(activate<ACT>(r[j][v] + bv), Y + at * N + c);
                else Y[at * N + c] = activate<ACT>(r[j][v] + bv);
            }
        }
    };
    if (M * N >= kStreamFloats) store(std::true_type());
    else store(std::false_type());
}

template <int TI, int TJ, int CH, int ACT>
__global__ __launch_bounds__(kThreads, 2) void mlp_gemm(const float *__restrict__ X, const float *__restrict__ W,
                                                        const float *__restrict__ bias, float *__restrict__ Y,
                                                        int64_t M, int N, int K, uint32_t n_tiles, uint32_t tiles)
{
    constexpr int BM = 64 * TI, BN = 64 * TJ, BK = 8 * CH;    // CH planes of eight k per step
    // rows per plane plus padding that spreads the planes one thread row writes over the banks
    constexpr int LA = BM + 8 / CH, LB = BN + 8 / CH;
    constexpr int SIDE_A = 3 * CH * LA, BUF = 3 * CH * (LA + LB);
    __shared__ u32x4 lds[2 * BUF];

    // XCD x gets the tiles [x * per, (x + 1) * per) in launch order
    const uint32_t per = (tiles + 7u) / 8u;
    const uint32_t tile = (blockIdx.x & 7u) * per + (blockIdx.x >> 3);
    if ((blockIdx.x >> 3) >= per || tile >= tiles) return;
    const int64_t m0 = (int64_t)(tile / n_tiles) * BM;
    const int n0 = (int)(tile % n_tiles) * BN;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = (wave >> 1) * 32 * TI, wn = (wave & 1) * 32 * TJ;
    const int half = lane >> 5, l32 = lane & 31;

    // thread tid stages planes c of rows r, r + 256 / CH, ...: CH threads read a row's step together
    constexpr int NA = BM * CH / kThreads, NB = BN * CH / kThreads, RSTEP = kThreads / CH;
    const int sr = tid / CH, sc = tid % CH;
    // rows past the last repeat it: what they give is not stored
    const float *xrow[NA], *wrow[NB];
#pragma unroll
    for (int i = 0; i < NA; ++i) {
        const int64_t row = m0 + sr + i * RSTEP;
        xrow[i] = X + (row < M ? row : M - 1) * K;
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int row = n0 + sr + i * RSTEP;
        wrow[i] = W + (int64_t)(row < N ? row : N - 1) * K;
    }
    struct Held { Chunk x[NA], w[NB]; } even, odd;            // of an even and of an odd step, on their way
    auto load = [&](Held &h, int k0, auto whole) {
#pragma unroll
        for (int i = 0; i < NA; ++i) h.x[i] = load_chunk<decltype(whole)::value>(xrow[i], k0 + 8 * sc, K);
#pragma unroll
        for (int i = 0; i < NB; ++i) h.w[i] = load_chunk<decltype(whole)::value>(wrow[i], k0 + 8 * sc, K);
    };
    const int steps = (K + BK - 1) / BK, full = K / BK;
    auto fetch = [&](Held &h, int step, auto whole) {         // nothing past the last step
        if (decltype(whole)::value || step < full) load(h, step * BK, std::true_type());
        else if (step < steps) load(h, step * BK, std::false_type());
    };
    auto put = [&](const Chunk &c, u32x4 *at, int plane) {    // the three parts lie CH planes apart
        u32x4 part[3];
        split(c, part);
#pragma unroll
        for (int p = 0; p < 3; ++p) at[p * CH * plane] = part[p];
    };
    auto stage = [&](const Held &h, int buf) {
#pragma unroll
        for (int i = 0; i < NA; ++i) put(h.x[i], lds + buf * BUF + sc * LA + sr + i * RSTEP, LA);
#pragma unroll
        for (int i = 0; i < NB; ++i) put(h.w[i], lds + buf * BUF + SIDE_A + sc * LB + sr + i * RSTEP, LB);
    };

    f32x16 acc[TI][TJ], low[TI][TJ];                          // sums of the first parts' products, of the rest
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < TJ; ++j) acc[i][j] = low[i][j] = 0.f;
    auto multiply = [&](int buf) {
#pragma unroll
        for (int kc = 0; kc < CH; kc += 2) {
            const u32x4 *pa = lds + buf * BUF + (kc + half) * LA + wm + l32;
            const u32x4 *pb = lds + buf * BUF + SIDE_A + (kc + half) * LB + wn + l32;
            bf16x8 a[3][TI], b[3][TJ];
#pragma unroll
            for (int p = 0; p < 3; ++p) {
#pragma unroll
                for (int i = 0; i < TI; ++i) a[p][i] = __builtin_bit_cast(bf16x8, pa[p * CH * LA + 32 * i]);
#pragma unroll
                for (int j = 0; j < TJ; ++j) b[p][j] = __builtin_bit_cast(bf16x8, pb[p * CH * LB + 32 * j]);
            }
#pragma unroll
            for (int o = 2; o >= 0; --o)                      // parts p and o - p
#pragma unroll
                for (int p = 0; p <= o; ++p)
#pragma unroll
                    for (int i = 0; i < TI; ++i)
#pragma unroll
                        for (int j = 0; j < TJ; ++j) {
                            f32x16 &sum = o ? low[i][j] : acc[i][j];
                            sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[p][i], b[o - p][j], sum, 0, 0, 0);
                        }
        }
    };

    // step t - 1 multiplied, step t put into the other buffer (nobody reads it now), step t + 2 asked for
    auto advance = [&](Held &h, int t, auto whole) {
        multiply((t - 1) & 1);
        stage(h, t & 1);
        fetch(h, t + 2, whole);
        // the reads first, then the splitting spread evenly behind the multiplies: 52 vector operations a chunk, asked
        // for as 72, so that the last multiplies have nothing left to hide (16384 x 1024 -> 512: 103.5 us as 52, 99.8)
        constexpr int kMfma = 3 * TI * TJ * CH, kValu = (72 * (NA + NB) + kMfma - 1) / kMfma, kWrites = 3 * (NA + NB);
        __builtin_amdgcn_sched_group_barrier(0x100, 3 * (TI + TJ) * CH / 2, 0);
#pragma unroll
        for (int i = 0; i < kMfma; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x002, kValu, 0);
            if ((i + 1) * kWrites / kMfma > i * kWrites / kMfma) __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x020, 2 * (NA + NB), 0);
        __syncthreads();
    };
    if (full >= 3) {
        load(even, 0, std::true_type());
        load(odd, BK, std::true_type());
        stage(even, 0);
        load(even, 2 * BK, std::true_type());
    } else {
        fetch(even, 0, std::false_type());
        fetch(odd, 1, std::false_type());
        stage(even, 0);
        fetch(even, 2, std::false_type());
    }
    __syncthreads();
    int t = 1;
    for (; t + 3 < full; t += 2) {                            // steps t + 2 and t + 3 are whole
        advance(odd, t, std::true_type());
        advance(even, t + 1, std::true_type());
    }
    for (; t < steps; t += 2) {
        advance(odd, t, std::false_type());
        if (t + 1 < steps) advance(even, t + 1, std::false_type());
    }
    multiply((steps - 1) & 1);
    if (K <= kAllK) {                                         // the three smallest products, of the only step
#pragma unroll 1
        for (int o = 4; o >= 2; --o) {
            const int p = o == 2 ? 1 : 2, q = o == 3 ? 1 : 2; // parts 2 2, 2 1, 1 2
#pragma unroll
            for (int i = 0; i < TI; ++i)
#pragma unroll
                for (int j = 0; j < TJ; ++j) {
                    const u32x4 a = lds[(p * CH + half) * LA + wm + l32 + 32 * i];
                    const u32x4 b = lds[SIDE_A + (q * CH + half) * LB + wn + l32 + 32 * j];
                    low[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b),
                                                                        low[i][j], 0, 0, 0);
                }
        }
    }

#pragma unroll
    for (int i = 0; i < TI; ++i) {
        f32x16 r[TJ];
#pragma unroll
        for (int j = 0; j < TJ; ++j) r[j] = acc[i][j] + low[i][j];
        finish<ACT>(r, X, W, bias, Y, M, N, K, m0 + wm + 32 * i, n0 + wn);
    }
}

// Tiles of 64 x 64 for the layers that do not fill the card with larger ones: few wavefronts per SIMD, so that
// splitting, LDS and multiplies of one wavefront follow each other more than they overlap (512 x 1024 -> 1024: 1300
// cycles a step of 32 k, of them 384 of multiplies).  Here they have wavefronts of their own: four multiply (32 x 32
// each), eight load, split and write, one chunk a step and thread, three per SIMD in all.  What bounds it: with one
// workgroup per compute unit or less the chain of a step, no part of which counts for more than an eighth (512 1024
// 1024, 18.3 us: without the splitting 16.5, without the loads 16.2, with a sixth of the multiplies 16.1); with two the
// multiplies (2048 1024 1024, 34.0: 29.5, 26.4, 23.0).
// us, four wavefronts for everything / this, M K N: 512 1024 1024 20.8 / 18.2, 512 415 1024 13.9 / 11.0, 512 512 256
// 12.2 / 10.5, 2048 1024 1024 34.1 / 32.7, 2048 1024 512 22.1 / 19.5, 2048 512 256 13.1 / 11.4, 16384 256 128
// 15.1 / 13.7.  Four wavefronts that split: 20.9 at the first; steps of 64 k: 18.2 there and 37.3 for 2048 1024 1024;
// tiles of 128 x 64 this way: 18.9 for 2048 415 1024 (17.3), 31.8 for 2048 1024 1024; three steps ahead: no change;
// no LDS, every wavefront splitting its own operands: 33.7 at the first, bound by the 32 lines a load touches.
// Every element is summed in mlp_gemm's order.
constexpr int kSplitThreads = 768;
template <int ACT>
__global__ __launch_bounds__(kSplitThreads, 6) void mlp_split(const float *__restrict__ X, const float *__restrict__ W,
                                                              const float *__restrict__ bias, float *__restrict__ Y,
                                                              int64_t M, int N, int K, uint32_t n_tiles, uint32_t tiles)
{
    constexpr int BM = 64, CH = 4, BK = 8 * CH;               // CH planes of eight k per step
    // rows of X, rows of W, and padding that spreads the planes one thread row writes over the banks
    constexpr int L = 2 * BM + 8 / CH, BUF = 3 * CH * L;
    __shared__ u32x4 lds[2 * BUF];

    // XCD x gets the tiles [x * per, (x + 1) * per) in launch order
    const uint32_t per = (tiles + 7u) / 8u;
    const uint32_t tile = (blockIdx.x & 7u) * per + (blockIdx.x >> 3);
    if ((blockIdx.x >> 3) >= per || tile >= tiles) return;
    const int64_t m0 = (int64_t)(tile / n_tiles) * BM;
    const int n0 = (int)(tile % n_tiles) * BM;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // scalar: the roles are a branch, not a mask
    const int steps = (K + BK - 1) / BK, full = K / BK;

    // Both roles pass `steps` barriers: step 0 is there, then one per further step.
    if (wave >= 4) {
        static_assert((kSplitThreads - 256) == 2 * BM * CH, "a chunk per thread");
        const int tid = threadIdx.x - 256, r = tid / CH, sc = tid % CH;
        // rows past the last repeat it: what they give is not stored
        const float *row = r < BM ? X + std::min<int64_t>(m0 + r, M - 1) * K : W + (int64_t)std::min(n0 + r - BM, N - 1) * K;
        auto load = [&](int step) {                           // past the last step its last eight again
            return load_chunk<true>(row, std::min(step * BK + 8 * sc, K - 8), K);
        };
        auto stage = [&](Chunk c, int step) {
            if (step == full) clear_before(c, step * BK + 8 * sc, K);
            u32x4 part[3];
            split(c, part);
#pragma unroll
            for (int p = 0; p < 3; ++p) lds[(step & 1) * BUF + (p * CH + sc) * L + r] = part[p];
        };
        Chunk even, odd;                                      // two steps on their way
        if (K >= 8) {
            even = load(0);
            odd = load(1);
            stage(even, 0);
            even = load(2);
        } else stage(load_chunk<false>(row, 8 * sc, K), 0);   // the only step
        __syncthreads();
        for (int t = 1; t < steps; t += 2) {
            stage(odd, t);
            odd = load(t + 2);
            __syncthreads();
            if (t + 1 < steps) {
                stage(even, t + 1);
                even = load(t + 3);
                __syncthreads();
            }
        }
        return;
    }

    const int lane = threadIdx.x & 63, half = lane >> 5, l32 = lane & 31;
    const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
    f32x16 acc[1], low = 0.f;                                 // sums of the first parts' products, of the rest
    acc[0] = 0.f;
    auto part = [&](int buf, int p, int c, int at) { return __builtin_bit_cast(bf16x8, lds[buf * BUF + (p * CH + c) * L + at]); };
    auto multiply = [&](int buf) {
#pragma unroll
        for (int kc = 0; kc < CH; kc += 2) {
            bf16x8 a[3], b[3];
#pragma unroll
            for (int p = 0; p < 3; ++p) {
                a[p] = part(buf, p, kc + half, wm + l32);
                b[p] = part(buf, p, kc + half, BM + wn + l32);
            }
#pragma unroll
            for (int o = 2; o >= 0; --o)                      // parts p and o - p
#pragma unroll
                for (int p = 0; p <= o; ++p) {
                    f32x16 &sum = o ? low : acc[0];
                    sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[p], b[o - p], sum, 0, 0, 0);
                }
        }
    };
    __syncthreads();
    for (int t = 1; t < steps; ++t) {
        multiply((t - 1) & 1);
        __syncthreads();
    }
    multiply((steps - 1) & 1);
    if (K <= kAllK) {                                         // the three smallest products, of the only step
#pragma unroll
        for (int o = 4; o >= 2; --o) {
            const int p = o == 2 ? 1 : 2, q = o == 3 ? 1 : 2; // parts 2 2, 2 1, 1 2
            low = __builtin_amdgcn_mfma_f32_32x32x16_bf16(part(0, p, half, wm + l32), part(0, q, half, BM + wn + l32), low, 0, 0, 0);
        }
    }
    acc[0] += low;
    finish<ACT>(acc, X, W, bias, Y, M, N, K, m0 + wm, n0 + wn);
}

// Layers of up to 64 k and 64 outputs, where a tile has nothing to keep the matrix pipe busy with: no LDS.  A lane's
// eight k of a row are the instruction's own layout, so a wavefront splits what it loads and multiplies; it keeps the
// parts of its 32 rows of W over `reps` blocks of 32 rows of X, the next block's loads in flight.  WN wavefronts side
// by side, 4 / WN below each other.
template <int WN, int STEPS, int ACT>
__global__ __launch_bounds__(kThreads) void mlp_short(const float *__restrict__ X, const float *__restrict__ W,
                                                      const float *__restrict__ bias, float *__restrict__ Y,
                                                      int64_t M, int N, int K, uint32_t n_tiles, uint32_t tiles, int reps)
{
    const uint32_t per = (tiles + 7u) / 8u;
    const uint32_t tile = (blockIdx.x & 7u) * per + (blockIdx.x >> 3);
    if ((blockIdx.x >> 3) >= per || tile >= tiles) return;
    constexpr int kRows = 32 * 4 / WN;
    const int half = (threadIdx.x & 63) >> 5, l32 = threadIdx.x & 31, wave = threadIdx.x >> 6;
    const int col = (int)(tile % n_tiles) * 32 * WN + 32 * (wave % WN);
    if (col >= N) return;
    int64_t row = (int64_t)(tile / n_tiles) * reps * kRows + 32 * (wave / WN);
    Chunk x[STEPS];
    auto chunk = [&](const float *at, int s) {                // K > 16 (STEPS - 1)
        const int k = 16 * s + 8 * half;
        return s + 1 < STEPS || K == 16 * STEPS ? load_chunk<true>(at, k, K) : load_chunk<false>(at, k, K);
    };
    auto load = [&]() {
        const float *at = X + std::min<int64_t>(row + l32, M - 1) * K;
#pragma unroll
        for (int s = 0; s < STEPS; ++s) x[s] = chunk(at, s);
    };
    load();
    u32x4 b[STEPS][3];
    const float *w = W + (int64_t)std::min(col + l32, N - 1) * K;
#pragma unroll
    for (int s = 0; s < STEPS; ++s) split(chunk(w, s), b[s]);
    for (int n = 0; n < reps && row < M; ++n) {
        u32x4 a[STEPS][3];
#pragma unroll
        for (int s = 0; s < STEPS; ++s) split(x[s], a[s]);
        const int64_t here = row;
        row += kRows;
        if (n + 1 < reps && row < M) load();
        f32x16 acc[1], low = 0.f;
        acc[0] = 0.f;
#pragma unroll
        for (int s = 0; s < STEPS; ++s)
#pragma unroll
            for (int o = 16 * STEPS <= kAllK ? 4 : 2; o >= 0; --o)    // parts p and o - p
#pragma unroll
                for (int p = std::max(0, o - 2); p <= std::min(o, 2); ++p) {
                    f32x16 &sum = o ? low : acc[0];
                    sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[s][p]),
                                                                  __builtin_bit_cast(bf16x8, b[s][o - p]), sum, 0, 0, 0);
                }
        acc[0] += low;
        finish<ACT>(acc, X, W, bias, Y, M, N, K, here, col);
    }
}

// One output per sample: a wavefront per row, the row's products summed lane by lane (k, k + 64, ...) and then
// across the lanes.  A matrix tile would split W for 64 columns.
constexpr int kNarrowK = 128;
template <int ACT>
__global__ __launch_bounds__(kThreads) void mlp_narrow(const float *__restrict__ X, const float *__restrict__ W,
                                                       const float *__restrict__ bias, float *__restrict__ Y, int64_t M, int K)
{
    const int lane = threadIdx.x & 63;
    const int64_t row = (int64_t)blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);
    if (row >= M) return;
    float sum = 0.f;
#pragma unroll 4
    for (int k = lane; k < K; k += 64) sum = fmaf(X[row * K + k], W[k], sum);
#pragma unroll
    for (int sh = 32; sh >= 1; sh >>= 1) sum += __shfl_xor(sum, sh, 64);
    if (lane == 0) Y[row] = activate<ACT>(sum + (bias ? bias[0] : 0.f));
}
// ---- dot interaction ---------------------------------------------------------------------------
//
// One workgroup per sample.  interact_gram (any D): the sample's T pooled vectors are copied to LDS (rows padded to a
// multiple of 32 with zeros, row stride odd so that 32 rows at one column fall in 32 banks); the
// 32 x 32 tiles on and below the diagonal of their Gram matrix are dealt to the wavefronts, each
// tile one accumulator over D / 2 matrix instructions; the last wavefront also takes the T
// products with the dense vector x.  Output row: x, then for i = 1..T the products of pooled
// vector i-1 with x and with pooled vectors 0..i-2.
// FROM_OUT: emb is the completed lookup [B][T][D].  FROM_SLOT, FROM_PARTIALS: emb is a ring slot in
// receive order and the copy to LDS is the completion itself - vector (b, t) is read where its owner put
// it, and for a row-wise partition the P partial vectors are added in increasing owner rank from
// +0, exactly as the copy-out kernel does.
// Memory bounds the kernel (16384 samples of 64 vectors of 128: 0.68 GB, 130 us at the rate of a copy).  A
// thread's eight loads of a round are all issued before the first is used: added up one by one as they
// come, a slot's took interact_gram 290 us at that size, this way 206 (interact_tiles 188).  Partial vectors of eight
// owners, interact_gram, us, one load after another / eight pieces of one partial at a time (four wavefronts per SIMD) /
// as it is (six): 16384 samples of 2 vectors 108 / 156 / 105, of 4 141 / 193 / 118, 8192 of 26 222 / 234 / 225.
enum Source { FROM_OUT, FROM_SLOT, FROM_PARTIALS };

// The sample's vectors in pieces of V (one float, or four), thread by thread, to rows of LD floats at Es.
// The d-th partial of vector t starts at vec0 + t_q[t] * vec_step + d * part_step (FROM_OUT: t for t_q[t]).
// A thread loads kFill pieces of a round together, of kParts partials each.  PIECES: every row of Es starts on a 16-byte
// boundary.  (Known when the kernel is built: asked while it runs, interact_gram took 3 to 5 % longer, 16384 samples of 8
// vectors of 24 35.1 / 36.8 us, and interact_tiles 2 %; both spilled a register for row-wise slots.)
template <Source SRC, typename V, int kFill, int kParts, bool PIECES>
__device__ __forceinline__ void fill_vectors(float *Es, uint32_t T, uint32_t D, uint32_t LD, int F, const float *vec0,
                                             const int32_t *__restrict__ t_q, int64_t vec_step, int64_t part_step)
{
    constexpr uint32_t W = sizeof(V) / sizeof(float);
    const uint32_t per = D / W, n = T * per, dr = kThreads / per, dc = kThreads % per;
    uint32_t r = threadIdx.x / per, c = threadIdx.x % per;
    for (uint32_t base = 0; base < n; base += kThreads * kFill) {
        const float *src[kFill];
        uint32_t at[kFill], col[kFill];
        int32_t q[kFill];
        bool live[kFill];
#pragma unroll
        for (int u = 0; u < kFill; ++u) {
            live[u] = r < T;
            at[u] = r * LD + c * W;
            col[u] = c * W;
            const uint32_t t = live[u] ? r : T - 1;           // no branch between the eight reads of t_q
            q[u] = SRC == FROM_OUT ? (int32_t)t : t_q[t];
            r += dr;
            c += dc;
            if (c >= per) { c -= per; ++r; }
        }
        // all of them waited for here, once: otherwise waits for t_q come between the vectors' loads
        if constexpr (SRC != FROM_OUT) {
#pragma unroll
            for (int u = 0; u < kFill; ++u) asm volatile("" : "+v"(q[u]));
        }
#pragma unroll
        for (int u = 0; u < kFill; ++u) src[u] = vec0 + q[u] * vec_step + col[u];
        V v[kFill];
#pragma unroll
        for (int u = 0; u < kFill; ++u) {
            v[u] = 0.f;
            if (SRC != FROM_PARTIALS && live[u]) v[u] = *reinterpret_cast<const V *>(src[u]);
        }
        if constexpr (SRC == FROM_SLOT) {
#pragma unroll
            for (int u = 0; u < kFill; ++u) v[u] = (V)(0.f) + v[u];   // a sum from +0: no negative zero
        }
        if constexpr (SRC == FROM_PARTIALS) {
            for (int d = 0; d < F; d += kParts) {
                V part[kParts][kFill];
#pragma unroll
                for (int p = 0; p < kParts; ++p)
#pragma unroll
                    for (int u = 0; u < kFill; ++u) {
                        part[p][u] = 0.f;
                        if (live[u] && d + p < F) part[p][u] = *reinterpret_cast<const V *>(src[u] + (d + p) * part_step);
                    }
#pragma unroll
                for (int p = 0; p < kParts; ++p)              // zeros past the last: no sum from +0 is -0
#pragma unroll
                    for (int u = 0; u < kFill; ++u) v[u] += part[p][u];
            }
        }
#pragma unroll
        for (int u = 0; u < kFill; ++u)
            if (live[u]) {
                if constexpr (W == 1) Es[at[u]] = v[u];
                else if constexpr (PIECES) *reinterpret_cast<V *>(Es + at[u]) = v[u];
                else {
#pragma unroll
                    for (uint32_t j = 0; j < W; ++j) Es[at[u] + j] = v[u][j];
                }
            }
    }
}

// The T vectors of a completed lookup in pieces of four floats: one stream, one address.  us, 16384 samples, interact_tiles
// with this / with fill_vectors: 1 vector of 128 42.3 / 47.2, 4 44.0 / 46.9, 12 50.2 / 48.3, 64 171 / 171; 2 of 64 30.5 /
// 33.6, 26 45.0 / 43.3; interact_gram, 12 of 20 34.3 / 38.9, 64 64.4 / 65.3; 2048 samples of 26 of 64 9.7 / 8.6.
template <int kFill, bool PIECES>
__device__ __forceinline__ void copy_vectors(float *Es, uint32_t T, uint32_t D, uint32_t LD, const float *vec0)
{
    const f32x4 *e = reinterpret_cast<const f32x4 *>(vec0);
    const uint32_t per = D / 4, n = T * per;
    for (uint32_t base = threadIdx.x; base < n; base += kThreads * kFill) {
        f32x4 v[kFill];
#pragma unroll
        for (int u = 0; u < kFill; ++u) {
            v[u] = 0.f;
            if (base + u * kThreads < n) v[u] = e[base + u * kThreads];
        }
#pragma unroll
        for (int u = 0; u < kFill; ++u) {
            const uint32_t i = base + u * kThreads, r = i / per, c = (i - r * per) * 4;
            if (i < n) {
                if constexpr (PIECES) *reinterpret_cast<f32x4 *>(Es + r * LD + c) = v[u];
                else {
#pragma unroll
                    for (int j = 0; j < 4; ++j) Es[r * LD + c + j] = v[u][j];
                }
            }
        }
    }
}

// Sample b's vectors to rows of LD floats at Es, from the completed lookup or out of a slot.
template <Source SRC, int kFill, int kParts, bool PIECES>
__device__ __forceinline__ void fetch_sample(const DevDesc &dd, float *Es, const float *emb, int64_t b, int T, int D, int LD, int vec4)
{
    int64_t slot_base = 0, slot_step = 0;                        // vector (q, b) of the slot: slot_base + q * slot_step
    if constexpr (SRC != FROM_OUT) {
        int s; uint32_t b_loc, n;
        bls_split_sample(dd, (uint32_t)b, s, b_loc, n);
        slot_base = (int64_t)dd.Q * dd.first[s] + b_loc;
        slot_step = n;
    }
    const float *vec0 = emb + (SRC == FROM_OUT ? b * T : slot_base) * D;
    const int64_t vec_step = SRC == FROM_OUT ? D : slot_step * D, part_step = dd.T * slot_step * D;
    if (SRC == FROM_OUT && vec4) copy_vectors<kFill, PIECES>(Es, T, D, LD, vec0);
    else if (vec4) fill_vectors<SRC, f32x4, kFill, kParts, PIECES>(Es, T, D, LD, dd.F, vec0, dd.t_q, vec_step, part_step);
    else fill_vectors<SRC, float, kFill, kParts, PIECES>(Es, T, D, LD, dd.F, vec0, dd.t_q, vec_step, part_step);
}

// D a multiple of 16: tiles of 16 x 16 on v_mfma_f32_16x16x4_f32 (lane l supplies A[l % 16][l / 16] and B[l / 16][l % 16];
// register v of lane l is element (4 * (l / 16) + v, l % 16)).  Lane group l / 16 takes the four k from 16 s + 4 (l / 16)
// of step s, so that four instructions are fed by one 16-byte read of a row; rows of D + 4 floats put the 16 rows of such
// a read on different banks.  Smaller tiles leave less above the diagonal and deal out evenly (64 vectors: 10 tiles of
// 1024 matrix cycles, three for the busiest wavefront, against three of 4096 and none for the fourth), the wavefronts
// change parts from sample to sample, so that no SIMD always has the longest, and the products with x are shared by all
// four.  Padding rows stay as they are: a product of theirs is stored nowhere.
// us, tiles of 32 x 32 / this: 16384 samples of 64 vectors of 128 185-199 / 178-190 (147 without the products: they
// still cost what the next samples' loads do not hide), 8192 of 26 of 128 50.2 / 38.8, of 64 of 112 94 / 89, 16384 of 2
// 78 / 42, 4096 of 30 of 256 51 / 39, 8192 of 100 of 64 139 / 117, 2048 of 26 of 64 10.2 / 9.0; a few samples of whole
// tiles of 32 x 32 lose: 64 vectors of 32, 128 samples 4.2 / 4.6, 2048 13.6 / 13.8, 16384 76 / 67; 200 of 16 13.1 / 14.6, 54 /
// 52, 559 / 526 (and a sample's result may not depend on how many others are in the call).  Half or a quarter of the
// columns at a time, for more workgroups per compute unit: 187, 227 at the first.
template <Source SRC, int kFill, int kParts>
__global__ __launch_bounds__(kThreads, SRC == FROM_PARTIALS ? 6 : 1) void interact_tiles(DevDesc dd, const float *__restrict__ x,
                                                           const float *__restrict__ emb, float *__restrict__ z, int T, int D,
                                                           int TP, uint32_t b0, int vec4)
{
    extern __shared__ __attribute__((aligned(16))) float lds[];
    const int LD = D + 4;
    float *Es = lds;                                          // [TP][LD]
    float *xsh = lds + (size_t)TP * LD;                       // [D]
    const int64_t b = (int64_t)b0 + blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = ((tid >> 6) + (blockIdx.x >> 3) + (blockIdx.x >> 8)) & 3;
    float *__restrict__ zb = z + b * ((int64_t)D + (int64_t)T * (T + 1) / 2);
    fetch_sample<SRC, kFill, kParts, true>(dd, Es, emb, b, T, D, LD, vec4);
    for (int c = tid; c < D; c += kThreads) {
        const float v = x[b * D + c];
        xsh[c] = v;
        zb[c] = v;
    }
    __syncthreads();

    const int g = lane >> 4, l16 = lane & 15;
    const int nt = TP / 16;
    int tile = 0;
    for (int ti = 0; ti < nt; ++ti)
        for (int tj = 0; tj <= ti; ++tj, ++tile) {
            if ((tile & 3) != wave) continue;
            f32x4 acc = 0.f;
            const float *pa = Es + (ti * 16 + l16) * LD + 4 * g;
            const float *pb = Es + (tj * 16 + l16) * LD + 4 * g;
            for (int k = 0; k < D; k += 16) {
                const f32x4 a = *reinterpret_cast<const f32x4 *>(pa + k), c = *reinterpret_cast<const f32x4 *>(pb + k);
#pragma unroll
                for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[j], c[j], acc, 0, 0, 0);
            }
            const int col = tj * 16 + l16;                    // the lower-numbered vector of the pair
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int row = ti * 16 + 4 * g + v;
                if (row < T && col < row) zb[D + (int64_t)(row + 1) * row / 2 + col + 1] = acc[v];
            }
        }
    for (int t0 = 16 * wave; t0 < T; t0 += 64) {
        const float *e = Es + (t0 + l16) * LD + 4 * g;
        float dot = 0.f;
        for (int k = 0; k < D; k += 16) {
            const f32x4 a = *reinterpret_cast<const f32x4 *>(e + k), c = *reinterpret_cast<const f32x4 *>(xsh + 4 * g + k);
#pragma unroll
            for (int j = 0; j < 4; ++j) dot = fmaf(a[j], c[j], dot);
        }
        dot += __shfl_xor(dot, 16, 64);
        dot += __shfl_xor(dot, 32, 64);
        const int t = t0 + l16;
        if (g == 0 && t < T) zb[D + (int64_t)(t + 1) * t / 2] = dot;
    }
}

template <Source SRC, int kFill, int kParts>
__global__ __launch_bounds__(kThreads, SRC == FROM_PARTIALS ? 6 : 1) void interact_gram(DevDesc dd, const float *__restrict__ x, const float *__restrict__ emb,
                                                          float *__restrict__ z, int T, int D, int TP, int LD,
                                                          uint32_t b0, int vec4)
{
    extern __shared__ float lds[];
    float *Es = lds;                                          // [TP][LD]
    float *xsh = lds + (size_t)TP * LD;                       // [D]
    const int64_t b = (int64_t)b0 + blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t Wz = (int64_t)D + (int64_t)T * (T + 1) / 2;
    float *__restrict__ zb = z + b * Wz;
    // zeros: the padding columns behind every vector and the padding rows behind the last one
    const int padc = LD - D;
    for (int i = tid; i < T * padc; i += kThreads) Es[(i / padc) * LD + D + i % padc] = 0.f;
    for (int i = T * LD + tid; i < TP * LD; i += kThreads) Es[i] = 0.f;
    fetch_sample<SRC, kFill, kParts, false>(dd, Es, emb, b, T, D, LD, vec4);
    for (int c = tid; c < D; c += kThreads) {
        const float v = x[b * D + c];
        xsh[c] = v;
        zb[c] = v;
    }
    __syncthreads();

    const int half = lane >> 5, l32 = lane & 31;
    const int nt = TP / 32;
    int tile = 0;
    for (int ti = 0; ti < nt; ++ti)
        for (int tj = 0; tj <= ti; ++tj, ++tile) {
            if ((tile & 3) != wave) continue;
            f32x16 acc;
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[v] = 0.f;
            const float *pa = Es + (ti * 32 + l32) * LD + half;
            const float *pb = Es + (tj * 32 + l32) * LD + half;
            for (int k = 0; k < D; k += 2)                    // column D of an odd D is a zero
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(pa[k], pb[k], acc, 0, 0, 0);
            const int col = tj * 32 + l32;                    // the lower-numbered vector of the pair
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int row = ti * 32 + 8 * (v >> 2) + 4 * half + (v & 3);
                if (row < T && col < row) zb[D + (int64_t)(row + 1) * row / 2 + col + 1] = acc[v];
            }
        }
    if (wave == 3) {
        for (int t = lane; t < T; t += 64) {
            float dot = 0.f;
            for (int c = 0; c < D; ++c) dot += Es[t * LD + c] * xsh[c];
            zb[D + (int64_t)(t + 1) * t / 2] = dot;
        }
    }
}

// The largest tile that still gives every compute unit two workgroups: a large tile splits and reads a
// value of X or W for more multiplies, but one workgroup alone does not fill a compute unit.  us with
// tiles of 128 x 128 / 128 x 64 / 64 x 64 (mlp_split), M K N: 16384 1024 512 (512 large tiles) 97 / 124 / -,
// 16384 512 256 (256) 37 / 33 / 34, 4096 1024 1024 (256) 58 / 57 / 62, 2048 1024 1024 (128) 50 / 36 / 33,
// 2048 512 256 (32) 29 / 19 / 11, 512 1024 1024 (32) 47 / 31 / 18.
template <int TI, int TJ, int CH, int ACT>
bool launch_tiles(const bls_ctx *ctx, const float *x, int64_t M, int K, const float *W, const float *bias, int N, float *y,
                  hipStream_t st)
{
    constexpr int BM = 64 * TI, BN = 64 * TJ;
    const uint64_t n_tiles = (uint64_t)((N + BN - 1) / BN), tiles = (uint64_t)((M + BM - 1) / BM) * n_tiles;
    if (tiles < 2 * (uint64_t)(ctx->compute_units > 0 ? ctx->compute_units : 256)) return false;
    const dim3 grid((unsigned)((tiles + 7u) / 8u * 8u));
    mlp_gemm<TI, TJ, CH, ACT><<<grid, kThreads, 0, st>>>(x, W, bias, y, M, N, K, (uint32_t)n_tiles, (uint32_t)tiles);
    return true;
}

template <int WN, int ACT>
void launch_short(const bls_ctx *ctx, const float *x, int64_t M, int K, const float *W, const float *bias, int N, float *y,
                  hipStream_t st)
{
    constexpr int kRows = 32 * 4 / WN;
    // eight workgroups for every compute unit, then up to four blocks of rows for each
    const uint64_t n_tiles = (uint64_t)((N + 32 * WN - 1) / (32 * WN)), blocks = (uint64_t)((M + kRows - 1) / kRows);
    const uint64_t enough = 8 * (uint64_t)(ctx->compute_units > 0 ? ctx->compute_units : 256);
    const int reps = (int)std::min<uint64_t>(std::max<uint64_t>(blocks * n_tiles / enough, 1), 4);
    const uint64_t tiles = (blocks + reps - 1) / reps * n_tiles;
    const dim3 grid((unsigned)((tiles + 7u) / 8u * 8u));
#define BLS_SHORT(steps) mlp_short<WN, steps, ACT><<<grid, kThreads, 0, st>>>(x, W, bias, y, M, N, K, (uint32_t)n_tiles, (uint32_t)tiles, reps)
    if (K <= 16) BLS_SHORT(1);
    else if (K <= 32) BLS_SHORT(2);
    else if (K <= 48) BLS_SHORT(3);
    else BLS_SHORT(4);
#undef BLS_SHORT
}

template <int ACT>
void launch_layer(const bls_ctx *ctx, const float *x, int64_t M, int K, const float *W, const float *bias, int N, float *y,
                  hipStream_t st)
{
    // 10^6 samples, us, fp32 instruction / tiles of 128 and 64 / this: K N 1 4 75 / 88 / 42, 13 16 83 / 97 / 39,
    // 64 4 166 / 162 / 98, 1 64 124 / 133 / 99, 64 64 204 / 195 / 185; from 65 outputs on the tiles are faster
    // (65536 samples, 13 512: 51 / 57) and so they are from 65 k on, where the parts of W do not fit the registers
    if (K <= 64 && N <= 64) {
        if (N <= 32) launch_short<1, ACT>(ctx, x, M, K, W, bias, N, y, st);
        else launch_short<2, ACT>(ctx, x, M, K, W, bias, N, y, st);
        return;
    }
    // a wavefront per row / tiles, us: N = 1, M = 16384 K = 256 9.2 / 10.9, K = 1024 16 / 22; M = 65536 K = 256 21 / 26;
    // M = 10^6 K = 96 246 / 196, K = 128 239 / 218, K = 256 373 / 375; N = 4, M = 65536 K = 256 46 / 26, K = 1024
    // 215 / 88.  By K and N alone: the sums' order, so that a sample's result does not depend on M.
    if (N == 1 && K >= kNarrowK) mlp_narrow<ACT><<<dim3((unsigned)((M + 3) / 4)), kThreads, 0, st>>>(x, W, bias, y, M, K);
    else if (launch_tiles<2, 2, 2, ACT>(ctx, x, M, K, W, bias, N, y, st)) return;
    else if (launch_tiles<2, 1, 4, ACT>(ctx, x, M, K, W, bias, N, y, st)) return;
    else {
        const uint64_t n_tiles = (uint64_t)((N + 63) / 64), tiles = (uint64_t)((M + 63) / 64) * n_tiles;
        const dim3 grid((unsigned)((tiles + 7u) / 8u * 8u));
        mlp_split<ACT><<<grid, kSplitThreads, 0, st>>>(x, W, bias, y, M, N, K, (uint32_t)n_tiles, (uint32_t)tiles);
    }
}

}  // namespace

int bls_launch_mlp_layer(bls_ctx *ctx, const float *x, int64_t M, int K, const float *W, const float *bias, int N,
                         int act, float *y, hipStream_t st)
{
    if (M == 0) return BLS_OK;
    const uint64_t tiles = (uint64_t)((M + 127) / 128) * (uint64_t)((N + 127) / 128);
    if (tiles > 0x7fffffffull - 8) return bls_fail(ctx, BLS_EINVAL, "bls_mlp_layer: too many tiles");
    // a grid has fewer than 2^32 threads (one of more is cut short without an error): the rows go in parts
    constexpr int64_t kGroups = ((int64_t)1 << 32) / kThreads - 8;
    const int64_t rows = N == 1 ? kGroups * (kThreads / 64) : kGroups / ((N + 63) / 64) * 64;
    for (int64_t m = 0; m < M; m += rows) {
        const int64_t part = std::min(rows, M - m);
        if (act == BLS_ACT_RELU) launch_layer<BLS_ACT_RELU>(ctx, x + m * K, part, K, W, bias, N, y + m * N, st);
        else if (act == BLS_ACT_SIGMOID) launch_layer<BLS_ACT_SIGMOID>(ctx, x + m * K, part, K, W, bias, N, y + m * N, st);
        else launch_layer<BLS_ACT_NONE>(ctx, x + m * K, part, K, W, bias, N, y + m * N, st);
        BLS_HIP(ctx, hipGetLastError());
    }
    return BLS_OK;
}

size_t bls_interact_lds_bytes(int T, int D)
{
    const int TP = (T + 31) / 32 * 32, LD = ((D + 1) & ~1) + 1;
    return ((size_t)TP * LD + (size_t)D) * sizeof(float);
}

int bls_launch_interact(bls_ctx *ctx, const float *x, const float *emb, int from_slot, float *z, uint32_t b0, uint32_t bn,
                        hipStream_t st)
{
    if (bn == 0) return BLS_OK;
    const int T = ctx->T, D = ctx->D;
    const int TP = (T + 31) / 32 * 32, LD = ((D + 1) & ~1) + 1;
    const int vec4 = D % 4 == 0 && ((uintptr_t)emb & 15u) == 0;   // every vector then starts 16-byte aligned
    const int tp16 = (T + 15) / 16 * 16;
    const size_t lds = bls_interact_lds_bytes(T, D), lds16 = ((size_t)tp16 * (D + 4) + (size_t)D) * sizeof(float);
    const bool tiles = D % 16 == 0 && lds16 <= 64 * 1024;     // else interact_gram: whole steps of k, and its LDS where that is less
#define BLS_INTERACT(src, fill, parts)                                                                                              \
    do {                                                                                                                           \
        if (tiles) interact_tiles<src, fill, parts><<<dim3(bn), kThreads, lds16, st>>>(ctx->desc, x, emb, z, T, D, tp16, b0, vec4);  \
        else interact_gram<src, fill, parts><<<dim3(bn), kThreads, lds, st>>>(ctx->desc, x, emb, z, T, D, TP, LD, b0, vec4);         \
    } while (0)
    // eight loads in flight: pieces of one partial, or fewer pieces and more owners' partials of each.  us, two
    // pieces of four partials / four of two: 8 owners, 2 vectors of 128 (16384 samples) 105 / 114, 26 (8192) 225 /
    // 234, 64 (2048) 160 / 155; 2 owners, 26 vectors (8192) 68 / 60
    const int pieces = (T * D / (vec4 ? 4 : 1) + kThreads - 1) / kThreads;   // of a thread
    if (!from_slot) BLS_INTERACT(FROM_OUT, 8, 1);
    else if (ctx->desc.F == 1) BLS_INTERACT(FROM_SLOT, 8, 1);
    else if (ctx->desc.F <= 2 || pieces > 4) BLS_INTERACT(FROM_PARTIALS, 4, 2);
    else BLS_INTERACT(FROM_PARTIALS, 2, 4);
#undef BLS_INTERACT
    BLS_HIP(ctx, hipGetLastError());
    return BLS_OK;
}
