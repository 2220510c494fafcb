// bls_mlp_layer and bls_interact: the dense part of the model around the lookup (apply_mlp and
// interact_features of Listings 1 and 2), fp32 in and out, on the matrix cores.
//
// Operand layouts.  v_mfma_f32_32x32x2_f32: lane l supplies A[l % 32][l / 32] and B[l / 32][l % 32].
// v_mfma_f32_32x32x16_bf16: lane l supplies the eight k from 8 * (l / 32) of row (column) l % 32.  Both:
// accumulator register v of lane l is element (8 * (v / 4) + 4 * (l / 32) + v % 4, l % 32).
#include <stdint.h>

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

template <int ACT>
__device__ __forceinline__ float activate(float v)
{
    if constexpr (ACT == BLS_ACT_RELU) return v > 0.f ? v : 0.f;
    else if constexpr (ACT == BLS_ACT_SIGMOID) return 1.f / (1.f + expf(-v));
    else return v;
}

// ---- one layer: Y[M][N] = act(X[M][K] * W[N][K]^T + bias[N]) ---------------------------------
//
// fp32 operands on the bf16 matrix instructions.  A float is the sum of three bf16 numbers, exactly
// (24 significant bits, eight in each, the second and third being what rounding to nearest left), and
// of the nine products of two such sums the six largest are added up in fp32; what is left out is
// below 2^-24 of the product, less than the rounding of one fp32 multiply-add.
// v_mfma_f32_32x32x16_bf16 takes 32 cycles for 16 k, v_mfma_f32_32x32x2_f32 64 for 2: six of the
// former against eight of the latter are 192 cycles against 512.  The products of the first parts and
// the five small ones have an accumulator each: one rounding of the large sum per 16 k.  Against 64
// bits the error is a third of the fp32 instruction's (2-norm, K = 1024: 1.5e-7 and 4.1e-7; K = 2208:
// 2.2e-7 and 5.9e-7; K = 13: 3.9e-8 and 6.7e-8); with one accumulator for all six it is larger
// (K = 1024: 4.7e-7).
//
// A result that is not finite says nothing (an infinity has no three parts, and a float that rounds
// up to the bf16 infinity neither): it is taken again on the fp32 matrix instructions.  A finite one
// had finite operands: no product of an infinity or a NaN is finite.
//
// A workgroup of four wavefronts, two by two, owns a tile of 64 TI x 64 TJ; each wavefront multiplies
// 32 TI x 32 TJ.  Every element is summed over k in the same order whatever the tile, so that a
// sample's result does not depend on how many others are in the call.
// Tiles are staged already split, in planes of eight k: what a lane needs of a row is one 16-byte
// read, rows consecutive; two buffers, and the loads of two further steps in flight while one is
// multiplied.  Whole steps are loaded without a branch and the splitting is spread behind the multiplies
// (a branch per chunk made the compiler wait for the loads before the first multiply: 394 us for
// 16384 x 2208 -> 1024 instead of 375, 28 for 512 x 1024 -> 1024 instead of 21).  Workgroups are numbered so that those that share rows of X follow each other on one XCD
// (one L2), N-tile fastest.
//
// M = 16384, us, fp32 instructions / this: 2208 -> 1024 593 / 375 (198 TFLOP/s), 1024 -> 1024 284 / 184,
// 1024 -> 512 152 / 95, 512 -> 256 55 / 32, 256 -> 128 32 / 13.  M = 2048: 415 -> 1024 54 / 19,
// 1024 -> 1024 94 / 33, 512 -> 256 52 / 12.  The first of these is 1.19 PFLOP/s of bf16 products, 48 % of
// the matrix pipe's peak; a step's 12 reads and 6 writes of 16 bytes a lane keep the LDS busy for about as
// many cycles as its 24 multiplies take.
__device__ __forceinline__ bool finite(float v) { return __builtin_fabsf(v) <= 3.402823466e38f; }

struct Chunk { float v[8]; };                                 // eight consecutive k of one row

// Eight floats from k of a row of K (zeros from K on); rows need no alignment beyond the float's.
// WHOLE: all eight are there.
template <bool WHOLE>
__device__ __forceinline__ Chunk load_chunk(const float *__restrict__ row, int k, int K)
{
    Chunk c;
    f32x4 lo = 0.f, hi = 0.f;
    if (WHOLE || k + 8 <= K) {
        lo = *reinterpret_cast<const f32x4_a4 *>(row + k);
        hi = *reinterpret_cast<const f32x4_a4 *>(row + k + 4);
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (k + j < K) lo[j] = row[k + j];
            if (k + 4 + j < K) hi[j] = row[k + 4 + j];
        }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) { c.v[j] = lo[j]; c.v[4 + j] = hi[j]; }
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

template <int TI, int TJ, int CH, int ACT>
__global__ __launch_bounds__(kThreads, TI * TJ > 1 ? 2 : 3) void mlp_gemm(const float *__restrict__ X, const float *__restrict__ W,
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
    auto put = [&](Chunk c, u32x4 *at, int plane) {           // the three parts lie CH planes apart
#pragma unroll
        for (int p = 0; p < 3; ++p) {
            u32x4 w;
#pragma unroll
            for (int j = 0; j < 4; ++j) w[j] = take_bf16(c.v[2 * j], c.v[2 * j + 1]);
            at[p * CH * plane] = w;
        }
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
        // the reads first, then the splitting spread evenly behind the multiplies
        constexpr int kMfma = 3 * TI * TJ * CH, kValu = (44 * (NA + NB) + kMfma - 1) / kMfma, kWrites = 3 * (NA + NB);
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

#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < TJ; ++j) {
            f32x16 r = acc[i][j] + low[i][j];
            bool redo = false;
#pragma unroll
            for (int v = 0; v < 16; ++v) redo = redo || !finite(r[v]);
            const int col = n0 + wn + j * 32 + l32;
            if (__any(redo)) {                                 // the results that are not finite once more, in fp32
                const int64_t arow = m0 + wm + i * 32 + l32;
                f32x16 s = 0.f;
                for (int k = 0; k < K; k += 2) {
                    const int kk = k + half;
                    const float a = arow < M && kk < K ? X[arow * K + kk] : 0.f;
                    const float b = col < N && kk < K ? W[(int64_t)col * K + kk] : 0.f;
                    s = __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, s, 0, 0, 0);
                }
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    if (!finite(r[v])) r[v] = s[v];
            }
            if (col >= N) continue;
            const float bv = bias ? bias[col] : 0.f;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int64_t row = m0 + wm + i * 32 + 8 * (v >> 2) + 4 * half + (v & 3);
                if (row < M) Y[row * N + col] = activate<ACT>(r[v] + bv);
            }
        }
}

// One to four outputs per sample: a wavefront per row, the row's products summed lane by lane (k, k + 64,
// ...) and then across the lanes.  A matrix tile would spend 128 columns on them.
constexpr int kNarrow = 4;
constexpr int64_t kNarrowRows = (int64_t)1 << 30;              // a grid of 2^28 workgroups
template <int ACT>
__global__ __launch_bounds__(kThreads) void mlp_narrow(const float *__restrict__ X, const float *__restrict__ W,
                                                       const float *__restrict__ bias, float *__restrict__ Y,
                                                       int64_t M, int N, int K)
{
    const int lane = threadIdx.x & 63;
    const int64_t row = (int64_t)blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);
    if (row >= M) return;
    float sum[kNarrow] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
    for (int k = lane; k < K; k += 64) {
        const float x = X[row * K + k];
#pragma unroll
        for (int n = 0; n < kNarrow; ++n)
            if (n < N) sum[n] = fmaf(x, W[(int64_t)n * K + k], sum[n]);
    }
#pragma unroll
    for (int n = 0; n < kNarrow; ++n) {
        if (n >= N) break;
#pragma unroll
        for (int sh = 32; sh >= 1; sh >>= 1) sum[n] += __shfl_xor(sum[n], sh, 64);
        if (lane == n) Y[row * N + n] = activate<ACT>(sum[n] + (bias ? bias[n] : 0.f));
    }
}
// ---- dot interaction ---------------------------------------------------------------------------
//
// One workgroup per sample.  The sample's T pooled vectors are copied to LDS (rows padded to a
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
// come, a slot's took 290 us at that size, now 206.
enum Source { FROM_OUT, FROM_SLOT, FROM_PARTIALS };

// The sample's vectors in pieces of V (one float, or four), thread by thread, to rows of LD floats at Es.
// The d-th partial of vector t starts at vec0 + t_q[t] * vec_step + d * part_step (FROM_OUT: t for t_q[t]).
template <Source SRC, typename V>
__device__ __forceinline__ void fill_vectors(float *Es, uint32_t T, uint32_t D, uint32_t LD, int F, const float *vec0,
                                             const int32_t *__restrict__ t_q, int64_t vec_step, int64_t part_step)
{
    constexpr uint32_t W = sizeof(V) / sizeof(float);
    constexpr int kFill = 8;
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
            for (int d = 0; d < F; ++d) {
                V part[kFill];
#pragma unroll
                for (int u = 0; u < kFill; ++u) {
                    part[u] = 0.f;
                    if (live[u]) part[u] = *reinterpret_cast<const V *>(src[u] + d * part_step);
                }
#pragma unroll
                for (int u = 0; u < kFill; ++u) v[u] += part[u];
            }
        }
#pragma unroll
        for (int u = 0; u < kFill; ++u)
            if (live[u]) {
                if constexpr (W == 1) Es[at[u]] = v[u];
                else {
#pragma unroll
                    for (uint32_t j = 0; j < W; ++j) Es[at[u] + j] = v[u][j];
                }
            }
    }
}

template <Source SRC>
__global__ __launch_bounds__(kThreads) void interact_gram(DevDesc dd, const float *__restrict__ x, const float *__restrict__ emb,
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
    int64_t slot_base = 0, slot_step = 0;                        // vector (q, b) of the slot: slot_base + q * slot_step
    if constexpr (SRC != FROM_OUT) {
        int s; uint32_t b_loc, n;
        bls_split_sample(dd, (uint32_t)b, s, b_loc, n);
        slot_base = (int64_t)dd.Q * dd.first[s] + b_loc;
        slot_step = n;
    }
    const float *vec0 = emb + (SRC == FROM_OUT ? b * T : slot_base) * D;
    const int64_t vec_step = SRC == FROM_OUT ? D : slot_step * D, part_step = dd.T * slot_step * D;

    // zeros: the padding columns behind every vector and the padding rows behind the last one
    const int padc = LD - D;
    for (int i = tid; i < T * padc; i += kThreads) Es[(i / padc) * LD + D + i % padc] = 0.f;
    for (int i = T * LD + tid; i < TP * LD; i += kThreads) Es[i] = 0.f;
    if (vec4) fill_vectors<SRC, f32x4>(Es, T, D, LD, dd.F, vec0, dd.t_q, vec_step, part_step);
    else fill_vectors<SRC, float>(Es, T, D, LD, dd.F, vec0, dd.t_q, vec_step, part_step);
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
// tiles of 128 x 128 / 128 x 64 / 64 x 64, M K N: 16384 1024 512 (512 large tiles) 98 / 106 / 116,
// 16384 512 256 (256) 39 / 33 / 37, 4096 1024 1024 (256) 64 / 55 / 64, 2048 1024 1024 (128) 64 / 42 / 35,
// 2048 512 256 (32) 33 / 20 / 14 (taken with one step of loads in flight).
template <int TI, int TJ, int CH, int ACT>
bool launch_tiles(const bls_ctx *ctx, const float *x, int64_t M, int K, const float *W, const float *bias, int N, float *y,
                  bool any, hipStream_t st)
{
    constexpr int BM = 64 * TI, BN = 64 * TJ;
    const uint64_t n_tiles = (uint64_t)((N + BN - 1) / BN), tiles = (uint64_t)((M + BM - 1) / BM) * n_tiles;
    if (!any && tiles < 2 * (uint64_t)(ctx->compute_units > 0 ? ctx->compute_units : 256)) return false;
    const dim3 grid((unsigned)((tiles + 7u) / 8u * 8u));
    mlp_gemm<TI, TJ, CH, ACT><<<grid, kThreads, 0, st>>>(x, W, bias, y, M, N, K, (uint32_t)n_tiles, (uint32_t)tiles);
    return true;
}

template <int ACT>
void launch_layer(const bls_ctx *ctx, const float *x, int64_t M, int K, const float *W, const float *bias, int N, float *y,
                  hipStream_t st)
{
    // M = 16384, K = 256, N = 1: 27 us as a column of tiles of 128, 9.2 of 64, 8.4 a wavefront per row
    if (N <= kNarrow && M <= kNarrowRows) mlp_narrow<ACT><<<dim3((unsigned)((M + 3) / 4)), kThreads, 0, st>>>(x, W, bias, y, M, N, K);
    else if (launch_tiles<2, 2, 2, ACT>(ctx, x, M, K, W, bias, N, y, false, st)) return;
    else if (launch_tiles<2, 1, 4, ACT>(ctx, x, M, K, W, bias, N, y, false, st)) return;
    else (void)launch_tiles<1, 1, 4, ACT>(ctx, x, M, K, W, bias, N, y, true, st);
}

}  // namespace

int bls_launch_mlp_layer(bls_ctx *ctx, const float *x, int64_t M, int K, const float *W, const float *bias, int N,
                         int act, float *y, hipStream_t st)
{
    if (M == 0) return BLS_OK;
    const uint64_t tiles = (uint64_t)((M + 127) / 128) * (uint64_t)((N + 127) / 128);
    if (tiles > 0x7fffffffull - 8) return bls_fail(ctx, BLS_EINVAL, "bls_mlp_layer: too many tiles");
    if (act == BLS_ACT_RELU) launch_layer<BLS_ACT_RELU>(ctx, x, M, K, W, bias, N, y, st);
    else if (act == BLS_ACT_SIGMOID) launch_layer<BLS_ACT_SIGMOID>(ctx, x, M, K, W, bias, N, y, st);
    else launch_layer<BLS_ACT_NONE>(ctx, x, M, K, W, bias, N, y, st);
    BLS_HIP(ctx, hipGetLastError());
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
    const size_t lds = bls_interact_lds_bytes(T, D);
    if (!from_slot) interact_gram<FROM_OUT><<<dim3(bn), kThreads, lds, st>>>(ctx->desc, x, emb, z, T, D, TP, LD, b0, vec4);
    else if (ctx->desc.F == 1) interact_gram<FROM_SLOT><<<dim3(bn), kThreads, lds, st>>>(ctx->desc, x, emb, z, T, D, TP, LD, b0, vec4);
    else interact_gram<FROM_PARTIALS><<<dim3(bn), kThreads, lds, st>>>(ctx->desc, x, emb, z, T, D, TP, LD, b0, vec4);
    BLS_HIP(ctx, hipGetLastError());
    return BLS_OK;
}
