// bls_step_tablewise: a whole synchronous iteration of a table-wise partition in one launch.
//
// Small batches spend their time in the hand-over between the seven to ten dependent kernels of
// the staged calls, not in the kernels.  With whole tables per rank nothing in the path depends on
// a pass over all lookups: a run (q, s) - the bags of one table in one rank's mini-batch - keeps
// its input order on the owner's side, so its place there follows from the run lengths alone, and
// those are differences of the offsets at the run edges.  Every workgroup reads the run edges for
// itself (a few hundred values out of L2), scans them in LDS, and then works on its own bags:
// segment start, the lookups' places in ridx and perm, the pooled vector, and that vector stored
// four times - pooled buffer, send region, receive region of the ring slot, output - each at its
// closed-form address.  Bit for bit what bls_plan, bls_embbag_pool, bls_pack, bls_alltoallv_local
// and bls_unpack leave behind.
#include <algorithm>
#include <type_traits>

#include "bls_internal.h"
#include "bls_rows.h"

namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;
constexpr int kMaxRuns = 2048;                 // runs (q, s) whose starts one workgroup scans in LDS
// Rows of a group in flight, in batches or in a ring: what is best with long bags among those that cost short ones little.  us, 26 tables, before
// the ring came / four / eight.  Batches, one table of 4.9 GB, 2048 bags of one, 512 of 1 to 100, 2048 of 1 to 40: 8-bit of 128 49.6 / 47.4 / 48.8, 63.8 / 64.3 /
// 60.9, 111 / 109 / 104, half precision of 64 24.3 / 22.4 / 24.0, 46.9 / 46.7 / 41.7, 58.9 / 56.8 / 54.4 (batches are its form for short bags, so
// four); 8192 bags of 1 to 15, 8-bit of 512 838 / 850 / 820.  Rings, half precision of 64, 2048 bags of one 23.4 / 23.4 / 24.5, 512 of 1 to 100 32.2 /
// 27.1 / 24.3; 8-bit of 128, 2048 bags of 1 to 23 81.0 / 74.7 / 100.
// Wavefronts per SIMD that a ring is held to (1: as it comes).  Held / as it comes, 4096 bags of up to 4, then 512 of 1 to 100: fp32 of 128 91 / 96, 43.2 / 42.6, of 64
// 43.0 / 45.6, 29.9 / 29.5; half precision of 128 67 / 72, 32.7 / 32.7; 8-bit of 128 86 / 88, 44.2 / 42.9, e4m3 86 / 88, 40.5 / 41.7.  Eight lanes of fp32 hold more
// registers than six wavefronts leave (two spilled): of 32, six / five, 2048 bags of one 18.8 / 18.3, 512 of 1 to 100 22.3 / 21.9.
template <int G, int DT, bool BATCH> constexpr int kRows = (BATCH ? DT == BLS_FP16 && G == 8 : is_rowq(DT)) ? 4 : 8;
template <int G, int DT> constexpr int kWavesHeld = DT == BLS_FP32 ? (G == 8 ? 5 : 6) : DT == BLS_FP16 ? (G < 16 ? 5 : 6) : G == 8 ? 5 : 1;

__device__ __forceinline__ void flag_error(const DevDesc &dd) { atomicOr(dd.err, 1); }

__device__ __forceinline__ int64_t wave_inclusive_scan(int64_t v, int lane)
{
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int64_t u = __shfl_up(v, o, 64);
        if (lane >= o) v += u;
    }
    return v;
}

// Position of run (q, s) in owner order (d, s, local table): the order of the owner-side blocks.
__device__ __forceinline__ int run_entry(const DevDesc &dd, int q, int s)
{
    const int d = dd.q_d[q];
    return dd.nsum[d] * dd.P + s * dd.n_loc[d] + (q - dd.nsum[d]);
}

// grid: x over (requester s, chunk of its mini-batch), y = q.  G lanes per bag, 16 bytes of a row per lane.
// BATCH: rows in batches through 64-bit addresses, where some shard is too large for 32-bit offsets and where bags are short (ring_rows).
// What bounds it is the chain from offsets to lookups to rows, and how many rows a group has in flight along a bag: the chain's
// start runs beside the count of the runs, and rows are read in a ring.  us a step, counted first and rows in
// batches of eight / this: 26 tables of 64, 512 bags of 1 to 100 41 / 37 (fp32), 32 / 28 (half precision), 52 / 38 (8-bit);
// 64 tables of 128, 2048 bags of 1 to 40 280 / 276, 211 / 204, 214 / 211; eight tables of 16, 128 bags of one 9.3 / 9.1.
template <int G, int DT, bool BATCH>
__global__ __launch_bounds__(kThreads, (BATCH ? 1 : kWavesHeld<G, DT>)) void step_tablewise(DevDesc dd, const int64_t *__restrict__ idx,
                                                           const int64_t *__restrict__ off, int64_t nnz,
                                                           int64_t *__restrict__ sendcounts, int64_t *__restrict__ sdispls,
                                                           int64_t *__restrict__ recvcounts, int64_t *__restrict__ rdispls,
                                                           int64_t *__restrict__ ridx, int64_t *__restrict__ segoff,
                                                           int64_t *__restrict__ perm, float *__restrict__ Y,
                                                           float *__restrict__ S, float *__restrict__ R,
                                                           float *__restrict__ out, uint32_t chunks)
{
    using A = Acc<DT, 16>;
    __shared__ int64_t rb[kMaxRuns + 1];       // run lengths in owner order, then their exclusive scan
    __shared__ int64_t part[kWaves];
    __shared__ int64_t red[kWaves];
    const int P = dd.P, nruns = dd.Q * P;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;

    // 1. this workgroup's bags: samples of requester s, table q.  Their rows need none of what the workgroups agree
    // on below, so the first of them are asked for here and come while the runs are counted.
    const int q = blockIdx.y;
    const int s = (int)(blockIdx.x / chunks);
    const uint32_t chunk = blockIdx.x - (uint32_t)s * chunks;
    const int t = dd.q_t[q], d = dd.q_d[q];
    const int64_t f = dd.first[s], n = dd.first[s + 1] - f;
    const int64_t g0 = (int64_t)t * dd.B + f;
    const int li = threadIdx.x & (G - 1);
    const int gbase = lane & ~(G - 1);
    const int64_t b_loc = (int64_t)chunk * (kThreads / G) + threadIdx.x / G;
    const bool live = b_loc < n;
    const uint32_t row_bytes = (uint32_t)payload_bytes(DT, dd.D), row_stride = (uint32_t)stride_bytes(DT, dd.D);
    const bool col_ok = (uint32_t)li * 16 < row_bytes;        // lanes past the row's end idle
    const int tail = (int)row_bytes - (col_ok ? li * 16 : 0);
    const int64_t rows = dd.q_rows[q];
    int64_t lo_run = off[g0], hi_run = off[g0 + n];
    int64_t beg = 0, len = 0, at_run = 0;
    if (live) {
        beg = off[g0 + b_loc];
        len = off[g0 + b_loc + 1] - beg;
    }
    if (lo_run < 0 || hi_run > nnz || hi_run < lo_run) lo_run = hi_run = 0;   // flagged below; the run counts as empty
    if (live) {
        const int64_t run_len = hi_run - lo_run;
        at_run = beg - lo_run;
        if (at_run < 0 || at_run > run_len || len < 0 || at_run + len > run_len) {   // a bag outside its run: treated as empty
            if (li == 0) flag_error(dd);
            at_run = at_run < 0 ? 0 : (at_run > run_len ? run_len : at_run);
            len = 0;
        }
    }
    constexpr int kU = kRows<G, DT, BATCH>, U = kU < G ? kU : G;     // rows in flight
    const __amdgpu_buffer_rsrc_t shard = shard_buffer(dd.q_base[q], BATCH ? 0u : (uint32_t)rows * row_stride);
    const char *__restrict__ base = (const char *)dd.q_base[q] + (col_ok ? (uint32_t)li * 16 : 0u);
    const uint32_t col = col_ok ? (uint32_t)li * 16 : 0u;
    auto ask = [&](int64_t c0) -> int64_t { return c0 + li < len ? idx[beg + c0 + li] : -1; };
    auto offset = [&](int64_t r) -> uint32_t { return (uint64_t)r < (uint64_t)rows ? (uint32_t)r * row_stride : kPastEnd; };
    int64_t here = ask(0), ahead = ask(G);                    // this lane's lookup of a block, and of the next
    typename A::Raw v[U];
    if constexpr (!BATCH) {
        const uint32_t mine = offset(here);
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = A::load_buffer(shard, (uint32_t)__shfl((int)mine, gbase + u, 64) + col, tail);
    }

    // 2. run lengths from the offsets at the run edges, scanned in owner order
    const int per = (nruns + kThreads - 1) / kThreads;        // runs of a thread in the scan
    for (int i = nruns + threadIdx.x; i < per * kThreads; i += kThreads) rb[i] = 0;
    bool bad_edges = false;
    for (int i = threadIdx.x; i < nruns; i += kThreads) {
        const int q = i / P, s = i - q * P;
        const int64_t g0 = (int64_t)dd.q_t[q] * dd.B;
        const int64_t lo = off[g0 + dd.first[s]], hi = off[g0 + dd.first[s + 1]];
        int64_t len = hi - lo;
        if (lo < 0 || hi > nnz || len < 0) { bad_edges = true; len = 0; }
        rb[run_entry(dd, q, s)] = len;
    }
    if (bad_edges) flag_error(dd);
    __syncthreads();
    {
        int64_t run = 0;
        for (int k = 0; k < per; ++k) run += rb[threadIdx.x * per + k];
        const int64_t inc = wave_inclusive_scan(run, lane);
        if (lane == 63) part[wv] = inc;
        __syncthreads();
        int64_t before = inc - run;
        for (int w = 0; w < wv; ++w) before += part[w];
        for (int k = 0; k < per; ++k) {
            const int64_t x = rb[threadIdx.x * per + k];
            rb[threadIdx.x * per + k] = before;
            before += x;
        }
        if (threadIdx.x == kThreads - 1) rb[per * kThreads] = before;
    }
    __syncthreads();
    const int64_t placed = rb[nruns];                         // the total
    auto edge = [&](int d, int s) -> int64_t {                // start of the owner-side block (d, s); (P, 0) is the end
        return rb[d >= P ? nruns : dd.nsum[d] * P + s * dd.n_loc[d]];
    };
    auto count = [&](int s, int d) -> int64_t {               // lookups rank s asks of rank d
        return (s + 1 < P ? edge(d, s + 1) : edge(d + 1, 0)) - edge(d, s);
    };

    // 3. the alltoallv counts and displacements, by the first workgroup
    if (blockIdx.x == 0 && blockIdx.y == 0) {
        for (int e = threadIdx.x; e < P * P; e += kThreads) {
            const int d = e / P, s = e - d * P;
            recvcounts[d * P + s] = count(s, d);
            sendcounts[s * P + d] = count(s, d);
            rdispls[d * P + s] = edge(d, s) - edge(d, 0);
            int64_t run = 0;
            for (int dd2 = 0; dd2 < d; ++dd2) run += count(s, dd2);
            sdispls[s * P + d] = run;
        }
        if (threadIdx.x == 0) segoff[dd.nseg] = placed;
    }

    // 4. owner-side place -> requester-side place of the run's lookups: start of bucket (s, d) in requester
    // order minus its start in owner order.  The requester-side start adds up every count of an
    // earlier requester and this requester's counts for earlier owners.
    const int64_t dst = rb[run_entry(dd, q, s)];
    int64_t to_send = 0;
    if (perm) {
        int64_t a = 0;
        for (int e = threadIdx.x; e < P * P; e += kThreads) {
            const int sp = e / P, dp = e - sp * P;
            if (sp < s || (sp == s && dp < d)) a += count(sp, dp);
        }
#pragma unroll
        for (int sh = 32; sh >= 1; sh >>= 1) a += __shfl_xor(a, sh, 64);
        if (lane == 0) red[wv] = a;
        __syncthreads();
        for (int w = 0; w < kWaves; ++w) to_send += red[w];
        to_send -= edge(d, s);
    }
    int64_t place = 0;
    if (live) {
        place = dst + at_run;
        const int64_t sg = (int64_t)dd.nsum[d] * dd.B + (int64_t)dd.n_loc[d] * f + (int64_t)(q - dd.nsum[d]) * n + b_loc;
        if (li == 0) segoff[sg] = place;
        if (place < 0 || place + len > nnz) {                 // run edges that decrease: the bag is empty, and its rows are dropped
            if (li == 0) flag_error(dd);
            len = 0;
            here = ahead = -1;
            if constexpr (!BATCH) {
#pragma unroll
                for (int u = 0; u < U; ++u) v[u] = A::none();
            }
        }
    }

    // 5. a block's lookups to their places on the owner's side, its rows added in order.  A ring of U rows in flight as in
    // the pooling kernels: lookups without a row read zeros, which change no sum.
    auto put = [&](int64_t c0, int64_t r) {
        if (c0 + li >= len) return;
        const bool ok = (uint64_t)r < (uint64_t)rows;
        if (!ok) flag_error(dd);                              // adds nothing to the bag
        ridx[place + c0 + li] = ok ? r : -1;
        if (perm) perm[beg + c0 + li] = place + c0 + li + to_send;
    };
    A acc;
    acc.zero();
    if constexpr (!BATCH) {
        put(0, here);
        uint32_t mine = offset(here);
        for (int64_t at = 0; __any(at < len); at += U) {
            const int64_t next = at + U;
            if ((next & (G - 1)) == 0) {
                here = ahead;
                ahead = ask(next + G);
                put(next, here);
                mine = offset(here);
            }
            uint32_t o[U];
#pragma unroll
            for (int u = 0; u < U; ++u) o[u] = (uint32_t)__shfl((int)mine, gbase + ((int)next & (G - 1)) + u, 64);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                acc.add(v[u]);
                v[u] = A::load_buffer(shard, o[u] + col, tail);
            }
        }
    } else {
        for (int64_t c0 = 0; __any(c0 < len); c0 += G) {
            put(c0, here);
            const int64_t mine = c0 + li < len && (uint64_t)here < (uint64_t)rows ? here : -1;
            here = ahead;
            ahead = ask(c0 + 2 * G);
            for (int j = 0; __any(c0 + j < len) && j < G; j += U) {
                int64_t r[U];
#pragma unroll
                for (int u = 0; u < U; ++u) r[u] = __shfl(mine, gbase + j + u, 64);
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    v[u] = A::none();
                    if (r[u] >= 0) v[u] = A::load(base + (uint64_t)r[u] * row_stride, tail);
                }
#pragma unroll
                for (int u = 0; u < U; ++u) acc.add(v[u]);
            }
        }
    }
    if (live && col_ok) {
        const int64_t b = f + b_loc;
        const int64_t sg = (int64_t)dd.nsum[d] * dd.B + (int64_t)dd.n_loc[d] * f + (int64_t)(q - dd.nsum[d]) * n + b_loc;
        const int64_t rho = (int64_t)dd.Q * f + (int64_t)q * n + b_loc;
        acc.store(Y + ((int64_t)q * dd.B + b) * dd.D + li * A::NV);
        acc.store(S + sg * dd.D + li * A::NV);
        acc.store(R + rho * dd.D + li * A::NV);
        acc.store(out + (b * dd.T + t) * dd.D + li * A::NV);
    }
}

template <int DT, bool BATCH>
bool dispatch(const bls_ctx *ctx, int lanes, dim3 grid, hipStream_t st, const int64_t *idx, const int64_t *off, int64_t nnz,
              int64_t *sc, int64_t *sd, int64_t *rc, int64_t *rd, int64_t *ridx, int64_t *segoff, int64_t *perm, float *Y,
              float *S, float *R, float *out, uint32_t chunks)
{
    switch (lanes) {
    case 1: step_tablewise<1, DT, BATCH><<<grid, kThreads, 0, st>>>(ctx->desc, idx, off, nnz, sc, sd, rc, rd, ridx, segoff, perm, Y, S, R, out, chunks); return true;
    case 2: step_tablewise<2, DT, BATCH><<<grid, kThreads, 0, st>>>(ctx->desc, idx, off, nnz, sc, sd, rc, rd, ridx, segoff, perm, Y, S, R, out, chunks); return true;
    case 4: step_tablewise<4, DT, BATCH><<<grid, kThreads, 0, st>>>(ctx->desc, idx, off, nnz, sc, sd, rc, rd, ridx, segoff, perm, Y, S, R, out, chunks); return true;
    case 8: step_tablewise<8, DT, BATCH><<<grid, kThreads, 0, st>>>(ctx->desc, idx, off, nnz, sc, sd, rc, rd, ridx, segoff, perm, Y, S, R, out, chunks); return true;
    case 16: step_tablewise<16, DT, BATCH><<<grid, kThreads, 0, st>>>(ctx->desc, idx, off, nnz, sc, sd, rc, rd, ridx, segoff, perm, Y, S, R, out, chunks); return true;
    case 32: step_tablewise<32, DT, BATCH><<<grid, kThreads, 0, st>>>(ctx->desc, idx, off, nnz, sc, sd, rc, rd, ridx, segoff, perm, Y, S, R, out, chunks); return true;
    case 64: step_tablewise<64, DT, BATCH><<<grid, kThreads, 0, st>>>(ctx->desc, idx, off, nnz, sc, sd, rc, rd, ridx, segoff, perm, Y, S, R, out, chunks); return true;
    }
    return false;
}

// Rows a bag from which the ring is the faster form.  A ring asks for at least twice U rows whatever a bag has, and a step of short bags is
// made of such requests: they are answered without an access, but take their turn.  Where the chip holds all workgroups at once nobody
// waits for that turn, and the longest bag's chain decides.  us, before the ring came / ring / batches, 26 tables, 2048 bags: fp32 of 128, of
// one row 40.9 / 42.0 / 34.2, 5 44.0 / 44.1 / 38.3, 12 64.8 / 67.2 / 59.0, 1024 of 16 37.8 / 37.0 / 36.2, of 24 44.5 / 43.8 / 44.5; of 32,
// one row 18.3 / 18.2 / 14.8, 1024 of 24 21.6 / 19.2 / 20.0; of 16, one row 13.2 / 12.3 / 11.7, 3 15.3 / 13.3 / 13.5; half precision of 128, one
// row 34.6 / 36.5 / 34.1, 8 39.2 / 41.7 / 40.8, 12 43.3 / 45.3 / 43.5, of 64, one row 24.6 / 25.1 / 22.2, 8 36.6 / 34.8 / 35.0, 12 42.9 / 38.9 / 41.9,
// 8192 of 8 124 / 122 / 119, of 12 146 / 138 / 140; 8-bit of 128, 8192 bags, 4 rows 199 / 209 / 193, 12 270 / 263 / 264, 24 349 / 339 / 332, of 512, 8
// rows 218 / 227 / 215, 16 260 / 266 / 258, 50 411 / 401 / 404 (never the ring).  By workgroups a compute unit: 6.6, fp32 of 128, 13 rows 29.7 / 27.2 / 28.0; 3.3,
// fp32 of 128, 4 rows 13.5 / 12.8 / 12.4; 2.6, half precision of 128, 12 rows 18.3 / 16.4 / 17.2; 1.6,
// half precision of 64, 6 rows 17.5 / 16.1 / 17.0; 0.5, fp32 of 64, 8 rows 9.3 / 8.9 / 9.3; 6.5, 8-bit of 128, 4 rows 57.3 / 56.2 / 55.6, 6 62.8 / 60.8 / 62.4, 24 112 / 103 / 105.
int64_t ring_rows(const bls_ctx *ctx, int lanes, int64_t workgroups)
{
    if (lanes < 4 || workgroups <= ctx->compute_units) return 0;
    const int64_t rows = lanes == 4 ? 3 : ctx->dtype == BLS_FP32 ? 16 : ctx->dtype == BLS_FP16 ? 13 : 1 << 20;
    return workgroups > 7 * (int64_t)ctx->compute_units ? rows : std::min<int64_t>(rows, 6);
}

}  // namespace

// BLS_EINVAL (and nothing launched) when the problem is not one this kernel takes: a row-wise
// partition, rows that 64 lanes of 16 bytes do not cover evenly, more than kMaxRuns runs.
int bls_launch_step_tablewise(bls_ctx *ctx, const int64_t *idx, const int64_t *off, int64_t nnz, int64_t *sendcounts,
                              int64_t *sdispls, int64_t *recvcounts, int64_t *rdispls, int64_t *ridx, int64_t *segoff,
                              int64_t *perm, float *Y, float *S, float *R, float *out, hipStream_t st)
{
    if (ctx->part_kind != BLS_TABLE_WISE) return bls_fail(ctx, BLS_EINVAL, "bls_step_tablewise: the partition is row-wise");
    const int64_t row_bytes = payload_bytes(ctx->dtype, ctx->D);
    if (row_bytes % 16 != 0 || row_bytes > 64 * 16 || (int64_t)ctx->Q * ctx->P > kMaxRuns)
        return bls_fail(ctx, BLS_EINVAL, "bls_step_tablewise: row length or number of runs outside what one launch takes; use the staged calls");
    int lanes = 1;
    while ((int64_t)lanes * 16 < row_bytes) lanes <<= 1;
    const uint32_t per_block = (uint32_t)(kThreads / lanes);
    const int64_t n_max = ctx->B / ctx->P + (ctx->B % ctx->P ? 1 : 0);
    const uint32_t chunks = (uint32_t)((n_max + per_block - 1) / per_block);
    const uint64_t gx = (uint64_t)chunks * ctx->P;
    if (gx > 0x7fffffffull) return bls_fail(ctx, BLS_EINVAL, "bls_step_tablewise: batch too large for one launch");
    const dim3 grid((unsigned)gx, (unsigned)ctx->Q);
    // in a ring unless a shard is too large for 32-bit offsets, or bags are short
    bool batch = ctx->tune_wide == 1 || (ctx->tune_wide != 0 && nnz < ring_rows(ctx, lanes, (int64_t)gx * ctx->Q) * ctx->nseg);
    for (int q = 0; q < ctx->Q; ++q) batch = batch || ctx->q_rows[q] >= (int64_t)kPastEnd / stride_bytes(ctx->dtype, ctx->D);
    auto go = [&](auto dt) -> bool {
        return batch ? dispatch<dt(), true>(ctx, lanes, grid, st, idx, off, nnz, sendcounts, sdispls, recvcounts, rdispls, ridx, segoff, perm, Y, S, R, out, chunks)
                    : dispatch<dt(), false>(ctx, lanes, grid, st, idx, off, nnz, sendcounts, sdispls, recvcounts, rdispls, ridx, segoff, perm, Y, S, R, out, chunks);
    };
    const bool ok = ctx->dtype == BLS_FP16    ? go(std::integral_constant<int, BLS_FP16>())
                  : ctx->dtype == BLS_U8_ROWQ ? go(std::integral_constant<int, BLS_U8_ROWQ>())
                  : ctx->dtype == BLS_F8_ROWQ ? go(std::integral_constant<int, BLS_F8_ROWQ>())
                                              : go(std::integral_constant<int, BLS_FP32>());
    if (!ok) return bls_fail(ctx, BLS_EINVAL, "bls_step_tablewise: unsupported row length");
    BLS_HIP(ctx, hipGetLastError());
    return BLS_OK;
}
