// bls_embbag_pool: EmbeddingBag sum over HBM-resident table shards.
//
// A group of G lanes owns one segment (one bag's lookups at one owner); lane i of the
// group keeps the columns stored in bytes [i*VB, (i+1)*VB) of a row in registers, so a row
// is fetched with one load per lane and consecutive lanes read consecutive addresses.
// G*VB covers the row: a 512-byte row is read by a whole wavefront with 8 bytes per lane
// or by half a wavefront with 16.  The group first loads up to G of its row numbers with
// one coalesced load, then walks them with U independent row loads in flight per lane: as a ring
// (RING), or U at a time, all of them waited for before the first add.  The adds follow in
// segment order, which keeps the fp32 result identical to a sequential sum.
//
// Bags are short (tens of rows), so a group does not stop at one: it streams the rows of
// several consecutive segments - they are contiguous in ridx - and stores and clears its
// accumulator whenever the stream crosses a segment boundary.  That amortises the
// dependent loads at the start (segment offsets, then row numbers, then rows) and evens out
// the lengths of the streams that share a wavefront.
#include <algorithm>
#include <type_traits>

#include "bls_internal.h"
#include "bls_rows.h"

namespace {

constexpr int kThreads = 256;
constexpr uint32_t kBadRow = 0xffffffffu;
#ifndef BLS_POOL_U
#define BLS_POOL_U 8
#endif
constexpr int kRowsInFlight = BLS_POOL_U;   // U: independent row loads issued per lane before the first add
#ifndef BLS_POOL_UQ
#define BLS_POOL_UQ 4
#endif
// row-quantised rows are four times shorter, so a load instruction carries four times as many rows:
// fewer per lane keep as many rows in flight with fewer registers (more wavefronts per SIMD)
constexpr int kRowsInFlightQuantised = BLS_POOL_UQ;

__device__ __forceinline__ void flag_error(const DevDesc &dd) { atomicOr(dd.err, 1); }

// Where a pooling launch leaves its vectors: Y alone (slot: Y is a ring slot, vectors in receive order), or
// pooled order, send order and, unless R is NULL, receive order at once.
struct PoolDst {
    float *Y, *S, *R;
    int slot, stores;
};
// PoolDst::stores: Y alone; three without the streaming hint; three, Y with it; three, Y and S with it
enum { kOneStore = 0, kThreePlain = 1, kThreeHintedY = 2, kThreeHinted = 3 };

// 64-bit value of lane (gbase + k), k uniform.  A whole-wavefront group reads it into scalar
// registers; narrower groups use the lane permute network (two ds_bpermute, no vector ALU
// work beyond the address), which pipelines when several are issued back to back.
template <int G>
__device__ __forceinline__ uint32_t group_broadcast32(uint32_t v, int gbase4, int k)
{
    if constexpr (G == 64) return (uint32_t)__builtin_amdgcn_readlane((int)v, k);
    else return (uint32_t)__builtin_amdgcn_ds_bpermute(gbase4 + 4 * k, (int)v);
}

template <int G>
__device__ __forceinline__ uint64_t group_broadcast64(uint64_t v, int gbase4, int k)
{
    if constexpr (G == 64) {
        const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, k);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), k);
        return ((uint64_t)hi << 32) | lo;
    } else {
        const uint32_t lo = (uint32_t)__builtin_amdgcn_ds_bpermute(gbase4 + 4 * k, (int)(uint32_t)v);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_ds_bpermute(gbase4 + 4 * k, (int)(uint32_t)(v >> 32));
        return ((uint64_t)hi << 32) | lo;
    }
}

// One segment per group of G lanes (G = 1 and 2: rows of 16 and 32 bytes with few rows a segment, and where lanes of 16 bytes are asked for, pool_shape).
// grid: x over groups of samples, y = q (owner, local table).
template <int G, int DT, int VB, int U>
__global__ __launch_bounds__(kThreads) void pool_rows(DevDesc dd, const int64_t *__restrict__ ridx,
                                                      const float *__restrict__ rw,
                                                      const int64_t *__restrict__ segoff, int64_t nnz,
                                                      float *__restrict__ Y, int to_slot, int q0)
{
    using A = Acc<DT, VB>;
    const int q = q0 + blockIdx.y;
    const int li = threadIdx.x & (G - 1);
    const int gbase = (threadIdx.x & 63) & ~(G - 1);
    const uint32_t b = blockIdx.x * (kThreads / G) + threadIdx.x / G;
    const bool live = b < (uint32_t)dd.B;
    const uint32_t row_bytes = (uint32_t)payload_bytes(DT, dd.D), row_stride = (uint32_t)stride_bytes(DT, dd.D);
    const bool col_ok = (uint32_t)li * VB < row_bytes;       // lanes past the row's end idle
    const char *__restrict__ base = (const char *)dd.q_base[q] + (uint32_t)li * VB;
    const int tail = (int)row_bytes - li * VB;               // from this lane's bytes to the row's scale and bias
    const int64_t shard_rows = dd.q_rows[q];

    int64_t beg = 0, len = 0, out = 0;
    if (live) {
        int s; uint32_t b_loc, n;
        bls_split_sample(dd, b, s, b_loc, n);
        const int64_t sg = bls_sigma(dd, q, s, b_loc, n);
        out = to_slot ? bls_rho(dd, q, s, b_loc, n) : (int64_t)q * dd.B + b;
        beg = segoff[sg];
        const int64_t end = segoff[sg + 1];
        len = end - beg;
        if (beg < 0 || len < 0 || end > nnz) { if (li == 0) flag_error(dd); len = 0; }
    }

    A acc;
    acc.zero();
    for (int64_t c0 = 0; __any(c0 < len); c0 += G) {
        const int64_t left = len - c0;
        const int rem = left < 0 ? 0 : (left > G ? G : (int)left);
        uint32_t mine = kBadRow;
        float wmine = 0.f;
        if (li < rem) {
            const int64_t r = ridx[beg + c0 + li];
            if (r < 0 || r >= shard_rows) flag_error(dd);
            else mine = (uint32_t)r;
            if (rw) wmine = rw[beg + c0 + li];
        }
        for (int j = 0; __any(j < rem); j += U) {
            uint32_t r[U];
            float wt[U];
            typename A::Raw v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                r[u] = (uint32_t)__shfl((int)mine, gbase + ((j + u) & (G - 1)), 64);
                wt[u] = __shfl(wmine, gbase + ((j + u) & (G - 1)), 64);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                v[u] = A::none();
                if (j + u < rem && r[u] != kBadRow && col_ok) v[u] = A::load(base + (uint64_t)r[u] * row_stride, tail);
                else wt[u] = 0.f;
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {                   // adding +0 for skipped rows changes nothing
                if (rw) acc.add_weighted(v[u], wt[u]);
                else acc.add(v[u]);
            }
        }
    }
    if (live && col_ok) acc.store(Y + out * dd.D + li * A::NV);
}

// The popular rows of the table a workgroup is working on, copied to LDS (pool_stream_hot), and
// an open-addressing table from row number to the row's place there.
constexpr uint32_t kHotBit = 0x80000000u;      // a row position with this bit set is a place in LDS
constexpr int kHotHash = 1024;                 // slots of the row -> place table (a power of two)
constexpr uint32_t kHotEmpty = 0xffffffffu;
struct HotRows {
    const unsigned char *data;                 // LDS: the rows, row_stride bytes each
    const uint32_t *keys;                      // LDS: row number per slot, or kHotEmpty
    const unsigned short *vals;                // LDS: the row's place
    int n;                                     // rows held (0: none)
};
__device__ __forceinline__ uint32_t hot_hash(uint32_t row) { return (row * 2654435761u) >> 22; }   // 10 bits

// One lane group's work: G >= 4 lanes stream up to nb_max (< G) consecutive segments of (q, s)
// block number gx / chunks_per_s, chunk gx % chunks_per_s.  HOT: rows found in `hot` are read from
// LDS instead of global memory.  RING: see below.
template <int G, int DT, int VB, int U, bool WIDE, bool WGT, bool HOT, bool RING, int STORES>
__device__ __forceinline__ void stream_group(const DevDesc &dd, int q, uint32_t gx, const int64_t *__restrict__ ridx,
                                             const float *__restrict__ rw, const int64_t *__restrict__ segoff, int64_t nnz,
                                             float *__restrict__ Y, float *__restrict__ S, float *__restrict__ R, int to_slot,
                                             int nb_max, uint32_t chunks_per_s, const HotRows &hot)
{
    using A = Acc<DT, VB>;
    const int lane = threadIdx.x & 63;
    const int li = lane & (G - 1);
    const int gbase = lane & ~(G - 1);
    const uint32_t s = gx / chunks_per_s;
    const uint32_t chunk = gx - s * chunks_per_s;
    const uint32_t row_bytes = (uint32_t)payload_bytes(DT, dd.D), row_stride = (uint32_t)stride_bytes(DT, dd.D);
    const bool col_ok = (uint32_t)li * VB < row_bytes;       // lanes past the row's end idle:
    // idle lanes re-read the row's first bytes (in bounds, same cache line) and never store
    const char *__restrict__ base = (const char *)dd.q_base[q] + (col_ok ? (uint32_t)li * VB : 0u);
    const int tail = (int)row_bytes - (col_ok ? li * VB : 0);   // to the row's scale and bias
    const int64_t shard_rows = dd.q_rows[q];

    // this group's segments: samples [b0, b0 + nb) of mini-batch s
    int nb = 0;
    int64_t sg0 = 0, out0 = 0;                                // first segment, its vector in the output
    uint32_t y_at = 0, s_at = 0, r_at = 0;                    // three stores: the first vector in Y, S and R
    if (s < (uint32_t)dd.P) {
        const int64_t f = dd.first[s], n = dd.first[s + 1] - f;
        const int64_t bl0 = (int64_t)chunk * nb_max;
        if (bl0 < n) {
            nb = n - bl0 < nb_max ? (int)(n - bl0) : nb_max;
            const int d = dd.q_d[q];
            sg0 = (int64_t)dd.nsum[d] * dd.B + (int64_t)dd.n_loc[d] * f + (int64_t)(q - dd.nsum[d]) * n + bl0;
            out0 = to_slot ? (int64_t)dd.Q * f + (int64_t)q * n + bl0 : (int64_t)q * dd.B + f + bl0;
            y_at = (uint32_t)out0;
            s_at = (uint32_t)sg0;
            r_at = (uint32_t)((int64_t)dd.Q * f + (int64_t)q * n + bl0);
        }
    }
    // lane i of the group holds the start of segment i (i <= nb); all must be in order
    int64_t seg = 0;
    if (nb > 0 && li <= nb) seg = segoff[sg0 + li];
    const int64_t seg_next = __shfl_down(seg, 1, G);
    const int64_t beg = __shfl(seg, gbase, 64);
    const int64_t end = __shfl(seg, gbase + nb, 64);
    const bool bad = nb > 0 && ((li < nb && seg_next < seg) || beg < 0 || end > nnz || end - beg > 0x7fffffffLL);
    const unsigned long long gmask = G == 64 ? ~0ull : ((1ull << (G & 63)) - 1ull) << gbase;
    if (__ballot(bad) & gmask) { if (bad) flag_error(dd); nb = 0; }
    const int rel = (int)(seg - beg);                        // segment starts relative to the stream
    const int total = nb > 0 ? (int)(end - beg) : 0;

    int cur = 0;                                             // segment being summed
    int cur_end = nb > 0 ? (int)__shfl(rel, gbase + 1, 64) : -1;
    A acc;
    acc.zero();

    // Store finished segments (also empty ones) once `pos` rows of the stream are consumed.  The
    // test is one compare against a uniform value; the rest runs only when some group of the
    // wavefront is at a boundary.  Every lane takes part in the lane exchange, the updates are
    // per group.  cur_end is -1 when the group has no segment left, which no position equals.
    auto flush = [&](int pos) {
        if (!__any(cur_end == pos)) return;
        do {
            const int nxt = __shfl(rel, gbase + (cur + 2 < G ? cur + 2 : G - 1), 64);
            if (cur_end == pos) {
                if (col_ok) {
                    if constexpr (STORES != kOneStore) {
                        // R is read by the completion, S only where there is no R (by the exchange), Y by nobody on the path
                        acc.template store<STORES >= kThreeHintedY>(Y + (int64_t)(y_at + cur) * dd.D + li * A::NV);
                        acc.template store<STORES == kThreeHinted>(S + (int64_t)(s_at + cur) * dd.D + li * A::NV);
                        if (R) acc.store(R + (int64_t)(r_at + cur) * dd.D + li * A::NV);
                    } else {
                        acc.store(Y + (out0 + cur) * dd.D + li * A::NV);
                    }
                }
                acc.zero();
                ++cur;
                cur_end = cur < nb ? nxt : -1;
            }
        } while (__any(cur_end == pos));
    };
    flush(0);

    // RING: U rows in flight all the time.  A row is added as soon as it has come, whatever is still on its way behind it,
    // and the next row of the stream is asked for into its registers; row numbers are asked for two blocks ahead and
    // tested when their block is next.  Rows are read through the shard's descriptor, so that a lookup without a row
    // (the stream's end, a bad index) needs no branch: it reads zeros, and adding +0 changes no sum, which is never -0.
    // Without branches between the loads the compiler knows how many are younger than the one it waits for.  What the
    // loop below costs beside this one: all U rows are waited for, with nothing in flight while they are added, a
    // block's row numbers are waited for before its rows, and every row has its execution mask.
    if constexpr (RING) {
        static_assert(!WIDE && !HOT);
        const __amdgpu_buffer_rsrc_t shard = shard_buffer(dd.q_base[q], (uint32_t)shard_rows * row_stride);
        const uint32_t col = col_ok ? (uint32_t)li * VB : 0u;
        auto ask = [&](int c0) -> int64_t { return c0 + li < total ? ridx[beg + c0 + li] : -1; };
        auto ask_weight = [&](int c0) -> float {
            if constexpr (WGT) return c0 + li < total ? rw[beg + c0 + li] : 0.f;
            else return 0.f;
        };
        // this lane's row of block c0 as an offset into the shard; the weight of a lookup without a row is 0 (it may be no number)
        auto place = [&](int c0, int64_t r, float &w) -> uint32_t {
            const bool ok = (uint64_t)r < (uint64_t)shard_rows;
            if (!ok && c0 + li < total) flag_error(dd);
            if (!ok) w = 0.f;
            return ok ? (uint32_t)r * row_stride : kPastEnd;
        };
        int64_t raw = ask(0);
        float wraw = ask_weight(0);
        uint32_t mine = place(0, raw, wraw);
        float wmine = wraw;
        raw = ask(G);
        wraw = ask_weight(G);
        typename A::Raw v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = A::load_buffer(shard, group_broadcast32<G>(mine, gbase * 4, u) + col, tail);
        for (int at = 0; __any(at < total); at += U) {
            float wt[WGT ? U : 1];
            if constexpr (WGT) {
#pragma unroll
                for (int u = 0; u < U; ++u) wt[u] = __uint_as_float(group_broadcast32<G>(__float_as_uint(wmine), gbase * 4, (at & (G - 1)) + u));
            }
            const int next = at + U;
            if ((next & (G - 1)) == 0) {
                mine = place(next, raw, wraw);
                wmine = wraw;
                raw = ask(next + G);
                wraw = ask_weight(next + G);
            }
            uint32_t off[U];
#pragma unroll
            for (int u = 0; u < U; ++u) off[u] = group_broadcast32<G>(mine, gbase * 4, (next & (G - 1)) + u);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if constexpr (WGT) acc.add_weighted(v[u], wt[u]);
                else acc.add(v[u]);
                v[u] = A::load_buffer(shard, off[u] + col, tail);
                flush(at + u + 1);                           // positions past the stream's end match nothing
            }
        }
        return;
    }

    // this lane's row of block c0 as a position in the shard (all ones: none or out of range)
    using pos_t = typename std::conditional<WIDE, uint64_t, uint32_t>::type;
    constexpr pos_t kNone = (pos_t)~(pos_t)0;
    const uint32_t row_units = WIDE ? row_stride : row_stride / VB;
    auto fetch = [&](int c0) -> pos_t {
        pos_t m = kNone;
        if (c0 + li < total) {
            const int64_t r = ridx[beg + c0 + li];
            if (r < 0 || r >= shard_rows) flag_error(dd);
            else {
                m = (pos_t)((pos_t)r * row_units);
                if constexpr (HOT) {
                    if (hot.n > 0) {                          // the table is never full: the walk ends at an empty slot
                        for (uint32_t h = hot_hash((uint32_t)r);; h = (h + 1u) & (kHotHash - 1)) {
                            const uint32_t key = hot.keys[h];
                            if (key == (uint32_t)r) { m = (pos_t)(kHotBit | hot.vals[h]); break; }
                            if (key == kHotEmpty) break;
                        }
                    }
                }
            }
        }
        return m;
    };
    auto is_row = [&](pos_t p) -> bool {
        if constexpr (WIDE) return (uint32_t)(p >> 32) != 0xffffffffu;
        else return p != kNone;
    };
    auto fetch_weight = [&](int c0) -> float {
        if constexpr (WGT) return c0 + li < total ? rw[beg + c0 + li] : 0.f;
        else return 0.f;
    };
    pos_t mine = fetch(0);
    float wmine = fetch_weight(0);
    typename A::Raw v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = A::none();
    for (int c0 = 0; __any(c0 < total); c0 += G) {
        const pos_t ahead = fetch(c0 + G);                   // next block of row numbers: waited for inside, by the test
        const float wahead = fetch_weight(c0 + G);
        const int left = total - c0;
        const int rem = left < 0 ? 0 : (left > G ? G : left);
        for (int j = 0; __any(j < rem); j += U) {
            pos_t off[U];
            float wt[WGT ? U : 1];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if constexpr (WIDE) off[u] = group_broadcast64<G>(mine, gbase * 4, j + u);
                else off[u] = group_broadcast32<G>(mine, gbase * 4, j + u);
                if constexpr (WGT) wt[u] = __uint_as_float(group_broadcast32<G>(__float_as_uint(wmine), gbase * 4, j + u));
            }
            // lanes without a row keep stale registers and skip the add: nothing to clear
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if constexpr (HOT) {
                    if (is_row(off[u])) {
                        if ((uint32_t)off[u] & kHotBit) v[u] = A::load_lds(hot.data + ((uint32_t)off[u] & ~kHotBit) * row_stride + (col_ok ? li * VB : 0), tail);
                        else v[u] = A::load(base + (uint64_t)off[u] * VB, tail);
                    }
                } else {
                    if (is_row(off[u])) v[u] = A::load(base + (WIDE ? (uint64_t)off[u] : (uint64_t)off[u] * VB), tail);
                }
            }
            // every load of the batch has landed before the first add: said once, here, so that
            // no wait is placed between the conditional loads of the next batch (the counter holds
            // stores as well: those of segments that ended in the batch before are waited for too)
            __builtin_amdgcn_s_waitcnt(0x0f70);              // vmcnt(0)
            const int at = c0 + j;                           // stream position of the batch (uniform)
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (is_row(off[u])) {
                    if constexpr (WGT) acc.add_weighted(v[u], wt[u]);
                    else acc.add(v[u]);
                }
                flush(at + u + 1);                           // positions past the stream's end match nothing
            }
        }
        mine = ahead;
        wmine = wahead;
    }
}

// Three stores with 32-bit positions: held to the 80 registers of six wavefronts per SIMD.  Four floats a lane fit them.  Eight
// (half-precision rows, 84) spill three, reloaded behind a wait for every block of G rows: a staged iteration, us, with the
// bound / without, table-wise 26 vectors of 64, 27 MB, bags of 40 to 100 224 / 194, 32 of 128, 268 MB, bags of 1 to 64
// 809 / 773, 26 of 128, 55 MB, bags of 20 to 60 255 / 246.  Blocks of 32 rows reload a quarter as often as those of 8, and
// the sixth wavefront is worth more: 16 of 256 row-wise, 200 MB, bags of 1 193 / 204, of 20 to 60 312 / 336.
// Eight 8-bit codes a lane spill seven, sixteen fit either way.
constexpr bool six_wavefronts(int G, int dt, int vb)
{
    return lane_floats(dt, vb) == 4 || (lane_floats(dt, vb) == 8 && dt == BLS_FP16 && G == 32);
}

// grid: x over groups (s-major, then chunks of nb_max samples), y = q.
// RING: rows one by one through the shard's descriptor, for shards below 4 GB (ring_pays says where).
// WIDE: row positions as 64-bit byte offsets; otherwise 32-bit, in units of VB bytes (shards
// below 2^32 * VB bytes), which halves the lane exchanges and the registers they occupy.
// WGT: per-sample weights rw[] (in ridx order) multiply every row before it is added.
// STORES not kOneStore: every vector goes to Y (pooled order), S (send order) and R (a ring slot) from the registers it was summed in,
// in place of pack and exchange, which read it again: five passes over the vectors up to the slot become three.  Vector
// numbers of 32 bits and, where six_wavefronts, the launch bound keep the six wavefronts per SIMD of the plain kernel.
// Y and S carry the streaming hint unless stores_that_pay says otherwise, the slot does not (the completion reads it).  A staged iteration, us, the separate
// kernels / plain stores / this / the slot hinted as well: 16384 samples of 64 vectors of 128, Zipf 1568 / 1549 / 1495 /
// 1488, bags of 1 to 4 743 / 656 / 640 / 522; row-wise 8192 of 26 over eight owners 1079 / 955 / 944 / 950, bags of one
// 924 / 720 / 676 / 695; table-wise 168 MB of short bags 203 / - / 153 / 183; 2048 of 26 of 64 46.5 / 35.7 / 34.8 / 35.5.
// Hinting the slot gains only for table-wise ones of 500 MB and loses up to a fifth elsewhere.
template <int G, int DT, int VB, int U, bool WIDE, bool WGT, bool RING, int STORES>
__global__ __launch_bounds__(kThreads, STORES != kOneStore && !WIDE && !RING && six_wavefronts(G, DT, VB) ? 6 : 1) void pool_stream(DevDesc dd, const int64_t *__restrict__ ridx,
                                                        const float *__restrict__ rw,
                                                        const int64_t *__restrict__ segoff, int64_t nnz,
                                                        float *__restrict__ Y, float *__restrict__ S, float *__restrict__ R,
                                                        int to_slot, int nb_max, uint32_t chunks_per_s, uint32_t wgx, int q0, int qn)
{
    // wgx = 0: grid y = q.  Otherwise a flat grid dealt out so that the workgroups an XCD receives
    // (every eighth one) all belong to the same few tables: q = 8 * (round of tables) + XCD.
    // Only the (owner, table) pairs q0 .. q0+qn-1 are worked on (all of them, or one owner's); all of them
    // are taken in the order dd.q_deal, which spreads the large shards evenly over the XCDs.
    uint32_t bx = blockIdx.x;
    int q = q0 + blockIdx.y;
    if (wgx) {
        const uint32_t xcd = blockIdx.x & 7u, r = blockIdx.x >> 3;
        const int pos = (int)((r / wgx) * 8u + xcd);
        bx = r % wgx;
        if (pos >= qn) return;
        q = qn == dd.Q ? dd.q_deal[pos] : q0 + pos;           // all shards: in the balanced order
    }
    const HotRows none{nullptr, nullptr, nullptr, 0};
    stream_group<G, DT, VB, U, WIDE, WGT, false, RING, STORES>(dd, q, bx * (kThreads / G) + threadIdx.x / G, ridx, rw, segoff, nnz, Y, S, R,
                                                      to_slot, nb_max, chunks_per_s, none);
}

// The same work by workgroups that stay: one workgroup of 1024 threads per compute unit, XCD x
// (workgroups x, x + 8, ...) takes the tables q0 + x, q0 + x + 8, ... one after the other, and its
// workgroups share a table's lane-group streams.  Before a table's first stream a workgroup copies
// the rows the caller named as popular (bls_set_hot_rows) to LDS and builds the row -> place table;
// lookups of those rows are then served from LDS, which takes them off the vector L1 path that
// bounds the kernel when a few rows receive most of the lookups.  Same adds in the same order.
constexpr int kHotThreads = 1024;
constexpr size_t kHotLdsBytes = 128 * 1024;     // LDS for the rows themselves (of 160 KB per compute unit)
template <int G, int DT, int VB, int U, bool WGT>
__global__ __launch_bounds__(kHotThreads) void pool_stream_hot(DevDesc dd, const int64_t *__restrict__ ridx,
                                                               const float *__restrict__ rw,
                                                               const int64_t *__restrict__ segoff, int64_t nnz,
                                                               float *__restrict__ Y, int to_slot, int nb_max,
                                                               uint32_t chunks_per_s, int q0, int qn, int cap_rows)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    const uint32_t row_stride = (uint32_t)stride_bytes(DT, dd.D);
    unsigned char *data = lds;
    uint32_t *keys = reinterpret_cast<uint32_t *>(lds + (size_t)cap_rows * row_stride);
    unsigned short *vals = reinterpret_cast<unsigned short *>(keys + kHotHash);
    const uint32_t xcd = blockIdx.x & 7u, j = blockIdx.x >> 3, per_xcd = gridDim.x >> 3;
    const uint32_t groups = chunks_per_s * (uint32_t)dd.P, per_wg = kHotThreads / G;
    const uint32_t blocks = (groups + per_wg - 1) / per_wg;
    for (int q = q0 + (int)xcd; q < q0 + qn; q += 8) {
        __syncthreads();                                      // the previous table's rows are no longer read
        const int n_hot = dd.hot_n[q] < cap_rows ? dd.hot_n[q] : cap_rows;
        if (n_hot > 0) {
            for (int i = threadIdx.x; i < kHotHash; i += kHotThreads) keys[i] = kHotEmpty;
            const uint32_t *rows = dd.hot_rows + dd.hot_off[q];
            const unsigned char *src = (const unsigned char *)dd.q_base[q];
            const uint32_t per_row = row_stride / 16;         // 16-byte pieces per row
            for (uint32_t i = threadIdx.x; i < (uint32_t)n_hot * per_row; i += kHotThreads) {
                const uint32_t r = i / per_row, piece = i - r * per_row;
                *reinterpret_cast<u32x4 *>(data + (size_t)r * row_stride + piece * 16) =
                    *reinterpret_cast<const u32x4 *>(src + (uint64_t)rows[r] * row_stride + piece * 16);
            }
            __syncthreads();                                  // the table is empty before anyone inserts
            for (int i = threadIdx.x; i < n_hot; i += kHotThreads) {
                const uint32_t row = rows[i];
                for (uint32_t h = hot_hash(row);; h = (h + 1u) & (kHotHash - 1)) {
                    const uint32_t seen = atomicCAS(&keys[h], kHotEmpty, row);
                    if (seen == kHotEmpty) { vals[h] = (unsigned short)i; break; }
                    if (seen == row) break;                   // named twice: the first copy serves
                }
            }
        }
        __syncthreads();
        const HotRows hot{data, keys, vals, n_hot};
        for (uint32_t blk = j; blk < blocks; blk += per_xcd)
            stream_group<G, DT, VB, U, false, WGT, true, false, kOneStore>(dd, q, blk * per_wg + threadIdx.x / G, ridx, rw, segoff, nnz, Y,
                                                                nullptr, nullptr, to_slot, nb_max, chunks_per_s, hot);
    }
}

// Rows that no lanes of 4, 8 or 16 bytes cover (half-precision rows of odd length, 8-bit ones of lengths that 4 does not divide, rows longer than 1 KB): one wavefront per
// segment, lanes stride the columns, scalar loads.  us, this / the streaming kernels, 8192 bags of one row of 26 tables and of 1 to 64: half
// precision of 20 85 / 35, 779 / 148, 8-bit of 20 88 / 38, 811 / 173; of one row fp32 of 10 88 / 36, of 5 83 / 31, 8-bit of 60 100 / 51.
template <int DT>
__global__ __launch_bounds__(kThreads) void pool_rows_generic(DevDesc dd, const int64_t *__restrict__ ridx,
                                                              const float *__restrict__ rw,
                                                              const int64_t *__restrict__ segoff, int64_t nnz,
                                                              float *__restrict__ Y, int to_slot, int q0)
{
    const int q = q0 + blockIdx.y;
    const int lane = threadIdx.x & 63;
    const uint32_t b = blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);
    if (b >= (uint32_t)dd.B) return;
    int s; uint32_t b_loc, n;
    bls_split_sample(dd, b, s, b_loc, n);
    const int64_t sg = bls_sigma(dd, q, s, b_loc, n);
    int64_t beg = segoff[sg], end = segoff[sg + 1];
    if (beg < 0 || end < beg || end > nnz) { if (lane == 0) flag_error(dd); end = beg = 0; }
    const int64_t shard_rows = dd.q_rows[q];
    const void *base = dd.q_base[q];
    float *y = Y + (to_slot ? bls_rho(dd, q, s, b_loc, n) : (int64_t)q * dd.B + b) * dd.D;
    for (int c = lane; c < dd.D; c += 64) {
        float acc = 0.f;
        for (int64_t j = beg; j < end; ++j) {
            const int64_t r = ridx[j];
            if (r < 0 || r >= shard_rows) { if (c == 0) flag_error(dd); continue; }
            float x;
            if constexpr (is_rowq(DT)) {
                const unsigned char *row = (const unsigned char *)base + r * stride_bytes(DT, dd.D);
                float scale, bias;                              // any D: no alignment to rely on
                __builtin_memcpy(&scale, row + dd.D, 4);
                __builtin_memcpy(&bias, row + dd.D + 4, 4);
                const float code = DT == BLS_F8_ROWQ ? __builtin_amdgcn_cvt_f32_fp8((int)row[c], 0) : (float)row[c];
                const float prod = code * scale;
                x = prod + bias;
            } else {
                const int64_t e = r * dd.D + c;
                x = DT == BLS_FP16 ? half_bits(((const unsigned short *)base)[e]) : ((const float *)base)[e];
            }
            if (rw) { const float term = rw[j] * x; acc += term; }
            else acc += x;
        }
        y[c] = acc;
    }
}

// Where rows are read in a ring (RING above): where the loop that waits for whole batches leaves time between them, which is
// wherever rows, not stored vectors, are most of the traffic.  A store counts among the accesses a later row waits behind,
// so that with a store every few rows a ring is no deeper than a batch and waits for its stores sooner.  us a pass with
// vectors of 128, batch / ring, by rows a segment and MB of vectors.  fp32: 32 rows, 134 MB 483 / 458, 32 of 64 floats 296 / 266, of
// 32 195 / 169, 8 rows, 250 MB 352 / 346, 2 of 64 floats 231 / 238, 1 row, 800 MB 399 / 408.  Half precision: 32 rows, 134 MB
// 355 / 321, 8, 800 MB 944 / 937, 4, 800 MB 541 / 545, staged 1024 / 1040.  8-bit: 32 rows, 134 MB 377 / 341, 250 MB
// 585 / 574, 8, 250 MB 310 / 312, 1 row, 800 MB 648 / 672.  What fits the memory-side cache gains earlier: fp32, 14 MB of 64 floats, 1 row 27.4 / 28.1,
// 60 MB, 5 rows 90 / 88, 8 rows 114 / 110, staged 67 MB, 1 row 83 / 89, 90 MB, 1.5 rows 131 / 134, 2 134.8 / 134.3, 5 159.5 / 158.9; ring over batches,
// geometric means of 20 to 90 MB, vectors of 16 to 512, 1, 2, 3, 4 and 6 rows: fp32 fused 0.998 0.994 0.985 0.976 0.968, staged 0.999 0.997 1.000 0.989 0.982,
// weighted 0.993 0.974 0.976 0.963 0.955; half precision 1.010 0.997 0.998 0.987 0.974, 1.009 1.006 1.010 0.995 0.983, 1.011 0.993 0.999 0.982 0.970; 8-bit
// 0.998 1.006 1.014 1.008 0.997, 1.002 1.011 1.015 1.005 0.998, 0.999 1.005 1.006 1.003 0.990.  Lanes of 8 and 4 bytes, 32 rows: half precision of
// 100 367 / 315, weighted 289 / 243, of 180 593 / 502, fp32 of 33 456 / 294, staged 246 / 167, of 62 366 / 320, 8-bit of 100 431 / 402.  Weights cost the batch a wavefront per SIMD (87
// registers; 80 here): fp32 1 row, 250 MB 202 / 196, 4 rows 220 / 209, 800 MB 611 / 587; half precision 4 rows 198 / 195.
static bool ring_pays(const bls_ctx *ctx, bool weighted, int64_t nnz, int qn)
{
    const int64_t rows = is_rowq(ctx->dtype) ? 12 : !weighted ? 8 : ctx->dtype == BLS_FP16 ? 4 : 2;
    if (nnz >= rows * ctx->nseg) return true;
    const int64_t cached = is_rowq(ctx->dtype) ? 6 : ctx->dtype == BLS_FP16 ? (weighted ? 2 : 4) : weighted ? 1 : 2;
    return nnz >= cached * ctx->nseg && (int64_t)qn * ctx->B * ctx->D * 4 <= (int64_t)96 << 20;
}
// Four workgroups per compute unit keep the memory busy in a ring, and with long segments of large shards more of them only share the caches: the
// kernels, which would run with five to seven, ask for LDS that they do not use.  us, as many as fit / four / three: fp32 rows of 128, 134 MB of vectors 463 /
// 458 / 456, of 64 275 / 265 / 267, of 32 173 / 169 / 173, with three stores 508 / 504 / 504, half precision 322 / 321 / 325, 8-bit 343 / 341 / 346, of 60, shards of 25 MB
// 360 / 327.  Segments of less than twelve rows are starts and stores as well and want all that fit, and so do a wavefront's lanes of 4 bytes and shards that an
// XCD's L2 of 4 MB holds: as many as fit / four / in batches, half precision of 32, weighted, 3.5 rows 86 / 94 / 90, fp32 of 16, weighted, 8 rows 52 / 54 / 53;
// fp32 of 33, 7 rows 959 / 1095 / 1029, 41 108 / 121 / 130, 8-bit of 100, weighted, 87 214 / 247 / 302; fp32 of 128, 38 rows, shards of 2 MB 78 / 83 / 77.
// 592 shapes, geometric means of the former over the latter: below twelve rows 0.99, shards of up to 2 MB 0.998, 4 to 16 1.002, 16 to 64 1.005 (up to 1.10).
// Beside other streams' kernels: the model's window of 64 tables of 128 with a lookup stream 7003 / 6765, of 26 1173 / 1190; per-rank streams level.
static constexpr size_t kRingLds = 36 * 1024;
static size_t ring_lds(const bls_ctx *ctx, int lanes, int lane_bytes, int64_t nnz, int64_t mean_shard)
{
    return nnz >= 12 * ctx->nseg && !(lane_bytes == 4 && lanes >= 32) && mean_shard > (int64_t)4 << 20 ? kRingLds : 0;
}

template <int G, int DT, int VB, int U>
void launch_rows(const bls_ctx *ctx, const int64_t *ridx, const float *rw, const int64_t *segoff, int64_t nnz, const PoolDst &to, int q0, int qn, hipStream_t st)
{
    constexpr int UU = U < G ? U : G;
    const uint32_t per_block = kThreads / G;
    if constexpr (G >= 4) {
        // segments per group: aim at a stream of two to three hundred rows (the lane groups of a wavefront finish
        // at different times, and the longer the streams the smaller the share of loads only one of them uses;
        // much longer streams lose again)
        const int64_t mean = nnz / std::max<int64_t>(1, ctx->nseg) + 1;
        int nb = 1;
        while (nb * 2 < G && nb * 2 <= 16 && nb * mean < 192) nb *= 2;
        // ... but a small batch takes shorter streams (down to eight rows) rather than fewer than two
        // workgroups per compute unit.  us a pass, down to sixty / this: 1024 bags of up to 4, 26 tables, half precision of 128 30.7 / 28.8; 1000 of
        // up to 6, 40 tables of 32 26.9 / 25.7; 3000 of up to 20, 12 tables of 64 8-bit 38.9 / 36.7, half precision 35.2 / 34.0; 300 of up to 2,
        // 64 tables of 256 39.9 / 39.0; 2048 bags of one, 26 tables of 64 27.8 / 27.4, of 128 36.6 / 35.7; in a ring of 64 34.3 / 34.1, down to four workgroups each 34.5
        const int64_t room = 2 * (int64_t)std::max(ctx->compute_units, 1);
        while (nb > 1 && nb * mean >= 8 && (int64_t)qn * ((ctx->B + nb - 1) / nb) < room * per_block) nb /= 2;
        if (ctx->tune_segs > 0) nb = ctx->tune_segs;
        nb = std::max(1, std::min(nb, G - 1));
        const int64_t n_max = ctx->B / ctx->P + (ctx->B % ctx->P ? 1 : 0);
        const uint32_t chunks = (uint32_t)((n_max + nb - 1) / nb);
        const int64_t groups = (int64_t)chunks * ctx->P;
        const uint32_t wgx = (uint32_t)((groups + per_block - 1) / per_block);
        // A shard's workgroups on one XCD leave the others idle where the shards are few: such launches are not dealt.  us, dealt /
        // not, vectors of 128, one store, fp32, 60 MB of bags of one: 1 shard 131 / 58, 2 88 / 60, 3 72 / 59, 5 65 / 60, 9 68 / 60, 10 67 / 61;
        // of 20 to 60 rows 1 shard 1028 / 228, 3 435 / 238, 5 312 / 248, 9 341 / 260, 10 322 / 259; 8 MB of them 1 130 / 43, 5 54 / 47,
        // 10 53 / 50; 8-bit, 60 MB 1 693 / 182, 9 262 / 199; row-wise, 4 owners 343 / 252.  Three stores and the calls they stand for (four launches, their pool
        // dealt), vectors of 64, bags of 1 to 4, calls / dealt / not: 1 table, 30 MB 99 / 112 / 46, 5, 100 MB 184 / 166 / 148, 8-bit, 8 MB 1
        // 54 / 82 / 34.  With most XCDs at work the deal's caches count for more with many rows a segment (three stores,
        // 7 tables, 8 MB, bags of 1 to 30 37 / 40), the even spread with few (30 MB 50 / 49).  Long rows of shards about as large as an XCD's L2 miss it eight times
        // when they are spread: fp32 of 128, one store, spread over dealt, 10 rows a segment with 20 MB and 150 MB of vectors, shards of 2.5 MB, 5 1.11 0.96, 9 1.10 1.08, 10 1.13
        // 1.18, 11 1.18 1.27, 4 rows 1.01 to 1.24, one 0.92 to 1.02, of 6 MB 1.00 to 1.22, of 1 MB 0.82 to 1.10; fp32 of 32 and 8-bit of 128 0.83.
        int64_t mean_shard = 0;
        const int64_t row_stride = stride_bytes(DT, ctx->D);
        for (int q = q0; q < q0 + qn; ++q) mean_shard += ctx->q_rows[q] * row_stride;
        mean_shard /= qn;
        const bool fits = to.stores == kOneStore && row_stride >= 512 && nnz >= 4 * ctx->nseg && mean_shard > (int64_t)3 << 19 && mean_shard <= (int64_t)8 << 20;
        const bool idle = 100 * qn < (fits ? 55 : 70) * 8 * ((qn + 7) / 8);
        const bool xcd = ctx->tune_xcd == 1 || (ctx->tune_xcd != 0 && !idle);
        const dim3 grid = xcd ? dim3((unsigned)((uint64_t)((qn + 7) / 8) * 8u * wgx)) : dim3(wgx, qn);
        const uint32_t deal = xcd ? wgx : 0u;
        // 32-bit row positions unless some shard is too large for them
        bool wide = ctx->tune_wide == 1;
        bool ring = ctx->tune_wide != 0 && ring_pays(ctx, rw != nullptr, nnz, qn);
        for (int q = q0; q < q0 + qn; ++q) {
            wide = wide || ctx->q_rows[q] * (row_stride / VB) >= 0xffffffffLL;
            ring = ring && ctx->q_rows[q] < (int64_t)kPastEnd / row_stride;
        }
        ring = ring && !wide;
        // popular rows named for some shard of this launch: the staying workgroups that keep them in LDS,
        // if every row position leaves the top bit free for the "in LDS" mark
        bool hot = VB == 16 && !wide && ctx->tune_hot != 0 && ctx->compute_units >= 8;
        bool any_hot = false;
        for (int q = q0; q < q0 + qn; ++q) {
            any_hot = any_hot || !ctx->q_hot[q].empty();
            hot = hot && ctx->q_rows[q] * (row_stride / VB) < (int64_t)kHotBit;
        }
        if constexpr (VB == 16) {
            if (hot && any_hot) {
                const int cap = (int)std::min<int64_t>(BLS_HOT_ROWS_MAX, (int64_t)kHotLdsBytes / row_stride);
                const size_t lds = (size_t)cap * row_stride + kHotHash * (sizeof(uint32_t) + sizeof(unsigned short));
                const dim3 hgrid((unsigned)(ctx->compute_units / 8 * 8));
                auto launch = [&](auto kernel) -> hipError_t {
                    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
                    if (e != hipSuccess) return e;
                    kernel<<<hgrid, kHotThreads, lds, st>>>(ctx->desc, ridx, rw, segoff, nnz, to.Y, to.slot, nb, chunks, q0, qn, cap);
                    return hipSuccess;
                };
                if (cap > 0 && (rw ? launch(pool_stream_hot<G, DT, VB, UU, true>) : launch(pool_stream_hot<G, DT, VB, UU, false>)) == hipSuccess)
                    return;
            }
        }
        auto launch = [&](auto kernel) {
            kernel<<<grid, kThreads, ring ? ring_lds(ctx, G, VB, nnz, mean_shard) : 0, st>>>(ctx->desc, ridx, rw, segoff, nnz, to.Y, to.S, to.R, to.slot, nb, chunks, deal, q0, qn);
        };
        auto pick = [&](auto weighted, auto stores) {
            if (ring) return launch(pool_stream<G, DT, VB, UU, false, weighted(), true, stores()>);
            if (wide) launch(pool_stream<G, DT, VB, UU, true, weighted(), false, stores()>);
            else launch(pool_stream<G, DT, VB, UU, false, weighted(), false, stores()>);
        };
        constexpr bool kThree = VB == 16 || G * VB >= 128;    // three stores: bls_pool_all_fits
        if (rw) {
            pick(std::true_type(), std::integral_constant<int, kOneStore>());
        } else if (to.stores == kOneStore) {
            pick(std::false_type(), std::integral_constant<int, kOneStore>());
        } else if (to.stores == kThreePlain) {
            if constexpr (kThree && (Acc<DT, VB>::NV == 16 || (Acc<DT, VB>::NV == 8 && G >= 16))) pick(std::false_type(), std::integral_constant<int, kThreePlain>());
        } else if (to.stores == kThreeHintedY) {
            if constexpr (kThree && (Acc<DT, VB>::NV == 8 || (Acc<DT, VB>::NV == 4 && G <= 16))) pick(std::false_type(), std::integral_constant<int, kThreeHintedY>());
        } else if constexpr (kThree && Acc<DT, VB>::NV <= 8) {
            pick(std::false_type(), std::integral_constant<int, kThreeHinted>());
        }
    } else {
        dim3 grid((unsigned)((ctx->B + per_block - 1) / per_block), qn);
        pool_rows<G, DT, VB, UU><<<grid, kThreads, 0, st>>>(ctx->desc, ridx, rw, segoff, nnz, to.Y, to.slot, q0);
    }
}

template <int DT, int VB, int U>
bool dispatch_lanes(const bls_ctx *ctx, int lanes, const int64_t *ridx, const float *rw, const int64_t *segoff, int64_t nnz,
                    const PoolDst &to, int q0, int qn, hipStream_t st)
{
    switch (lanes) {
    case 1: if constexpr (VB == 16) { launch_rows<1, DT, VB, U>(ctx, ridx, rw, segoff, nnz, to, q0, qn, st); return true; } break;
    case 2: if constexpr (VB == 16) { launch_rows<2, DT, VB, U>(ctx, ridx, rw, segoff, nnz, to, q0, qn, st); return true; } break;
    case 4: launch_rows<4, DT, VB, U>(ctx, ridx, rw, segoff, nnz, to, q0, qn, st); return true;
    case 8: launch_rows<8, DT, VB, U>(ctx, ridx, rw, segoff, nnz, to, q0, qn, st); return true;
    case 16: launch_rows<16, DT, VB, U>(ctx, ridx, rw, segoff, nnz, to, q0, qn, st); return true;
    case 32: launch_rows<32, DT, VB, U>(ctx, ridx, rw, segoff, nnz, to, q0, qn, st); return true;
    case 64: launch_rows<64, DT, VB, U>(ctx, ridx, rw, segoff, nnz, to, q0, qn, st); return true;
    }
    return false;
}

template <int DT>
bool dispatch_rows(const bls_ctx *ctx, int vb, int lanes, const int64_t *ridx, const float *rw,
                   const int64_t *segoff, int64_t nnz, const PoolDst &to, int q0, int qn, hipStream_t st)
{
    switch (vb) {
    case 16: return dispatch_lanes<DT, 16, (is_rowq(DT) ? kRowsInFlightQuantised : kRowsInFlight)>(ctx, lanes, ridx, rw, segoff, nnz, to, q0, qn, st);
    case 8: return dispatch_lanes<DT, 8, kRowsInFlight>(ctx, lanes, ridx, rw, segoff, nnz, to, q0, qn, st);
    case 4: return dispatch_lanes<DT, 4, kRowsInFlight>(ctx, lanes, ridx, rw, segoff, nnz, to, q0, qn, st);
    }
    return false;
}


}  // namespace

// Whether rows that one or two lanes of 16 bytes cover take four narrower ones.  Figures with 26 tables at pool_shape.  A row of a small shard comes out of the
// caches, and with many vectors the launch is full without streams: pool_rows is ahead then up to more rows a segment.  Four lanes over pool_rows, 12
// tables, fused, 7, 10 and 20 rows a segment, by MB of vectors.  Shards of 0.25 MB: fp32 of 8, 10 MB 1.05 1.02 0.89, 60 MB 1.19 1.22 1.12; half precision of 16, 10 MB
// 1.02 0.97 0.87, 60 MB 1.08 1.06 1.08, 150 MB 1.16 1.19 1.11; of 8, 10 MB 0.83 0.69 0.55, 60 MB 1.01 0.96 0.83, 150 MB 1.11 1.05; fp32 of 4, 60 MB 1.07 1.00; 8-bit of 16, 60 MB
// 0.89 0.76 0.70, 150 MB 1.07 1.02 0.91.  Of 25 MB: fp32 of 8, 60 MB 0.99 0.92 0.81, 150 MB 1.06 0.97, half precision of 16 0.94 0.89 0.79, 1.01 0.92 0.82, one lane below 0.92.
// 8-bit of 32, either shard, 1 row 0.84 to 0.97, 5 0.97 to 1.03, 7 to 10, 60 MB 0.97 to 1.03, 150 MB 1.01 to 1.04, 400 MB 1.04 to 1.11, 20, 60 MB 0.91 0.98, 150 MB 0.96 1.05.
static bool four_lanes_pay(const bls_ctx *ctx, int64_t nnz, int lanes)
{
    const bool rowq = is_rowq(ctx->dtype);
    const int64_t vectors = ctx->nseg * ctx->D * 4;
    const bool little = vectors <= (int64_t)24 << 20, many = vectors > (int64_t)96 << 20;
    int64_t shards = 0;
    for (int q = 0; q < ctx->Q; ++q) shards += ctx->q_rows[q] * stride_bytes(ctx->dtype, ctx->D);
    const bool small = shards <= ctx->Q * ((int64_t)4 << 20);
    if (rowq && lanes == 2) return !many || nnz < 4 * ctx->nseg || (!small && nnz >= 16 * ctx->nseg);
    if (!small) return nnz >= (lanes == 2 && many ? 8 : 6) * ctx->nseg;
    if (rowq) return nnz >= (many ? 16 : 6) * ctx->nseg;
    if (lanes == 2) return little && nnz >= 16 * ctx->nseg;
    return nnz >= (little ? 6 : many ? 16 : 12) * ctx->nseg;
}

// Bytes per lane and lanes per row of the kernels that read whole pieces of rows; false: pool_rows_generic.
static bool pool_shape(const bls_ctx *ctx, int64_t nnz, int *lane_bytes, int *row_lanes)
{
    const int64_t row_bytes = payload_bytes(ctx->dtype, ctx->D);
    // bytes per lane and row: 16 when the row length allows, unless bls_set_pool_tuning says otherwise
    int vb = ctx->tune_lane_bytes ? ctx->tune_lane_bytes : 16;
    while (vb > 4 && row_bytes % vb != 0) vb >>= 1;          // lanes must split the row evenly
    while (vb < 16 && row_bytes > 64 * (int64_t)vb) vb <<= 1; // and 64 of them must cover it
    if (row_bytes % vb != 0 || row_bytes > 64 * (int64_t)vb) return false;
    int lanes = 1;
    while ((int64_t)lanes * vb < row_bytes) lanes <<= 1;
    // Rows that one or two lanes cover whole: four lanes with a part each, which stream several segments, or with few rows a segment
    // pool_rows, whose groups are done after one.  us, pool_rows / four lanes: 8192 bags of 26 tables of 1 to 64 rows, half precision of 16 163 /
    // 125, of 8 166 / 96, fp32 of 8 155 / 111, 8-bit of 16 185 / 130, of 32 187 / 167; over four owners (8 rows) 108 / 99, 122 / 89, 98 / 91, 130 / 101,
    // 138 / 126; up to 6 rows (3) 34.6 / 37.8, 32 / 35, 31 / 36, 38.1 / 38.8, 48 / 47; one row 29 / 31, 25 / 28, 25 / 28, 32 / 32, 42 / 39.
    // A width that the caller chose is kept; of four lanes some idle then.
    const bool chosen = ctx->tune_lane_bytes != 0;
    if (lanes < 4 && (vb < 16 || (!chosen && four_lanes_pay(ctx, nnz, lanes)))) {
        while (!chosen && lanes < 4 && vb > 4) { vb >>= 1; lanes <<= 1; }
        lanes = 4;
    }
    *lane_bytes = vb;
    *row_lanes = lanes;
    return true;
}

static int launch_pool(bls_ctx *ctx, const int64_t *ridx, const float *rw, const int64_t *segoff, int64_t nnz, const PoolDst &to, int q0, int qn, hipStream_t st)
{
    if (qn == 0) return BLS_OK;                               // a rank that owns no table
    int vb = 0, lanes = 0;
    bool done = false;
    if (pool_shape(ctx, nnz, &vb, &lanes))
        done = ctx->dtype == BLS_U8_ROWQ ? dispatch_rows<BLS_U8_ROWQ>(ctx, vb, lanes, ridx, rw, segoff, nnz, to, q0, qn, st)
             : ctx->dtype == BLS_F8_ROWQ ? dispatch_rows<BLS_F8_ROWQ>(ctx, vb, lanes, ridx, rw, segoff, nnz, to, q0, qn, st)
             : ctx->dtype == BLS_FP16  ? dispatch_rows<BLS_FP16>(ctx, vb, lanes, ridx, rw, segoff, nnz, to, q0, qn, st)
                                       : dispatch_rows<BLS_FP32>(ctx, vb, lanes, ridx, rw, segoff, nnz, to, q0, qn, st);
    if (!done) {
        dim3 grid((unsigned)((ctx->B + kThreads / 64 - 1) / (kThreads / 64)), qn);
        if (ctx->dtype == BLS_U8_ROWQ) pool_rows_generic<BLS_U8_ROWQ><<<grid, kThreads, 0, st>>>(ctx->desc, ridx, rw, segoff, nnz, to.Y, to.slot, q0);
        else if (ctx->dtype == BLS_F8_ROWQ) pool_rows_generic<BLS_F8_ROWQ><<<grid, kThreads, 0, st>>>(ctx->desc, ridx, rw, segoff, nnz, to.Y, to.slot, q0);
        else if (ctx->dtype == BLS_FP16) pool_rows_generic<BLS_FP16><<<grid, kThreads, 0, st>>>(ctx->desc, ridx, rw, segoff, nnz, to.Y, to.slot, q0);
        else pool_rows_generic<BLS_FP32><<<grid, kThreads, 0, st>>>(ctx->desc, ridx, rw, segoff, nnz, to.Y, to.slot, q0);
    }
    BLS_HIP(ctx, hipGetLastError());
    return BLS_OK;
}

int bls_launch_pool(bls_ctx *ctx, const int64_t *ridx, const float *rw, const int64_t *segoff, int64_t nnz, float *Y, int to_slot, int q0, int qn, hipStream_t st)
{
    return launch_pool(ctx, ridx, rw, segoff, nnz, PoolDst{Y, nullptr, nullptr, to_slot, kOneStore}, q0, qn, st);
}

// What three stores from the pool's registers are made of where they take no longer than the pool, pack and exchange;
// kOneStore where they do.  A lane stores its NV floats in pieces of 16 bytes, so one store of a group covers all of the
// vector for NV = 4, every other piece for 8, every fourth for 16: the more pieces, the more the stores cost beside the
// permutes, which always store whole lines.  us a staged iteration, the calls / one launch hinted / plain:
// NV = 16 (8-bit rows): every piece that is hinted goes past the caches by itself, which shows as soon as the rows come out
// of a cache (24 vectors of 64, 30 MB, 3 rows a segment 68 / 92 / 63, 50 MB 98 / 146 / 93; 32 of 128, 200 MB, 1 row 304 /
// 498 / 310) and gains little where they do not (48 of 64, 32 MB, 2 rows 77 / 70 / 73).  Plain, up to 24 MB (48 of 48 65 / 84 /
// 59; 14 of 64, 30 MB, 4 rows 88 / 91 / 93; 32 of 128, 60 MB, 5 rows 130 / 127 / 134) or, with many rows a segment, 16 MB (48 of
// 128, 40 rows 82 / 77 / 79, 32 MB 140 / 144 / 144; 48 of 48, 24 MB 146 / 155 / 155).
// NV = 8 (half-precision rows): a shorter pool, so that with many rows a segment its fifth wavefront per SIMD counts for
// more than pack and exchange: 26 vectors of 64, 27 MB, 70 rows 201 / 214, 32 of 128, 200 MB, 40 rows 550 / 560, 20 rows 460 /
// 463, 5 rows 321 / 305; small ones gain with any number (10 MB, 70 rows 104 / 96).  Hinted, but for long vectors
// of hardly any rows: row-wise 21 of 512, 150 MB, 1/7 of a row 182 / 204 / 149, of 256 171 / 184 / 151, of 128 175 / 180 / 158,
// but of 64 174 / 163 / 174; table-wise 24 of 256, 1 row 214 / 201 / 195, 2 rows 199 / 176 / 216, of 128, 1 row 191 / 187 / 191;
// and of 192, where a quarter of the lanes idles, 178 / 152 / 181 (row-wise, 1/3 of a row).
// NV = 4: faster everywhere (100 rows, 17 MB, 149 / 140; 70 rows, 60 MB 435 / 415) for vectors of whole 64-byte pieces.
// Two of the others share one, which hinted stores write twice; the shorter the vector, the more of its pieces are shared
// and the more lanes of a store have nothing to do.  Bags of 1 to 4, the calls / Y and S hinted / Y alone / neither:
// table-wise 48 vectors of 20, 25 MB 86 / 86 / 79 / 85, 50 MB 141 / 164 / 142 / 140, 400 MB 1034 / 1231 / 1088 / 1034; of 28, 130
// MB 288 / 369 / 343 / 313; of 52, 50 MB 116 / 114 / 108 / 114, 130 MB 259 / 282 / 273 / 264; row-wise 12 of 20, 60 MB 119 / 134 /
// 99 / 117, 200 MB 352 / 429 / 363 / 335; of 28, 200 MB 301 / 386 / 342 / 314; of 36, 130 MB 228 / 224 / 169 / 209; of 52, 260 MB
// 358 / 369 / 351 / 362; half-precision, row-wise of 24, 50 MB 96 / 128 / 77 / 101, of 104, 130 MB 173 / 192 / 150 / 186.  Many rows
// a segment, the calls / Y alone: 48 of 28, 20 MB, 10 rows 111 / 112, 45 MB 202 / 213; row-wise 12 of 28, 120 MB, 7 rows 327 /
// 358, half-precision of 24 346 / 385.  From 64
// floats on (four a lane) both hinted: 48 of 68, 400 MB 858 / 794 / 753 / 753, row-wise 12 of 104 507 / 355 / 437 / 449.
// NV < 4: no hint (stores of 4 and 8 bytes), half again as fast as the calls (48 of 33, 130 MB 657 / 400).
static int stores_that_pay(const bls_ctx *ctx, int nv, int64_t nnz)
{
    const size_t MB = size_t(1) << 20;
    const int D = ctx->D;
    if (nv == 16) return ctx->slot_bytes <= (nnz <= 12 * ctx->nseg ? 24 : 16) * MB ? kThreePlain : kOneStore;
    if (nv == 8 && nnz > 32 * ctx->nseg && ctx->slot_bytes > 24 * MB) return kOneStore;
    const bool whole = (D & (D - 1)) == 0;                    // every lane of a group stores
    if (nv == 8 && (D >= 256 ? nnz <= ctx->nseg : D >= 128 && whole && 2 * nnz <= ctx->nseg)) return kThreePlain;
    if (nv < 4 || D % 16 == 0 || (nv == 4 && D >= 64)) return kThreeHinted;
    const bool tables = ctx->part_kind == BLS_TABLE_WISE;
    if (D < 32 && (nnz > 4 * ctx->nseg || ctx->slot_bytes > (tables ? 48 : 96) * MB)) return kOneStore;
    return tables && D < 64 && ctx->slot_bytes > 48 * MB ? kOneStore : kThreeHintedY;
}

static int pool_all_stores(const bls_ctx *ctx, int64_t nnz)
{
    int vb = 0, lanes = 0;
    if (!pool_shape(ctx, nnz, &vb, &lanes) || ctx->nvec >= (int64_t)1 << 31) return kOneStore;   // 32-bit vector numbers
    if (lanes < (vb == 16 ? 4 : 128 / vb)) return kOneStore;  // pool_rows, or lanes of 4 and 8 bytes without kernels of three stores
    for (const auto &h : ctx->q_hot)
        if (!h.empty()) return kOneStore;
    return stores_that_pay(ctx, lane_floats(ctx->dtype, vb), nnz);
}

bool bls_pool_all_fits(const bls_ctx *ctx, int64_t nnz) { return pool_all_stores(ctx, nnz) != kOneStore; }

int bls_launch_pool_all(bls_ctx *ctx, const int64_t *ridx, const int64_t *segoff, int64_t nnz, float *Y, float *S, float *R, hipStream_t st)
{
    return launch_pool(ctx, ridx, nullptr, segoff, nnz, PoolDst{Y, S, R, 0, pool_all_stores(ctx, nnz)}, 0, ctx->Q, st);
}
