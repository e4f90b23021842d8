// GROUP BY with SUM / COUNT / SUM of products, int64 exact modulo 2^64.
//
// Sort-based path (general).  After the keys are sorted, every group is a run.
// A first kernel counts the run heads of every block of rows; a second one takes
// the blocks again, starts at the sum of the counts before its block (so no
// block waits for another), and writes each run that begins in the block:
// key and aggregates, summed by a segmented scan.  A run that goes on past its
// block leaves a partial sum in its slot, and every later block it covers
// leaves its part in an edge record; a third, small kernel adds the edges.
// Integer addition modulo 2^64 is exact in any order, so the output is the
// same bytes on every run.
//
// Dense path.  When the caller bounds the key to a small domain
// [key_lo, key_lo + span), each workgroup accumulates into LDS counters
// indexed by key - key_lo and adds its totals to device accumulators; a final
// one-workgroup kernel emits the non-empty keys in ascending order.  Integer
// addition is order-free, so this path is bit-identical to the sorted one.
#include "tqp_internal.hpp"

namespace tqp {

constexpr int kGbNT = 512;
constexpr int kGbIPT = 4;
constexpr int kGbTile = kGbNT * kGbIPT;
constexpr int kGbNW = kGbNT / kWave;
constexpr int kGbMaxSteps = 8;          // tiles per block
constexpr int kMaxAgg = 4;
constexpr int kMaxVals = 8;

// The aggregates as the kernels take them: `nsum` sums (COUNT needs none: it
// is a count of rows either way) over the `nv` distinct value columns they
// name; sum g is column sa[g], times column sb[g] (or ic[g] minus it) when
// sb[g] >= 0.  src[agg] is the agg's sum, -1 for COUNT.
struct AggArgs {
    const void *val[kMaxVals];
    uint32_t vlen[kMaxVals];            // rows in [0, vlen) exist (at most 2^31: row ids are int32)
    int32_t vdt[kMaxVals];
    int32_t nv;
    int32_t op[kMaxAgg];
    int32_t sa[kMaxAgg];
    int32_t sb[kMaxAgg];
    int64_t ic[kMaxAgg];
    int32_t nsum;
    int32_t src[kMaxAgg];
    int32_t nagg;
    const int32_t *val_rows;
};
// Value columns loaded together, before any is used; aggregates over more
// distinct columns load each one when its sum is formed.
constexpr int kTogether = 2;

// The elements of R rows of a column, as loaded: 8-byte elements whole,
// narrower ones sign-extended to 32 bits by the load.  One branch on the type
// for all R, with nothing but loads in it, so that the loads of several
// columns stay in flight together; typed_value finishes the conversion.
template <int R>
__device__ __forceinline__ void load_typed(const void *p, int dt, const uint32_t (&row)[R],
                                           uint64_t (&out)[R]) {
    if (dt == TQP_INT64) {
#pragma unroll
        for (int r = 0; r < R; r++) out[r] = static_cast<const uint64_t *>(p)[row[r]];
    } else if (dt == TQP_INT32) {
#pragma unroll
        for (int r = 0; r < R; r++) out[r] = static_cast<const uint32_t *>(p)[row[r]];
    } else {
#pragma unroll
        for (int r = 0; r < R; r++) out[r] = uint32_t(int32_t(static_cast<const int8_t *>(p)[row[r]]));
    }
}
__device__ __forceinline__ int64_t typed_value(uint64_t raw, int dt) {
    return dt == TQP_INT64 ? int64_t(raw) : int64_t(int32_t(uint32_t(raw)));
}

// Value column c of R rows; rows outside it (or with a clear bit of valid)
// read row 0 here and count as 0 in take_value.  An empty column reads nothing.
template <int R>
__device__ __forceinline__ void load_value(const AggArgs &a, int c, const int32_t (&row)[R],
                                           uint32_t valid, uint64_t (&out)[R]) {
    uint32_t at[R];
    if (a.vlen[c] == 0) {
#pragma unroll
        for (int r = 0; r < R; r++) out[r] = 0;
        return;
    }
#pragma unroll
    for (int r = 0; r < R; r++)
        at[r] = ((valid >> r) & 1) && uint32_t(row[r]) < a.vlen[c] ? uint32_t(row[r]) : 0u;
    load_typed<R>(a.val[c], a.vdt[c], at, out);
}
template <int R>
__device__ __forceinline__ void take_value(const AggArgs &a, int c, const int32_t (&row)[R],
                                           uint32_t valid, const uint64_t (&raw)[R], int64_t (&v)[R]) {
    const int dt = a.vdt[c];
#pragma unroll
    for (int r = 0; r < R; r++)
        v[r] = ((valid >> r) & 1) && uint32_t(row[r]) < a.vlen[c] ? typed_value(raw[r], dt) : 0;
}

// The term of sum g for R rows (0 where valid is clear): its first column, or
// the product with its second (int64, wrapping, so exact modulo 2^64).
// TOG: the columns are already loaded in raw.
template <int R, bool TOG>
__device__ __forceinline__ void sum_terms(const AggArgs &a, int g, const int32_t (&row)[R], uint32_t valid,
                                          const uint64_t (&raw)[kTogether][R], int64_t (&t)[R]) {
    auto column = [&](int c, int64_t (&v)[R]) {
        if constexpr (TOG) {
#pragma unroll
            for (int k = 0; k < kTogether; k++)
                if (c == k) take_value<R>(a, k, row, valid, raw[k], v);
        } else {
            uint64_t w[R];
            load_value<R>(a, c, row, valid, w);
            take_value<R>(a, c, row, valid, w, v);
        }
    };
    column(a.sa[g], t);
    if (a.sb[g] >= 0) {
        int64_t y[R];
        column(a.sb[g], y);
        const bool diff = a.op[g] == TQP_AGG_SUM_DIFF_PRODUCT;
#pragma unroll
        for (int r = 0; r < R; r++) {
            const uint64_t f = diff ? uint64_t(a.ic[g]) - uint64_t(y[r]) : uint64_t(y[r]);
            t[r] = ((valid >> r) & 1) ? int64_t(uint64_t(t[r]) * f) : 0;
        }
    }
}

// Tiles per block for cnt rows, the same on the device in every kernel: the
// widest of 8, 4, 2, 1 that still gives sixteen blocks per compute unit.
__host__ __device__ inline int gb_steps(int64_t cnt) {
    int st = kGbMaxSteps;
    while (st > 1 && cnt < int64_t(kGbTile) * st * 16 * kComputeUnits) st >>= 1;
    return st;
}
// Blocks any count up to n can take (one tile each up to twice sixteen per
// CU, then at most that many until the blocks are at their longest).
static int64_t gb_max_blocks(int64_t n) {
    const int64_t few = int64_t(2) * 16 * kComputeUnits;
    const int64_t tiles = ceil_div(n > 0 ? n : 1, kGbTile);
    const int64_t longest = ceil_div(n > 0 ? n : 1, int64_t(kGbTile) * kGbMaxSteps);
    const int64_t most = longest > few ? longest : few;
    return tiles < most ? tiles : most;
}

// This thread's kGbIPT keys and the ones before and after them, and the bits
// of the rows that exist.
template <class K>
__device__ __forceinline__ void load_run_keys(const K *keys, int64_t row0, int64_t cnt, bool vec,
                                              K (&v)[kGbIPT], K &before, K &after) {
    constexpr int R = kGbIPT;
    if (vec && row0 + R <= cnt) {
        constexpr int kPer = 16 / sizeof(K);
        const int4 *q = reinterpret_cast<const int4 *>(keys + row0);
#pragma unroll
        for (int j = 0; j < R / kPer; j++) {
            const int4 x = q[j];
            const K *e = reinterpret_cast<const K *>(&x);
#pragma unroll
            for (int t = 0; t < kPer; t++) v[j * kPer + t] = e[t];
        }
    } else {
#pragma unroll
        for (int r = 0; r < R; r++) v[r] = row0 + r < cnt ? keys[row0 + r] : K(0);
    }
    before = row0 > 0 && row0 <= cnt ? keys[row0 - 1] : K(0);
    after = row0 + R < cnt ? keys[row0 + R] : K(0);
}
// Bit r of head: row r starts a run; of end: row r ends one.
template <class K>
__device__ __forceinline__ void run_bits(const K (&v)[kGbIPT], K before, K after, int64_t row0,
                                         int64_t cnt, uint32_t &head, uint32_t &end) {
    constexpr int R = kGbIPT;
    head = end = 0;
#pragma unroll
    for (int r = 0; r < R; r++) {
        const int64_t i = row0 + r;
        const K prv = r == 0 ? before : v[r - 1];
        const K nxt = r == R - 1 ? after : v[r + 1];
        head |= (i < cnt && (i == 0 || v[r] != prv) ? 1u : 0u) << r;
        end |= (i < cnt && (i == cnt - 1 || v[r] != nxt) ? 1u : 0u) << r;
    }
}

// Run heads of every block.
template <class K>
__global__ __launch_bounds__(kGbNT) void k_gb_heads(const K *__restrict__ keys, int64_t n,
                                                    const int64_t *d_n, int32_t *__restrict__ bcnt) {
    __shared__ int32_t s_cnt[kGbNW];
    const int64_t cnt = count_of(d_n, n);
    const int steps = gb_steps(cnt);
    const int64_t nblocks = ceil_div(cnt, int64_t(kGbTile) * steps);
    const bool vec = reinterpret_cast<uintptr_t>(keys) % 16 == 0;
    for (int64_t b = blockIdx.x; b < nblocks; b += gridDim.x) {
        int32_t heads = 0;
        for (int st = 0; st < steps; st++) {
            const int64_t row0 = (b * steps + st) * kGbTile + int64_t(threadIdx.x) * kGbIPT;
            K v[kGbIPT], before, after;
            uint32_t head, end;
            load_run_keys(keys, row0, cnt, vec, v, before, after);
            run_bits(v, before, after, row0, cnt, head, end);
            heads += __popc(head);
        }
        heads = wave_sum(heads);
        if (lane_id() == 0) s_cnt[wave_id()] = heads;
        __syncthreads();
        if (threadIdx.x == 0) {
            int32_t tot = 0;
#pragma unroll
            for (int w = 0; w < kGbNW; w++) tot += s_cnt[w];
            bcnt[b] = tot;
        }
        __syncthreads();
    }
}

// The part of a run that lies in a block it did not begin in: the run's slot
// (-1: the block begins with a run of its own) and the block's share of
// each aggregate.
struct GbEdges {
    int64_t *slot;                 // [blocks]
    int64_t *part;                 // [nagg][blocks]
    int64_t stride;
};
struct GbOut {
    int64_t *agg[kMaxAgg];
    int64_t cap;
};

// The runs of every block.  Per tile: each thread's sums since its last run
// head, a segmented scan of those over the workgroup (NSUM sums, the number of
// heads, and the last head's position, which gives COUNT), then each thread walks
// its rows from the sum carried into it.  The open run is carried from tile to
// tile of a block.
//
// What bounds it: keys, row ids and values (16 B per row for one 8-byte sum).
// The version before this carried running sums through a look-back, every tile
// waiting for the one before it, and wrote them per group for a later
// difference.  30M sorted int32 keys in 1.5M groups, SUM of an int64 column
// through row ids and COUNT: 265 + 11 us (scan, differences) -> 23 + 158 + 5 us
// (heads, runs, edges).  512 threads of 4 rows: with 256 of 8 the rows' terms
// spill with one sum already.  (Here two sums of columns loaded together spill 2 registers, of
// int64 keys 5; three 13 and 17; four 32 and 42, and 20 to 23 loaded one by one.)
template <class K, int NSUM, bool TOG>
__global__ __launch_bounds__(kGbNT, 4) void k_gb_runs(const K *__restrict__ keys, int64_t n,
                                                      const int64_t *d_n, AggArgs a,
                                                      K *__restrict__ out_key, GbOut o,
                                                      int64_t *d_ngroups,
                                                      const int32_t *__restrict__ bcnt, GbEdges e) {
    constexpr int R = kGbIPT;
    constexpr int NS = NSUM > 0 ? NSUM : 1;
    struct Wave {
        uint64_t sum[NS];
        int32_t heads, last;
    };
    __shared__ Wave s_wave[2][kGbNW];
    __shared__ int64_t s_base[kGbNW];
    const int64_t cnt = count_of(d_n, n);
    const int steps = gb_steps(cnt);
    const int64_t brows = int64_t(kGbTile) * steps;
    const int64_t nblocks = ceil_div(cnt, brows);
    const bool vec = reinterpret_cast<uintptr_t>(keys) % 16 == 0;
    const bool rvec = a.val_rows && reinterpret_cast<uintptr_t>(a.val_rows) % 16 == 0;
    const int w = wave_id(), lane = lane_id();
    if (cnt == 0 && blockIdx.x == 0 && threadIdx.x == 0) *d_ngroups = 0;
    int64_t base = 0, from = 0;
    for (int64_t b = blockIdx.x; b < nblocks; b += gridDim.x) {
        int64_t part = 0;
#pragma unroll 4
        for (int64_t i = from + threadIdx.x; i < b; i += kGbNT) part += bcnt[i];
        part = wave_sum(part);
        __syncthreads();                               // s_base and s_wave of the block before
        if (lane == 0) s_base[w] = part;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kGbNW; i++) base += s_base[i];
        from = b;
        const int64_t blk0 = b * brows;
        const int64_t blk1 = blk0 + brows < cnt ? blk0 + brows : cnt;
        int64_t hc = base;                             // heads before the tile
        int32_t open_at = -1;                          // the open run's head in the block (-1: before it)
        uint64_t open[NS];                             // and its sums so far
#pragma unroll
        for (int g = 0; g < NS; g++) open[g] = 0;
        for (int st = 0; st < steps; st++) {
            const int64_t tile0 = blk0 + int64_t(st) * kGbTile;
            if (tile0 >= blk1) break;
            const int64_t row0 = tile0 + int64_t(threadIdx.x) * R;
            K v[R], before, after;
            load_run_keys(keys, row0, cnt, vec, v, before, after);
            int32_t rows[R];
            if (rvec && row0 + R <= cnt) {
                const int4 *q = reinterpret_cast<const int4 *>(a.val_rows + row0);
#pragma unroll
                for (int j = 0; j < R / 4; j++) {
                    const int4 x = q[j];
                    rows[4 * j] = x.x; rows[4 * j + 1] = x.y; rows[4 * j + 2] = x.z; rows[4 * j + 3] = x.w;
                }
            } else {
#pragma unroll
                for (int r = 0; r < R; r++)
                    rows[r] = row0 + r < cnt ? (a.val_rows ? a.val_rows[row0 + r] : int32_t(row0 + r)) : 0;
            }
            const uint32_t valid = row0 >= cnt ? 0u : row0 + R <= cnt ? (1u << R) - 1u : (1u << int(cnt - row0)) - 1u;
            uint64_t raw[kTogether][R];
            if constexpr (TOG && NSUM > 0) {
#pragma unroll
                for (int c = 0; c < kTogether; c++)
                    if (c < a.nv) load_value<R>(a, c, rows, valid, raw[c]);
            }
            uint32_t head, end;
            run_bits(v, before, after, row0, cnt, head, end);
            int64_t term[NS][R];
            uint64_t sum[NS];                          // since the thread's last head
#pragma unroll
            for (int g = 0; g < NSUM; g++) {
                sum_terms<R, TOG>(a, g, rows, valid, raw, term[g]);
                sum[g] = 0;
#pragma unroll
                for (int r = 0; r < R; r++) sum[g] = (head >> r & 1 ? 0 : sum[g]) + uint64_t(term[g][r]);
            }
            const int32_t local0 = int32_t(row0 - blk0);
            int32_t last = head ? local0 + 31 - __builtin_clz(head) : -1;
            int32_t heads = __popc(head);
            const int32_t my_heads = heads;
            // segmented inclusive scan over the wave (a thread's flag is last >= 0)
#pragma unroll
            for (int d = 1; d < kWave; d <<= 1) {
                const int32_t uh = shfl_up(heads, d), ul = shfl_up(last, d);
#pragma unroll
                for (int g = 0; g < NSUM; g++) {
                    const uint64_t us = shfl_up(sum[g], d);
                    if (lane >= d && last < 0) sum[g] += us;
                }
                if (lane >= d) {
                    heads += uh;
                    last = last > ul ? last : ul;
                }
            }
            Wave *sw = s_wave[st & 1];
            if (lane == kWave - 1) {
#pragma unroll
                for (int g = 0; g < NSUM; g++) sw[w].sum[g] = sum[g];
                sw[w].heads = heads;
                sw[w].last = last;
            }
            __syncthreads();
            // what is carried into this wave, and out of the tile
            int32_t in_at = open_at, wheads = 0;
            uint64_t in[NS];
#pragma unroll
            for (int g = 0; g < NSUM; g++) in[g] = open[g];
            int32_t theads = 0;
#pragma unroll
            for (int i = 0; i < kGbNW; i++) {
                if (i == w) {
                    in_at = open_at;
                    wheads = theads;
#pragma unroll
                    for (int g = 0; g < NSUM; g++) in[g] = open[g];
                }
                const int32_t l = sw[i].last;
#pragma unroll
                for (int g = 0; g < NSUM; g++) open[g] = (l >= 0 ? 0 : open[g]) + sw[i].sum[g];
                if (l >= 0) open_at = l;
                theads += sw[i].heads;
            }
            // carried into this thread
            int32_t at = shfl_up(last, 1);
            uint64_t acc[NS];
#pragma unroll
            for (int g = 0; g < NSUM; g++) {
                const uint64_t u = shfl_up(sum[g], 1);
                acc[g] = lane == 0 ? in[g] : u + (at < 0 ? in[g] : 0);
            }
            at = lane == 0 || at < 0 ? in_at : at;
            int64_t slot = hc + wheads + (heads - my_heads);       // heads before the row
            hc += theads;
#pragma unroll
            for (int r = 0; r < R; r++) {
                if (!((valid >> r) & 1)) continue;
                if (head >> r & 1) {
                    if (slot < o.cap) out_key[slot] = v[r];
                    slot++;
                    at = local0 + r;
#pragma unroll
                    for (int g = 0; g < NSUM; g++) acc[g] = 0;
                }
#pragma unroll
                for (int g = 0; g < NSUM; g++) acc[g] += uint64_t(term[g][r]);
                const bool close = (end >> r & 1) || row0 + r == blk1 - 1;
                if (!close) continue;
#pragma unroll
                for (int k = 0; k < kMaxAgg; k++) {
                    if (k >= a.nagg) break;
                    int64_t x = local0 + r + 1 - (at < 0 ? 0 : at);          // COUNT
#pragma unroll
                    for (int g = 0; g < NSUM; g++)
                        if (a.src[k] == g) x = int64_t(acc[g]);
                    if (at < 0) e.part[k * e.stride + b] = x;
                    else if (slot - 1 < o.cap) o.agg[k][slot - 1] = x;
                }
            }
        }
        if (threadIdx.x == 0) {
            // the block's first row continues a run exactly when its head
            // lies before the block
            e.slot[b] = blk0 > 0 && keys[blk0] == keys[blk0 - 1] ? base - 1 : -1;
            if (b == nblocks - 1) *d_ngroups = hc;
        }
    }
}

// Adds the edges, a wave combining those of neighbouring blocks that belong to
// one run (a run can cover thousands of blocks).
__global__ __launch_bounds__(256) void k_gb_edges(int64_t n, const int64_t *d_n, int nagg, GbOut o, GbEdges e) {
    const int64_t cnt = count_of(d_n, n);
    const int64_t nblocks = ceil_div(cnt, int64_t(kGbTile) * gb_steps(cnt));
    const int lane = lane_id();
    for (int64_t b0 = blockIdx.x * int64_t(blockDim.x); b0 < nblocks; b0 += int64_t(gridDim.x) * blockDim.x) {
        const int64_t b = b0 + threadIdx.x;
        const int64_t slot = b < nblocks ? e.slot[b] : -1;
        const int64_t prev = shfl_up(slot, 1);
        const bool leader = slot >= 0 && slot < o.cap && (lane == 0 || prev != slot);
        for (int k = 0; k < nagg; k++) {
            uint64_t x = slot >= 0 ? uint64_t(e.part[k * e.stride + b]) : 0;
#pragma unroll
            for (int d = 1; d < kWave; d <<= 1) {
                const uint64_t ux = uint64_t(__shfl_down((unsigned long long)x, d, kWave));
                const int64_t us = __shfl_down((long long)slot, d, kWave);
                if (lane + d < kWave && us == slot) x += ux;
            }
            if (leader) atomicAdd(reinterpret_cast<unsigned long long *>(&o.agg[k][slot]), (unsigned long long)x);
        }
    }
}

// ---- dense key domain ------------------------------------------------------
//
// Each workgroup accumulates into LDS: one 64-bit cell per sum and key, and one
// 32-bit row count per key.  LDS atomics on one address serialize, so every
// cell has up to 32 copies (as many as fit), one per lane modulo 32: with 32 the
// lanes of a wave's half never meet, whatever the keys.  A thread takes kDenseR
// rows per step in three rounds of loads: row ids, then the key terms' and the
// value columns' elements, then the additions.
//
// What bounds it: the bytes of the row ids and values (or, gathered from a
// table, their cache lines).  A domain of at most 8 keys used to keep every
// group's accumulators in registers, adding each row to all of them under a
// mask: that was bound by vector arithmetic.  30M rows of 29 bytes in 6 groups:
// 290 -> 184 us; 11.4M rows of 2 bytes in 5 groups: 72 -> 34 us.  A larger domain
// had one copy of each cell, and a grid with 64 rows per thread: 500K rows in 25
// groups 43 -> 12 us.
constexpr int kDenseNT = 512;
constexpr int kDenseR = 4;
constexpr int kDenseMaxCopies = 32;
constexpr int kDenseLds = 40 * 1024;        // LDS the copies may fill (four workgroups per CU)
constexpr int kDenseRows = kDenseNT * kDenseR;

// NT: at least the number of key terms (1, 2 or 4).  key(i) is as pack_keys
// gives it.  Cell of sum g, key b, copy c: s_acc[((g * span + b) << lgc) + c];
// the counts follow.
template <int NT, bool TOG>
__global__ __launch_bounds__(kDenseNT) void k_gb_dense(PackArgs k, int64_t n, const int64_t *d_n,
                                                       int64_t key_lo, int span, int lgc, AggArgs a,
                                                       unsigned long long *__restrict__ gacc) {
    constexpr int R = kDenseR;
    extern __shared__ unsigned long long s_acc[];
    const int cells = span << lgc;
    const int nsum = a.nsum;
    uint32_t *s_cnt = reinterpret_cast<uint32_t *>(s_acc + nsum * cells);
    const int64_t cnt = count_of(d_n, n);
    // only as many workgroups take part as the actual row count feeds: each one costs an
    // addition per cell at the end.  Counts alone take so little per row that these additions
    // show beside them, so there a workgroup takes sixteen rows per cell: 1.5M rows of 300, 800
    // and 1500 keys 21.6, 24.8 and 28.4 -> 18.2, 19.1 and 19.0 us a call.  With a sum, 100K rows of
    // 1500 keys would go from 20 to 33.
    const int64_t feed = nsum == 0 && 16 * span > kDenseRows ? 16 * span : kDenseRows;
    int64_t active = ceil_div(cnt, feed);
    if (active > int64_t(gridDim.x)) active = gridDim.x;
    if (int64_t(blockIdx.x) >= active) return;
    for (int i = threadIdx.x; i < nsum * cells; i += kDenseNT) s_acc[i] = 0;
    for (int i = threadIdx.x; i < cells; i += kDenseNT) s_cnt[i] = 0;
    __syncthreads();
    const int copy = int(threadIdx.x) & ((1 << lgc) - 1);
    for (int64_t base = int64_t(blockIdx.x) * kDenseRows; base < cnt; base += active * kDenseRows) {
        uint32_t in = 0;
        int32_t at[R], row[R], trow[NT][R];
#pragma unroll
        for (int r = 0; r < R; r++) {
            const int64_t i = base + r * kDenseNT + threadIdx.x;
            in |= (i < cnt ? 1u : 0u) << r;
            at[r] = int32_t(i < cnt ? i : 0);               // cnt >= 1 here
        }
        if (a.val_rows) {
#pragma unroll
            for (int r = 0; r < R; r++) row[r] = a.val_rows[at[r]];
        } else {
#pragma unroll
            for (int r = 0; r < R; r++) row[r] = at[r];
        }
#pragma unroll
        for (int t = 0; t < NT; t++) {
            if (t < k.nterms && k.rows[t]) {
#pragma unroll
                for (int r = 0; r < R; r++) trow[t][r] = k.rows[t][at[r]];
            } else {
#pragma unroll
                for (int r = 0; r < R; r++) trow[t][r] = at[r];
            }
        }
        uint64_t traw[NT][R], raw[kTogether][R];
#pragma unroll
        for (int t = 0; t < NT; t++) {
            if (t < k.nterms && k.col[t] && k.len[t] > 0) {
                uint32_t p[R];
#pragma unroll
                for (int r = 0; r < R; r++)
                    p[r] = trow[t][r] >= 0 && trow[t][r] < k.len[t] ? uint32_t(trow[t][r]) : 0u;
                load_typed<R>(k.col[t], k.dt[t], p, traw[t]);
            }
        }
        if constexpr (TOG) {
#pragma unroll
            for (int c = 0; c < kTogether; c++)
                if (c < a.nv) load_value<R>(a, c, row, in, raw[c]);
        }
        uint64_t b[R];
#pragma unroll
        for (int r = 0; r < R; r++) b[r] = 0 - uint64_t(key_lo);
#pragma unroll
        for (int t = 0; t < NT; t++) {
            if (t >= k.nterms) break;
            const uint64_t mul = uint64_t(k.mul[t]);
            if (!k.col[t]) {                                 // constant term
#pragma unroll
                for (int r = 0; r < R; r++) b[r] += mul;
                continue;
            }
            int64_t v[R];
#pragma unroll
            for (int r = 0; r < R; r++)
                v[r] = trow[t][r] >= 0 && trow[t][r] < k.len[t] ? typed_value(traw[t][r], k.dt[t]) : 0;
            const int64_t m = k.mod[t];
            if (m > 0 && (m & (m - 1)) == 0) {
#pragma unroll
                for (int r = 0; r < R; r++) v[r] &= m - 1;
            } else if (m > 0) {
#pragma unroll
                for (int r = 0; r < R; r++) {
                    v[r] %= m;
                    if (v[r] < 0) v[r] += m;
                }
            }
#pragma unroll
            for (int r = 0; r < R; r++) b[r] += mul * uint64_t(v[r]);
        }
        uint32_t ok = 0;
        int cell[R];
#pragma unroll
        for (int r = 0; r < R; r++) {
            const bool hit = ((in >> r) & 1) && b[r] < uint64_t(span);
            ok |= (hit ? 1u : 0u) << r;
            cell[r] = ((hit ? int(b[r]) : 0) << lgc) + copy;
            if (hit) atomicAdd(&s_cnt[cell[r]], 1u);
        }
        for (int g = 0; g < nsum; g++) {
            int64_t t[R];
            sum_terms<R, TOG>(a, g, row, in, raw, t);
#pragma unroll
            for (int r = 0; r < R; r++)
                if ((ok >> r) & 1) atomicAdd(&s_acc[g * cells + cell[r]], (unsigned long long)t[r]);
        }
    }
    __syncthreads();
    // one thread per key and sum (the counts as the last row), its copies read
    // from a different one per lane so that they do not share a bank
    const int ncopy = 1 << lgc;
    for (int i = threadIdx.x; i < (nsum + 1) * span; i += kDenseNT) {
        const int g = i / span, key = i - g * span;
        unsigned long long x = 0;
        if (g < nsum) {
            for (int c = 0; c < ncopy; c++)
                x += s_acc[g * cells + (key << lgc) + ((c + threadIdx.x) & (ncopy - 1))];
        } else {
            for (int c = 0; c < ncopy; c++) x += s_cnt[(key << lgc) + ((c + threadIdx.x) & (ncopy - 1))];
        }
        if (x) atomicAdd(&gacc[i], x);
    }
}

// The groups that occur, from the accumulators [(nsum sums, then counts)][span].
template <class K>
__global__ __launch_bounds__(1024) void k_gb_dense_emit(const unsigned long long *__restrict__ gacc,
                                                        int64_t key_lo, int64_t span, AggArgs a,
                                                        K *out_key, int64_t cap, int64_t *o0,
                                                        int64_t *o1, int64_t *o2, int64_t *o3,
                                                        int64_t *d_ngroups) {
    // 1024 threads x 4 consecutive bins each covers span <= 4096.
    __shared__ int64_t s_scan[1024 / kWave];
    int64_t *outs[4] = {o0, o1, o2, o3};
    const int64_t c0 = int64_t(threadIdx.x) * 4;
    uint32_t live = 0;
    for (int r = 0; r < 4; r++)
        if (c0 + r < span && gacc[a.nsum * span + c0 + r] != 0) live |= 1u << r;
    int64_t total;
    int64_t q = block_excl_scan<1024>(int64_t(__popc(live)), &total, s_scan);
    for (int r = 0; r < 4; r++) {
        if (!(live & (1u << r))) continue;
        if (q < cap) {
            out_key[q] = K(key_lo + c0 + r);
            for (int g = 0; g < a.nagg; g++)
                outs[g][q] = int64_t(gacc[(a.src[g] < 0 ? a.nsum : a.src[g]) * span + c0 + r]);
        }
        q++;
    }
    if (threadIdx.x == 0) *d_ngroups = total;
}

struct GbLayout {
    void *skey;
    int32_t *srows;
    void *sval[kTogether];    // value columns carried through the sort
    void *sort_ws;
    size_t sort_ws_bytes;
    int32_t *bcnt;            // run heads per block
    GbEdges edges;
    int64_t nblocks;          // at most
    unsigned long long *gacc;
    size_t bytes;
};

static bool dense_ok(uint32_t flags, int64_t span, int nagg) {
    return (flags & TQP_GB_DENSE) && span > 0 && span <= TQP_GB_DENSE_MAX &&
           int64_t(nagg + 1) * span * 8 <= 48 * 1024;
}

// An unsorted group-by either sorts row ids along with the keys and reads its values
// through them, a cache line per row and column, or, from kCarryRows rows on (below
// that the columns stay in the caches, and the two are equal), lets up to kTogether
// value columns move along themselves.  A carried byte costs about 0.5 ps per row and
// pass, a line read through a row id 16 ps: so columns are carried up to passes *
// (bytes - 4) = 32 per column, the 4 being the row id's.  us through row ids / carried,
// 12M rows, 3, 5 and 8 passes:
//   one int64     509/404  848/760  1116/1076     int64 + int8    695/476  1116/899  1380/1266
//   two int64     745/564 1148/1129 1419/1620     two int32       729/446  1139/845  1399/1176
constexpr int64_t kCarryRows = int64_t(1) << 20;
static bool carry_values(const AggArgs &a, int64_t n, int key_bits) {
    if (n < kCarryRows || a.val_rows || a.nv < 1 || a.nv > kTogether) return false;
    int bytes = 0;
    for (int c = 0; c < a.nv; c++) bytes += dtype_size(a.vdt[c]);     // (each has n rows at least)
    const int passes = (key_bits + 7) / 8;
    return passes > 0 && passes * (bytes - 4) <= 32 * a.nv;
}

static GbLayout gb_layout(void *ws, int64_t n, int dtype, int nagg, uint32_t flags, int64_t span) {
    GbLayout L = {};
    Carver c(ws);
    const int ks = dtype_size(dtype);
    if (dense_ok(flags, span, nagg)) {
        L.gacc = c.take<unsigned long long>(size_t(nagg + 1) * span);
        L.bytes = c.bytes();
        return L;
    }
    const int64_t nn = n > 0 ? n : 1;
    if (!(flags & TQP_GB_SORTED)) {
        L.skey = c.take<char>(size_t(nn) * ks);
        L.srows = c.take<int32_t>(size_t(nn));
        const bool carry = n >= kCarryRows && nagg > 0;
        for (int v = 0; carry && v < kTogether; v++) L.sval[v] = c.take<int64_t>(size_t(nn));
        L.sort_ws_bytes = sort_ws_bytes(nn, dtype, ks * 8, carry ? 8 * kTogether : 0);
        L.sort_ws = c.take<char>(L.sort_ws_bytes);
    }
    L.nblocks = gb_max_blocks(nn);
    L.bcnt = c.take<int32_t>(size_t(L.nblocks));
    L.edges.slot = c.take<int64_t>(size_t(L.nblocks));
    L.edges.part = c.take<int64_t>(size_t(L.nblocks) * kMaxAgg);
    L.edges.stride = L.nblocks;
    L.bytes = c.bytes();
    return L;
}

// Dense domains: zero the accumulators, aggregate, emit the groups that occur.
// The key is packed from terms as the rows are read (a key column is one term).
template <class OK>
static int dense_groupby(const PackArgs &k, int64_t n, const int64_t *d_n, int64_t key_lo,
                         int64_t key_span, const AggArgs &args, unsigned long long *gacc,
                         OK *out_key, int64_t out_cap, int64_t *const *o, int64_t *d_ngroups,
                         hipStream_t s) {
    int rc = fill_u64(gacc, 0, int64_t(args.nsum + 1) * key_span, s);
    if (rc) return rc;
    if (n > 0) {
        const size_t one = size_t(key_span) * (8 * size_t(args.nsum) + 4);
        int lgc = 0;
        while ((2 << lgc) <= kDenseMaxCopies && (one << (lgc + 1)) <= kDenseLds) lgc++;
        // as many workgroups as are resident; the kernel lets as many of them
        // work as there are rows for
        const unsigned grid = persistent_grid(ceil_div(n, kDenseRows), 2);
        const bool tog = args.nv <= kTogether;
        const int nt = k.nterms;
#define TQP_DENSE(NT, TOG)                                                                          \
        TQP_LAUNCH("gb_dense", (k_gb_dense<NT, TOG>), dim3(grid), dim3(kDenseNT), one << lgc, s, k, n,   \
                   d_n, key_lo, int(key_span), lgc, args, gacc)
        if (tog && nt == 1) TQP_DENSE(1, true);
        else if (tog && nt == 2) TQP_DENSE(2, true);
        else if (tog) TQP_DENSE(4, true);
        else if (nt <= 2) TQP_DENSE(2, false);
        else TQP_DENSE(4, false);
#undef TQP_DENSE
        if ((rc = check_launch("group-by dense"))) return rc;
    }
    TQP_LAUNCH("gb_dense_emit", k_gb_dense_emit<OK>, dim3(1), dim3(1024), 0, s, gacc, key_lo,
               key_span, args, out_key, out_cap, o[0], o[1], o[2], o[3], d_ngroups);
    return check_launch("group-by dense emit");
}

template <class K>
static int groupby_typed(const tqp_col *key, const int64_t *d_n, uint32_t flags, int64_t key_lo,
                         int64_t key_span, const AggArgs &args, const tqp_col *out_key,
                         int64_t *const *out_aggs, int64_t *d_ngroups, void *ws, hipStream_t s) {
    const int64_t n = key->len;
    const int nagg = args.nagg;
    GbLayout L = gb_layout(ws, n, key->dtype, nagg, flags, key_span);
    int64_t *o[4] = {nullptr, nullptr, nullptr, nullptr};
    for (int g = 0; g < nagg; g++) o[g] = out_aggs[g];
    int rc;
    if (dense_ok(flags, key_span, nagg)) {
        PackArgs p = {};
        p.col[0] = key->data;
        p.len[0] = n;
        p.mul[0] = 1;
        p.dt[0] = key->dtype;
        p.nterms = 1;
        return dense_groupby<K>(p, n, d_n, key_lo, key_span, args, L.gacc,
                                static_cast<K *>(out_key->data), out_key->len, o, d_ngroups, s);
    }
    const K *k = static_cast<const K *>(key->data);
    AggArgs a = args;
    if (!(flags & TQP_GB_SORTED)) {
        int64_t kmin = key_lo;
        int kbits = 0;
        if (key_span > 0) {
            while (kbits < 64 && (uint64_t(key_span - 1) >> kbits) != 0) kbits++;
        } else {
            rc = derive_key_range(k, key->dtype, n, d_n, L.sort_ws, L.sort_ws_bytes, s, &kmin,
                                  &kbits);
            if (rc) return rc;
        }
        if (carry_values(args, n, kbits)) {
            rc = sort_columns(k, key->dtype, n, d_n, kbits, kmin, L.skey, args.val, L.sval, args.vdt,
                              args.nv, L.sort_ws, L.sort_ws_bytes, s);
            for (int c = 0; c < args.nv; c++) a.val[c] = L.sval[c];
        } else {
            rc = sort_impl(k, key->dtype, args.val_rows, n, d_n, kbits, kmin, L.skey, L.srows,
                           L.sort_ws, L.sort_ws_bytes, s);
            a.val_rows = L.srows;
        }
        if (rc) return rc;
        k = static_cast<const K *>(L.skey);
    }
    K *ok = static_cast<K *>(out_key->data);
    GbOut out = {};
    out.cap = out_key->len;
    for (int g = 0; g < nagg; g++) out.agg[g] = o[g];
    TQP_LAUNCH("gb_heads", k_gb_heads<K>, dim3(block_grid(L.nblocks, d_n)), dim3(kGbNT), 0, s, k, n, d_n,
               L.bcnt);
    if ((rc = check_launch("group-by heads"))) return rc;
    const unsigned grid = persistent_grid(L.nblocks, tune(kTuneGbScanPerCu));
#define TQP_SCAN(NSUM, TOG)                                                                         \
    TQP_LAUNCH("gb_scan", (k_gb_runs<K, NSUM, TOG>), dim3(grid), dim3(kGbNT), 0, s, k, n, d_n, a, ok, out, \
               d_ngroups, L.bcnt, L.edges)
    const bool tog = a.nv <= kTogether;
    switch (a.nsum) {
    case 0: TQP_SCAN(0, true); break;
    case 1: TQP_SCAN(1, true); break;                    // one sum names at most two columns
    case 2: if (tog) TQP_SCAN(2, true); else TQP_SCAN(2, false); break;
    case 3: if (tog) TQP_SCAN(3, true); else TQP_SCAN(3, false); break;
    default: if (tog) TQP_SCAN(4, true); else TQP_SCAN(4, false); break;
    }
#undef TQP_SCAN
    if ((rc = check_launch("group-by runs"))) return rc;
    if (L.nblocks == 1) return TQP_OK;                   // one block has no edges
    TQP_LAUNCH("gb_edges", k_gb_edges, dim3(unsigned(ceil_div(L.nblocks, 256))), dim3(256), 0, s, n, d_n, nagg,
               out, L.edges);
    return check_launch("group-by edges");
}

}  // namespace tqp

using namespace tqp;

// Checks the value columns and aggregates of a group-by call and fills
// AggArgs; n is the row count value columns must cover without val_rows.
static int agg_args(const tqp_col *vals, int nvals, const int32_t *val_rows, const tqp_agg *aggs,
                    int nagg, int64_t n, int64_t out_cap, int64_t *const *out_aggs, AggArgs *a,
                    const char *who) {
    *a = AggArgs{};
    for (int c = 0; c < nvals; c++) {
        if (!dtype_ok(vals[c].dtype) || (vals[c].len > 0 && !vals[c].data) ||
            !col_aligned(vals[c].data, vals[c].dtype))
            return set_error(TQP_EINVAL, "%s: value column %d is invalid or unaligned", who, c);
        if (!val_rows && vals[c].len < n)
            return set_error(TQP_EINVAL, "%s: value column %d is shorter than keys", who, c);
    }
    // the distinct columns the sums name, in order of first use
    const int64_t most = int64_t(1) << 31;
    auto slot = [&](int c) {
        const int64_t l = vals[c].len;
        const uint32_t len = uint32_t(l < 0 ? 0 : l < most ? l : most);
        for (int v = 0; v < a->nv; v++)
            if (a->val[v] == vals[c].data && a->vdt[v] == vals[c].dtype && a->vlen[v] == len) return v;
        a->val[a->nv] = vals[c].data;
        a->vdt[a->nv] = vals[c].dtype;
        a->vlen[a->nv] = len;
        return int(a->nv++);
    };
    for (int g = 0; g < nagg; g++) {
        const tqp_agg &x = aggs[g];
        if (x.op < TQP_AGG_SUM || x.op > TQP_AGG_SUM_DIFF_PRODUCT)
            return set_error(TQP_EINVAL, "%s: aggregate %d has a bad op", who, g);
        if (x.op != TQP_AGG_COUNT && (x.a < 0 || x.a >= nvals))
            return set_error(TQP_EINVAL, "%s: aggregate %d names a missing column", who, g);
        if (x.op >= TQP_AGG_SUM_PRODUCT && (x.b < 0 || x.b >= nvals))
            return set_error(TQP_EINVAL, "%s: aggregate %d names a missing column", who, g);
        if (out_cap > 0 && !out_aggs[g]) return set_error(TQP_EINVAL, "%s: output %d is null", who, g);
        a->src[g] = -1;
        if (x.op == TQP_AGG_COUNT) continue;
        const int t = a->nsum++;
        a->src[g] = t;
        a->op[t] = x.op;
        a->sa[t] = slot(x.a);
        a->sb[t] = x.op >= TQP_AGG_SUM_PRODUCT ? slot(x.b) : -1;
        a->ic[t] = x.c;
    }
    if (val_rows && !col_aligned(val_rows, TQP_INT32))
        return set_error(TQP_EINVAL, "%s: val_rows must be 4-byte aligned", who);
    a->nagg = nagg;
    a->val_rows = val_rows;
    return TQP_OK;
}

TQP_API size_t tqp_groupby_workspace_bytes(int64_t n, int dtype, int nagg, uint32_t flags,
                                           int64_t key_span) {
    if (n < 0 || (dtype != TQP_INT32 && dtype != TQP_INT64) || nagg < 1 || nagg > kMaxAgg)
        return 0;
    return gb_layout(nullptr, n, dtype, nagg, flags, key_span).bytes;
}

TQP_API int tqp_groupby_agg(const tqp_col *key, const int64_t *d_n, uint32_t flags, int64_t key_lo,
                            int64_t key_span, const tqp_col *vals, int nvals,
                            const int32_t *val_rows, const tqp_agg *aggs, int nagg,
                            const tqp_col *out_key, int64_t *const *out_aggs, int64_t *d_ngroups,
                            void *ws, size_t ws_bytes, void *stream) {
    clear_error();
    if (!key || !out_key || !aggs || !out_aggs || !d_ngroups)
        return set_error(TQP_EINVAL, "tqp_groupby_agg: null argument");
    if (key->dtype != TQP_INT32 && key->dtype != TQP_INT64)
        return set_error(TQP_EINVAL, "tqp_groupby_agg: keys must be int32 or int64");
    if (out_key->dtype != key->dtype)
        return set_error(TQP_EINVAL, "tqp_groupby_agg: out_key dtype must equal the key dtype");
    if (nagg < 1 || nagg > kMaxAgg)
        return set_error(TQP_EINVAL, "tqp_groupby_agg: nagg must be in [1, %d]", kMaxAgg);
    if (nvals < 0 || nvals > kMaxVals || (nvals > 0 && !vals))
        return set_error(TQP_EINVAL, "tqp_groupby_agg: nvals must be in [0, %d]", kMaxVals);
    if (flags & ~(TQP_GB_SORTED | TQP_GB_DENSE))
        return set_error(TQP_EINVAL, "tqp_groupby_agg: unknown flag bits");
    if ((flags & TQP_GB_DENSE) && (key_span < 1 || key_span > TQP_GB_DENSE_MAX))
        return set_error(TQP_EINVAL, "tqp_groupby_agg: dense needs 1 <= key_span <= %d",
                         TQP_GB_DENSE_MAX);
    if (key_span < 0) return set_error(TQP_EINVAL, "tqp_groupby_agg: negative key_span");
    const int64_t n = key->len;
    if (n < 0 || n > (int64_t(1) << 30) - 1)
        return set_error(TQP_EINVAL, "tqp_groupby_agg: n must be in [0, 2^30 - 1]");
    if ((n > 0 && !key->data) || (out_key->len > 0 && !out_key->data))
        return set_error(TQP_EINVAL, "tqp_groupby_agg: null key data");
    AggArgs a = {};
    int rc = agg_args(vals, nvals, val_rows, aggs, nagg, n, out_key->len, out_aggs, &a,
                      "tqp_groupby_agg");
    if (rc) return rc;
    const size_t need = tqp_groupby_workspace_bytes(n, key->dtype, nagg, flags, key_span);
    if (!ws || ws_bytes < need)
        return set_error(TQP_ECAPACITY, "tqp_groupby_agg: workspace needs %zu bytes", need);
    hipStream_t s = as_stream(stream);
    if (key->dtype == TQP_INT32)
        return groupby_typed<int32_t>(key, d_n, flags, key_lo, key_span, a, out_key, out_aggs,
                                      d_ngroups, ws, s);
    return groupby_typed<int64_t>(key, d_n, flags, key_lo, key_span, a, out_key, out_aggs,
                                  d_ngroups, ws, s);
}

TQP_API size_t tqp_groupby_terms_workspace_bytes(int nagg, int64_t key_span) {
    if (nagg < 1 || nagg > kMaxAgg || !dense_ok(TQP_GB_DENSE, key_span, nagg)) return 0;
    Carver c(nullptr);
    c.take<unsigned long long>(size_t(nagg + 1) * size_t(key_span));
    return c.bytes();
}

TQP_API int tqp_groupby_agg_terms(const tqp_keyterm *terms, int nterms, int64_t n,
                                  const int64_t *d_n, int64_t key_lo, int64_t key_span,
                                  const tqp_col *vals, int nvals, const int32_t *val_rows,
                                  const tqp_agg *aggs, int nagg, const tqp_col *out_key,
                                  int64_t *const *out_aggs, int64_t *d_ngroups, void *ws,
                                  size_t ws_bytes, void *stream) {
    clear_error();
    if (!terms || !out_key || !aggs || !out_aggs || !d_ngroups)
        return set_error(TQP_EINVAL, "tqp_groupby_agg_terms: null argument");
    if (nterms < 1 || nterms > 4)
        return set_error(TQP_EINVAL, "tqp_groupby_agg_terms: nterms must be in [1, 4]");
    if (out_key->dtype != TQP_INT32 && out_key->dtype != TQP_INT64)
        return set_error(TQP_EINVAL, "tqp_groupby_agg_terms: out_key must be int32 or int64");
    if (out_key->len > 0 && !out_key->data)
        return set_error(TQP_EINVAL, "tqp_groupby_agg_terms: null out_key data");
    if (nagg < 1 || nagg > kMaxAgg)
        return set_error(TQP_EINVAL, "tqp_groupby_agg_terms: nagg must be in [1, %d]", kMaxAgg);
    if (nvals < 0 || nvals > kMaxVals || (nvals > 0 && !vals))
        return set_error(TQP_EINVAL, "tqp_groupby_agg_terms: nvals must be in [0, %d]", kMaxVals);
    if (!dense_ok(TQP_GB_DENSE, key_span, nagg))
        return set_error(TQP_EINVAL,
                         "tqp_groupby_agg_terms: need 1 <= key_span and (nagg + 1) * key_span <= 6144");
    if (out_key->dtype == TQP_INT32 &&
        (key_lo < INT32_MIN || key_lo + key_span - 1 > INT32_MAX))
        return set_error(TQP_EINVAL, "tqp_groupby_agg_terms: the key range does not fit int32");
    if (n < 0 || n > (int64_t(1) << 30) - 1)
        return set_error(TQP_EINVAL, "tqp_groupby_agg_terms: n must be in [0, 2^30 - 1]");
    PackArgs p;
    int rc = pack_args(terms, nterms, n, &p, "tqp_groupby_agg_terms");
    if (rc) return rc;
    AggArgs a;
    rc = agg_args(vals, nvals, val_rows, aggs, nagg, n, out_key->len, out_aggs, &a,
                  "tqp_groupby_agg_terms");
    if (rc) return rc;
    const size_t need = tqp_groupby_terms_workspace_bytes(nagg, key_span);
    if (!ws || ws_bytes < need)
        return set_error(TQP_ECAPACITY, "tqp_groupby_agg_terms: workspace needs %zu bytes", need);
    int64_t *o[4] = {nullptr, nullptr, nullptr, nullptr};
    for (int g = 0; g < nagg; g++) o[g] = out_aggs[g];
    hipStream_t s = as_stream(stream);
    unsigned long long *gacc = static_cast<unsigned long long *>(ws);
    if (out_key->dtype == TQP_INT32)
        return dense_groupby<int32_t>(p, n, d_n, key_lo, key_span, a, gacc,
                                      static_cast<int32_t *>(out_key->data), out_key->len, o,
                                      d_ngroups, s);
    return dense_groupby<int64_t>(p, n, d_n, key_lo, key_span, a, gacc,
                                  static_cast<int64_t *>(out_key->data), out_key->len, o,
                                  d_ngroups, s);
}
