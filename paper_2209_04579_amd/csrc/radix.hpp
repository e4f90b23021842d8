#pragma once
// Stable LSD radix passes over an ordinal of each key, carrying row ids and up
// to four payload columns.  The ordinal is a functor: the key itself (minus
// its minimum) for the sort, or a bucket number for a partitioner.
//
// Keys are ranked on u = key - key_min (unsigned), which orders signed keys
// correctly and drops the bits that never vary.  The b significant bits are
// cut into ceil(b / 8) digits of equal width (at most 8 bits: 21 bits take
// three 7-bit digits, not 8 + 8 + 5), so each pass has as few bins, and as
// long runs per bin, as its pass count allows.  A pass first counts each tile's
// digits; then
//   * a workgroup takes a 4096-key tile,
//   * ranks its keys stably: each wave walks its items in input order, finds
//     the lanes holding the same digit with one ballot per digit bit, and
//     bumps a per-wave LDS counter once per distinct digit,
//   * adds the counts of the tiles before for the global start of each digit run,
//   * then, column by column (keys, payloads, row ids), stages the tile in LDS
//     in digit order and writes each digit run out with consecutive threads on
//     consecutive addresses.
// A sort of one tile does all of its passes in LDS, in one launch.
// Carrying the payload through the passes keeps every later read of it
// sequential, instead of a random gather through a permutation.
#include "rowtest.hpp"

namespace tqp {

constexpr int kSortNT = 1024;
constexpr int kSortIPT = 4;
constexpr int kSortTile = kSortNT * kSortIPT;
constexpr int64_t kSortLargeRows = int64_t(1) << 25;
constexpr int kRadixBits = 8;
constexpr int kBins = 1 << kRadixBits;
constexpr int kSortNW = kSortNT / kWave;
constexpr int kMaxSortPay = 4;
constexpr int kMaxPassCols = kMaxSortPay + 1;   // payload columns + row ids
constexpr int kMaxSortPred = 4;            // predicates of a filtered first pass
// Consecutive tiles write adjacent parts of every digit run, so the cache lines
// they share are completed in one L2 if one XCD takes them: workgroups are
// dispatched to the chip's 8 XCDs round robin by index, so the workgroups b with
// equal b % kXcds share tile groups of kTileGroup consecutive tiles.
constexpr int kXcds = 8;
constexpr int kTileGroup = 8;

// ---- where every tile's digit runs go ------------------------------------------
//
// The global position of tile t's run of digit d is the number of items with a
// smaller digit, plus those of digit d in the tiles before t.  The tiles are
// taken in groups of G consecutive ones (G from the item count, so that every
// kernel agrees on it without the host):
//   k_radix_count  counts[t][d] for every tile, csum[g][d] for every group;
//   k_radix_scan   turns csum into the counts of the groups before, per digit,
//                  and leaves the digit's total in dtot;
//   k_onesweep     adds up to G - 1 rows of counts of its own group.
// Up to kDirectTiles tiles, k_onesweep adds up all the rows itself and there is no
// scan.
// No workgroup waits for another.  (A decoupled look-back over the tiles, which
// this replaces, took one pass over the keys less per digit, but its chain of
// dependent loads cost more: 5M int64 keys with row ids 45 us a pass against
// 8 + 6 + 28 for these three, 1.5M int32 keys with row ids 21 against 4 + 3 + 11,
// 30M rows of 21 bytes 312 against 20 + 7 + 268.)
__host__ __device__ inline uint32_t tile_count(int64_t cnt) { return uint32_t((cnt + kSortTile - 1) / kSortTile); }
__host__ __device__ inline uint32_t tiles_per_group(uint32_t ntiles) {
    return ntiles >= 8192 ? 8 : ntiles >= 4096 ? 4 : ntiles >= 2048 ? 2 : 1;
}
// groups any count up to the one of ntiles can make
inline int64_t max_tile_groups(int64_t ntiles) {
    const int64_t g = ceil_div(ntiles, int64_t(tiles_per_group(uint32_t(ntiles))));
    return ntiles < 2048 ? ntiles : g < 2048 ? 2048 : g;
}

constexpr uint32_t kDirectTiles = 32;

// Counting uses LDS atomics, and atomics on one address serialize (skewed keys,
// or a digit with few values): every bin has kCopies copies, lane l using copy l
// modulo their number, so that lanes rarely meet on an address or a bank.
constexpr int kCountNT = 512;
constexpr int kCountIPT = 8;
static_assert(kCountNT * kCountIPT == kSortTile, "a counting step is one tile");
constexpr int kCopiesLg = 4;
constexpr int kCopies = 1 << kCopiesLg;

// kCountIPT consecutive keys from row0; those at or past cnt read as 0.
template <class K>
__device__ __forceinline__ void count_keys(const K *keys, int64_t row0, int64_t cnt, bool vec,
                                           K (&v)[kCountIPT]) {
    if (vec && row0 + kCountIPT <= cnt) {
        constexpr int kPer = 16 / sizeof(K);
        const int4 *q = reinterpret_cast<const int4 *>(keys + row0);
#pragma unroll
        for (int j = 0; j < kCountIPT / kPer; j++) {
            const int4 x = q[j];
            const K *e = reinterpret_cast<const K *>(&x);
#pragma unroll
            for (int t = 0; t < kPer; t++) v[j * kPer + t] = e[t];
        }
    } else {
#pragma unroll
        for (int r = 0; r < kCountIPT; r++) v[r] = row0 + r < cnt ? keys[row0 + r] : K(0);
    }
}

// ND > 0: only rows that pass the tests t (on at most ND columns, loaded
// together) count, and one keep bit per row is written: bit i % 8 of byte i / 8,
// in every byte up to the last row's.
template <class K, class Ord, int ND>
__global__ __launch_bounds__(kCountNT) void k_radix_count(const K *__restrict__ keys, int64_t n,
                                                          const int64_t *d_n, Ord ord, int shift, int dbits,
                                                          uint32_t *__restrict__ counts,
                                                          uint32_t *__restrict__ csum, RowTests t, int vec,
                                                          uint8_t *__restrict__ keep) {
    __shared__ uint32_t s_c[2][kBins << kCopiesLg];
    const int64_t cnt = count_of(d_n, n);
    const uint32_t ntiles = tile_count(cnt);
    const uint32_t G = tiles_per_group(ntiles);
    const uint32_t nbins = 1u << dbits, dmask = nbins - 1;
    const int tid = threadIdx.x;
    const bool kvec = reinterpret_cast<uintptr_t>(keys) % 16 == 0;
    for (int i = tid; i < kBins << kCopiesLg; i += kCountNT) s_c[0][i] = s_c[1][i] = 0;
    __syncthreads();
    int buf = 0;
    for (uint32_t g = blockIdx.x; g * G < ntiles; g += gridDim.x) {
        uint32_t sum = 0;
        for (uint32_t tile = g * G; tile < g * G + G && tile < ntiles; tile++) {
            const int64_t row0 = int64_t(tile) * kSortTile + tid * kCountIPT;
            uint32_t *mine = s_c[buf] + (tid & (kCopies - 1));
            uint32_t m = row0 + kCountIPT <= cnt ? 0xffu : row0 < cnt ? (1u << int(cnt - row0)) - 1u : 0u;
            K v[kCountIPT];
            if constexpr (ND > 0) {
                RawRows<kCountIPT> raw[ND];
#pragma unroll
                for (int c = 0; c < ND; c++)
                    if (c < t.ncol) load_rawrows<kCountIPT>(t.col[c], t.dt[c], row0, cnt, vec != 0, raw[c]);
                count_keys(keys, row0, cnt, kvec, v);
#pragma unroll
                for (int c = 0; c < ND; c++)
                    if (c < t.ncol) m &= test_rows<kCountIPT>(t, t.beg[c], t.beg[c + 1], t.dt[c], raw[c]);
                if (row0 < cnt) keep[row0 / kCountIPT] = uint8_t(m);
            } else {
                count_keys(keys, row0, cnt, kvec, v);
            }
#pragma unroll
            for (int r = 0; r < kCountIPT; r++)
                if ((m >> r) & 1) atomicAdd(&mine[(uint32_t(ord(v[r]) >> shift) & dmask) << kCopiesLg], 1u);
            __syncthreads();
            // read (and clear for the tile after next) the copies, each lane
            // starting at another one; the next tile counts into the other half
            if (tid < int(nbins)) {
                uint32_t x = 0;
#pragma unroll
                for (int j = 0; j < kCopies; j++) {
                    uint32_t *p = &s_c[buf][(tid << kCopiesLg) + ((j + tid) & (kCopies - 1))];
                    x += *p;
                    *p = 0;
                }
                counts[tile * kBins + tid] = x;
                sum += x;
            }
            buf ^= 1;
        }
        if (tid < int(nbins)) csum[g * kBins + tid] = sum;
        __syncthreads();
    }
}

// csum[g][d] becomes the sum over the groups before g, dtot[d] the total.  A
// workgroup takes kScanDigits digits (one 32-byte part of every row), a column of
// kScanLanes threads per digit, each kScanPer consecutive groups.
constexpr int kScanNT = 1024;
constexpr int kScanDigits = 8;
constexpr int kScanLanes = kScanNT / kScanDigits;
constexpr int kScanPer = 16;
static __global__ __launch_bounds__(kScanNT) void k_radix_scan(uint32_t *csum, uint32_t *dtot, int64_t n,
                                                               const int64_t *d_n) {
    __shared__ uint32_t s_sum[kScanDigits][kScanLanes + 1];
    const uint32_t ntiles = tile_count(count_of(d_n, n));
    const uint32_t G = tiles_per_group(ntiles);
    const uint32_t ng = (ntiles + G - 1) / G;
    const int d = threadIdx.x % kScanDigits, col = threadIdx.x / kScanDigits;
    uint32_t *p = csum + blockIdx.x * kScanDigits + d;
    const int w = wave_id(), lane = lane_id();
    uint32_t carry = 0;
    for (uint32_t g0 = 0; g0 < ng; g0 += kScanLanes * kScanPer) {
        const uint32_t gb = g0 + col * kScanPer;
        uint32_t v[kScanPer], sum = 0;
#pragma unroll
        for (int j = 0; j < kScanPer; j++) {
            v[j] = gb + j < ng ? p[(gb + j) * kBins] : 0u;
            sum += v[j];
        }
        s_sum[d][col] = sum;
        __syncthreads();
        if (w < kScanDigits) {                          // wave w scans digit w's column
            uint32_t base = 0;
#pragma unroll
            for (int h = 0; h < kScanLanes; h += kWave) {
                const uint32_t x = s_sum[w][h + lane];
                const uint32_t inc = wave_incl_scan(x);
                s_sum[w][h + lane] = base + inc - x;
                base += shfl(inc, kWave - 1);
            }
            if (lane == 0) s_sum[w][kScanLanes] = base;
        }
        __syncthreads();
        uint32_t ex = carry + s_sum[d][col];
        carry += s_sum[d][kScanLanes];
#pragma unroll
        for (int j = 0; j < kScanPer; j++) {
            if (gb + j < ng) p[(gb + j) * kBins] = ex;
            ex += v[j];
        }
        __syncthreads();
    }
    if (col == 0) dtot[blockIdx.x * kScanDigits + d] = carry;
}

// ---- passes ------------------------------------------------------------------

// The columns a pass moves with its keys: the payload columns, then the row
// ids when they are produced.  A null source is the item's position (the row
// ids of a first pass).
struct PassCols {
    const void *pin[kMaxPassCols];
    void *pout[kMaxPassCols];
    int32_t pdt[kMaxPassCols];
    int32_t ncols;
};

// One wave's items of a tile: item k of a lane is position at + k * 64, `at` the
// lane's first.  Whole tiles read from one address with constant offsets; in
// the last tile, positions past the end read the last item instead (a tile
// exists only if cnt >= 1).
template <class T, class O>
__device__ __forceinline__ void load_items(const T *p, uint32_t at, uint32_t cnt, bool whole,
                                           O (&out)[kSortIPT]) {
    if (whole) {
        const T *q = p + at;
#pragma unroll
        for (int k = 0; k < kSortIPT; k++) out[k] = O(q[k * kWave]);
    } else {
#pragma unroll
        for (int k = 0; k < kSortIPT; k++) {
            const uint32_t i = at + k * kWave;
            out[k] = O(p[i < cnt ? i : cnt - 1]);
        }
    }
}

// Column p of a wave's items, zero-extended: one branch on the type around its
// loads.
__device__ __forceinline__ void load_column(const PassCols &c, int p, uint32_t at, uint32_t cnt,
                                            bool whole, uint64_t (&out)[kSortIPT]) {
    const void *src = c.pin[p];
    const int dt = c.pdt[p];
    if (!src) {
#pragma unroll
        for (int k = 0; k < kSortIPT; k++) out[k] = at + k * kWave;
    } else if (dt == TQP_INT64) {
        load_items(static_cast<const uint64_t *>(src), at, cnt, whole, out);
    } else if (dt == TQP_INT32) {
        load_items(static_cast<const uint32_t *>(src), at, cnt, whole, out);
    } else {
        load_items(static_cast<const uint8_t *>(src), at, cnt, whole, out);
    }
}

// Stages a column of the tile in digit order: item k at pos[k] (kNoPos: missing).
constexpr uint32_t kNoPos = ~0u;
template <class T>
__device__ __forceinline__ void stage_items(void *s_stage, const uint32_t (&pos)[kSortIPT], bool all,
                                            const uint64_t (&v)[kSortIPT]) {
    T *st = static_cast<T *>(s_stage);
#pragma unroll
    for (int k = 0; k < kSortIPT; k++)
        if (all || pos[k] != kNoPos) st[pos[k]] = T(v[k]);
}

// Writes a staged column to its runs: thread t writes tile positions t,
// t + kSortNT, ... below tile_cnt to the global positions in gpos[].
template <class T>
__device__ __forceinline__ void flush_stage(const void *s_stage, const uint32_t (&gpos)[kSortIPT],
                                            int tile_cnt, void *dst) {
    const T *st = static_cast<const T *>(s_stage) + threadIdx.x;
    T *out = static_cast<T *>(dst);
    if (tile_cnt == kSortTile) {
#pragma unroll
        for (int k = 0; k < kSortIPT; k++) out[gpos[k]] = st[k * kSortNT];
    } else {
#pragma unroll
        for (int k = 0; k < kSortIPT; k++)
            if (int(threadIdx.x) + k * kSortNT < tile_cnt) out[gpos[k]] = st[k * kSortNT];
    }
}

// One LSD pass.  The columns of c (dtypes at run time) move with the keys, one
// after another through the same 32 KiB of LDS: a column's loads are issued
// while the one before it is written.
//
// What bounds it: on wide rows the traffic itself (each column read and
// written once, the writes in runs of about 4096 / bins items); on narrow ones
// the phases between barriers.  So the kernel is kept to 64
// registers (2 of them in scratch, 6 with int64 keys and a filter) and 42 KiB of LDS, and two workgroups of 16 waves (all a CU can
// hold) share a CU: one's waits are the other's work.  (512 threads of 8 items
// take 100 to 128 registers, so half the waves.)  10M rows of 21 bytes: 139 -> 100
// us (4.2 TB/s); 30M of them: 312 -> 268 (4.7); the filtered first pass of 60M,
// half of them kept: 572 -> 466.  Slower than
// with those tiles: 30M rows with four 8-byte columns, by 4 to 13% (64-bit keys, the whole
// sort 5467 -> 6272), whose runs of 16 items are half as long.
//
// FILT: items whose bit in keep_bits is clear (bit i % 64 of
// word i / 64, written by the filtered count) are dropped, as items past
// the end are, so the pass also compacts: its output holds the kept items,
// sorted by the digit, in their input order within a digit, and their number
// (the digits' total) goes to *d_kept.
template <class K, class Ord, bool FILT>
__global__ __launch_bounds__(kSortNT, 8) void k_onesweep(
    const K *__restrict__ keys_in, K *__restrict__ keys_out, PassCols c, int64_t n,
    const int64_t *d_n, Ord ord, int shift, int digit_bits, const uint32_t *__restrict__ counts,
    const uint32_t *__restrict__ csum, const uint32_t *__restrict__ dtot,
    const uint64_t *__restrict__ keep_bits, int64_t *d_kept) {
    static_assert(kSortNW * kBins * 2 == kSortNT * 8, "one 8-byte store per thread clears the counters");
    __shared__ uint64_t s_stage[kSortTile];     // one column of the tile, in digit order
    // per wave and digit: items counted so far, then the tile position of the
    // wave's first item of the digit
    __shared__ __attribute__((aligned(8))) uint16_t s_hist[kSortNW][kBins];
    __shared__ uint32_t s_gbase[kBins];         // global start of the run minus its local start (wrapping)
    // per wave of digits: items of the tile, items of all tiles
    __shared__ uint32_t s_wtot[kBins / kWave], s_wall[kBins / kWave];

    const uint32_t cnt = uint32_t(count_of(d_n, n));
    const uint32_t ntiles = tile_count(cnt);
    const uint32_t G = tiles_per_group(ntiles);
    const int tid = threadIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(wave_id());
    const int lane = lane_id();
    const bool direct = ntiles <= kDirectTiles;
    // this workgroup's tiles: every (grid / kXcds)-th of its XCD's (one, when the
    // grid has a workgroup for every tile)
    const uint32_t xcd = blockIdx.x % kXcds;
    for (uint32_t j = blockIdx.x / kXcds;; j += gridDim.x / kXcds) {
    const uint32_t tile = ((j / kTileGroup) * kXcds + xcd) * kTileGroup + j % kTileGroup;
    if ((j / kTileGroup) * (kXcds * kTileGroup) >= ntiles) break;
    if (tile >= ntiles) continue;
    if (j != blockIdx.x / kXcds) __syncthreads();    // the tile before is out of LDS
    // opaque here, so that no test of it is kept in registers across tiles
    int dbits = digit_bits;
    asm volatile("" : "+s"(dbits));
    const uint32_t nbins = 1u << dbits;
    const uint32_t tile0 = tile * kSortTile;
    const uint32_t wave0 = tile0 + w * (kWave * kSortIPT);
    const uint32_t at = wave0 + lane;
    const bool whole = tile0 + kSortTile <= cnt;
    const bool all = whole && !FILT;             // no item is missing

    K key[kSortIPT];
    load_items(keys_in, at, cnt, whole, key);
    uint64_t kept[FILT ? kSortIPT : 1];
    if constexpr (FILT) {
        // item k of every lane lies in one 64-item word (wave0 is a multiple of 64)
        const uint32_t last = (cnt - 1) >> 6;
#pragma unroll
        for (int k = 0; k < kSortIPT; k++) {
            const uint32_t wi = (wave0 >> 6) + k;
            kept[k] = keep_bits[wi < last ? wi : last];
        }
    }
    // items of digit tid in the tiles before, and in all tiles
    uint32_t toff = 0, dall = 0;
    if (tid < int(nbins)) {
        if (direct) {
#pragma unroll 8
            for (uint32_t t = 0; t < ntiles; t++) {
                const uint32_t x = counts[t * kBins + tid];
                dall += x;
                toff += t < tile ? x : 0;
            }
        } else {
            const uint32_t g = tile / G;
            dall = dtot[tid];
            toff = csum[g * kBins + tid];
            for (uint32_t t = g * G; t < tile; t++) toff += counts[t * kBins + tid];
        }
    }
    reinterpret_cast<uint64_t *>(s_hist)[tid] = 0;
    __syncthreads();

    // Stable rank of each item among the items of this wave with its digit:
    // dp = digit << 16 | rank, kNoPos for a missing item.
    uint32_t dp[kSortIPT];
#pragma unroll
    for (int k = 0; k < kSortIPT; k++) {
        const uint32_t d = uint32_t(ord(key[k]) >> shift) & (nbins - 1);
        bool valid = true;
        uint64_t peers = ~uint64_t(0);
        if (!all) {
            valid = at + k * kWave < cnt;
            if constexpr (FILT) valid = valid && ((kept[k] >> lane) & 1);
            peers = ballot(valid);
        }
        uint32_t plo = uint32_t(peers), phi = uint32_t(peers >> 32);
#pragma unroll
        for (int b = 0; b < kRadixBits; b++) {
            if (b >= dbits) break;                   // higher digit bits are all zero
            const uint32_t set = uint32_t(int32_t(d << (31 - b)) >> 31);     // 0 or ~0
            const uint64_t bb = ballot(set != 0);
            plo &= ~(uint32_t(bb) ^ set);
            phi &= ~(uint32_t(bb >> 32) ^ set);
        }
        const uint32_t before = __builtin_amdgcn_mbcnt_hi(phi, __builtin_amdgcn_mbcnt_lo(plo, 0));
        uint16_t *h = &s_hist[w][d];
        const uint32_t old = *h;
        dp[k] = valid ? (d << 16) | (old + before) : kNoPos;
        if (valid && before == 0) *h = uint16_t(old + __popc(plo) + __popc(phi));
    }
    __syncthreads();

    // Per digit (threads below kBins): the tile total, the tile-local start of
    // the digit's run in each wave, and where the run goes.
    uint32_t local = 0, start = 0;
    if (tid < kBins) {
        uint32_t tot = 0;
#pragma unroll
        for (int ww = 0; ww < kSortNW; ww++) tot += s_hist[ww][tid];
        local = wave_incl_scan(tot);
        start = wave_incl_scan(dall);
        if (lane == kWave - 1) {
            s_wtot[w] = local;
            s_wall[w] = start;
        }
        local -= tot;
        start -= dall;
    }
    __syncthreads();
    if (tid < kBins) {
        for (int i = 0; i < w; i++) {
            local += s_wtot[i];
            start += s_wall[i];
        }
        if (FILT && tile == 0 && tid == kBins - 1) *d_kept = int64_t(start) + dall;
        s_gbase[tid] = start + toff - local;
        uint32_t run = local;
#pragma unroll
        for (int ww = 0; ww < kSortNW; ww++) {
            const uint32_t cw = s_hist[ww][tid];
            s_hist[ww][tid] = uint16_t(run);
            run += cw;
        }
    }
    int tile_cnt = whole ? kSortTile : int(cnt - tile0);
    if constexpr (FILT) {
        tile_cnt = 0;
#pragma unroll
        for (int i = 0; i < kBins / kWave; i++) tile_cnt += int(s_wtot[i]);
    }
    __syncthreads();

    // Tile position of each item; stage the keys in digit order.
#pragma unroll
    for (int k = 0; k < kSortIPT; k++) {
        if (all || dp[k] != kNoPos) {
            const uint32_t p = (dp[k] & 0xffffu) + s_hist[w][dp[k] >> 16];
            dp[k] = p;
            reinterpret_cast<K *>(s_stage)[p] = key[k];
        }
    }
    uint64_t cur[kSortIPT];                      // the column being moved
    if (c.ncols > 0) load_column(c, 0, at, cnt, whole, cur);
    __syncthreads();

    // The keys out, and where every staged position goes (row counts are below
    // 2^30, so positions fit 32 bits).
    uint32_t gpos[kSortIPT];
    {
        const K *st = reinterpret_cast<const K *>(s_stage) + tid;
#pragma unroll
        for (int k = 0; k < kSortIPT; k++) {
            gpos[k] = 0;
            if (tile_cnt == kSortTile || tid + k * kSortNT < tile_cnt) {
                const K x = st[k * kSortNT];
                const uint32_t d = uint32_t(ord(x) >> shift) & (nbins - 1);
                gpos[k] = s_gbase[d] + uint32_t(tid + k * kSortNT);
                keys_out[gpos[k]] = x;
            }
        }
    }
    // The columns one after another through the same buffer.
    for (int p = 0; p < c.ncols; p++) {
        const int dt = c.pdt[p];
        void *out = c.pout[p];
        __syncthreads();                         // the column before is out of the buffer
        if (dt == TQP_INT64) stage_items<uint64_t>(s_stage, dp, all, cur);
        else if (dt == TQP_INT32) stage_items<uint32_t>(s_stage, dp, all, cur);
        else stage_items<uint8_t>(s_stage, dp, all, cur);
        __syncthreads();
        if (p + 1 < c.ncols) load_column(c, p + 1, at, cnt, whole, cur);
        if (dt == TQP_INT64) flush_stage<uint64_t>(s_stage, gpos, tile_cnt, out);
        else if (dt == TQP_INT32) flush_stage<uint32_t>(s_stage, gpos, tile_cnt, out);
        else flush_stage<uint8_t>(s_stage, gpos, tile_cnt, out);
    }
    }
}

// A whole sort of at most one tile in one launch: every pass in LDS, over keys and
// local positions, the columns then read through the positions.  Small sorts are
// bound by their launches, two per pass of about 4 us each, so this is taken
// whenever the capacity is one tile.  Row ids out, a captured sort in us, one
// launch per pass with its histograms / this one:
//   keys                  100       1000       4000
//   int32, 24 bits      34/7.4     36/11      38/14
//   int64, 64 bits      82/17      88/24      96/34
template <class K, class Ord>
__global__ __launch_bounds__(kSortNT) void k_sort_tile(const K *__restrict__ keys_in, K *__restrict__ keys_out,
                                                       PassCols c, int64_t n, const int64_t *d_n, Ord ord,
                                                       int npass, int dbits) {
    __shared__ K s_key[kSortTile];
    __shared__ uint16_t s_idx[kSortTile];
    __shared__ __attribute__((aligned(8))) uint16_t s_hist[kSortNW][kBins];
    __shared__ uint32_t s_wtot[kBins / kWave];
    const uint32_t cnt = uint32_t(count_of(d_n, n));
    if (cnt == 0) return;
    const int tid = threadIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(wave_id());
    const int lane = lane_id();
    const uint32_t nbins = 1u << dbits;
    const uint32_t wave0 = w * (kWave * kSortIPT), at = wave0 + lane;
    K key[kSortIPT];
    uint32_t idx[kSortIPT];
    load_items(keys_in, at, cnt, false, key);
#pragma unroll
    for (int k = 0; k < kSortIPT; k++) idx[k] = at + k * kWave;
    for (int pass = 0; pass < npass; pass++) {
        const int shift = pass * dbits;
        reinterpret_cast<uint64_t *>(s_hist)[tid] = 0;
        __syncthreads();
        // stable rank of each item among the items of this wave with its digit
        uint32_t dp[kSortIPT];
#pragma unroll
        for (int k = 0; k < kSortIPT; k++) {
            dp[k] = kNoPos;
            if (wave0 + k * kWave >= cnt) continue;          // (the same for the wave)
            const uint32_t d = uint32_t(ord(key[k]) >> shift) & (nbins - 1);
            const bool valid = at + k * kWave < cnt;
            uint64_t peers = ballot(valid);
            for (int b = 0; b < dbits; b++) {
                const bool set = (d >> b) & 1u;
                const uint64_t bb = ballot(set);
                peers &= set ? bb : ~bb;
            }
            const uint32_t before = __popcll(peers & lanemask_lt());
            uint16_t *h = &s_hist[w][d];
            const uint32_t old = *h;
            if (valid) dp[k] = (d << 16) | (old + before);
            if (valid && before == 0) *h = uint16_t(old + __popcll(peers));
        }
        __syncthreads();
        // per digit: its start, then the start of each wave's items of it
        uint32_t local = 0;
        if (tid < kBins) {
            uint32_t tot = 0;
#pragma unroll
            for (int ww = 0; ww < kSortNW; ww++) tot += s_hist[ww][tid];
            local = wave_incl_scan(tot);
            if (lane == kWave - 1) s_wtot[w] = local;
            local -= tot;
        }
        __syncthreads();
        if (tid < kBins) {
            for (int i = 0; i < w; i++) local += s_wtot[i];
#pragma unroll
            for (int ww = 0; ww < kSortNW; ww++) {
                const uint32_t cw = s_hist[ww][tid];
                s_hist[ww][tid] = uint16_t(local);
                local += cw;
            }
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kSortIPT; k++) {
            if (dp[k] == kNoPos) continue;
            const uint32_t p = (dp[k] & 0xffffu) + s_hist[w][dp[k] >> 16];
            s_key[p] = key[k];
            s_idx[p] = uint16_t(idx[k]);
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kSortIPT; k++) {
            const uint32_t i = at + k * kWave;
            key[k] = s_key[i < cnt ? i : 0];
            idx[k] = s_idx[i < cnt ? i : 0];
        }
    }
#pragma unroll
    for (int k = 0; k < kSortIPT; k++)
        if (at + k * kWave < cnt) keys_out[at + k * kWave] = key[k];
    for (int p = 0; p < c.ncols; p++) {
        uint64_t v[kSortIPT];
        const void *src = c.pin[p];
        const int dt = c.pdt[p];
#pragma unroll
        for (int k = 0; k < kSortIPT; k++) {
            const uint32_t i = idx[k];
            if (!src) v[k] = i;
            else if (dt == TQP_INT64) v[k] = static_cast<const uint64_t *>(src)[i];
            else if (dt == TQP_INT32) v[k] = static_cast<const uint32_t *>(src)[i];
            else v[k] = static_cast<const uint8_t *>(src)[i];
        }
#pragma unroll
        for (int k = 0; k < kSortIPT; k++)
            if (at + k * kWave < cnt) store_any(c.pout[p], dt, at + k * kWave, int64_t(v[k]));
    }
}

template <class K>
__global__ __launch_bounds__(256) void k_copy_sorted(const K *__restrict__ keys_in, K *__restrict__ keys_out,
                                                     PassCols c, int64_t n, const int64_t *d_n) {
    const int64_t cnt = count_of(d_n, n);
    for (int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; i < cnt;
         i += int64_t(gridDim.x) * blockDim.x) {
        keys_out[i] = keys_in[i];
        for (int p = 0; p < c.ncols; p++)
            store_any(c.pout[p], c.pdt[p], i, c.pin[p] ? load_any(c.pin[p], c.pdt[p], i) : i);
    }
}


// Ordinal of a key for the plain sort: its offset from the smallest key.
template <class K> struct KeyOrd {
    K key_min;
    __device__ __forceinline__ uint64_t operator()(K k) const {
        using U = typename KeyTraits<K>::U;
        return uint64_t(U(U(k) - U(key_min)));
    }
};

struct SortCols {
    const int32_t *rows_in;
    int32_t *rows_out;
    const void *pin[kMaxSortPay];
    void *pout[kMaxSortPay];
    int32_t pdt[kMaxSortPay];
    int32_t npay;
};

inline int npass_for(int key_bits) { return (key_bits + kRadixBits - 1) / kRadixBits; }
// Equal digit widths: the fewest bits per digit that keep npass_for's count.
inline int digit_bits_for(int key_bits) {
    const int np = npass_for(key_bits);
    return np ? (key_bits + np - 1) / np : 0;
}

// Workspace of run_radix: ping-pong buffers (when more than one pass), the
// counts of every tile and group, and the keep bits of a filtered sort.
inline size_t radix_ws_bytes(int64_t n, int key_size, int npass, int pay_bytes) {
    const int64_t ntiles = n > 0 ? ceil_div(n, kSortTile) : 1;
    Carver c(nullptr);
    if (npass > 1) {
        c.take<char>(size_t(n) * key_size);
        c.take<int32_t>(size_t(n));
        for (int b = 0; b < pay_bytes; b++) c.take<char>(size_t(n));
    }
    c.take<uint32_t>(size_t(ntiles + max_tile_groups(ntiles) + 1) * kBins);
    c.take<uint64_t>(size_t(ceil_div(n > 0 ? n : 1, 64)));     // keep bits of a filtered sort
    return c.bytes();
}

// Sorts by the low `bits` bits of the ordinal: npass_for(bits) stable passes
// over equal-width digits (least significant first) from key_in into key_out
// (they must not overlap), with the columns of sc moving along.  bits == 0
// copies.  With pred (then bits >= 1 and d_n null): only the items the
// predicates keep are sorted -- the first pass counts only them, drops the
// others and writes their number to *d_kept, and the later passes run over
// *d_kept items.
template <class K, class Ord>
int run_radix(const K *key_in, int64_t n, const int64_t *d_n, int bits, Ord ord, K *key_out,
              const SortCols &sc, void *ws, hipStream_t s, const RowTests *pred = nullptr,
              int64_t *d_kept = nullptr) {
    if (pred && (bits < 1 || d_n || !d_kept))
        return set_error(TQP_EINVAL, "radix: a filtered sort needs key bits and a kept counter");
    const int npass = npass_for(bits);
    const int dbits = digit_bits_for(bits);
    const int64_t ntiles = ceil_div(n > 0 ? n : 1, kSortTile);
    // every XCD's tiles have their workgroups
    const int64_t turns = ceil_div(ntiles, int64_t(kXcds) * kTileGroup) * kXcds * kTileGroup;
    PassCols pc = {};
    for (int p = 0; p < sc.npay; p++) {
        pc.pin[p] = sc.pin[p];
        pc.pout[p] = sc.pout[p];
        pc.pdt[p] = sc.pdt[p];
    }
    pc.ncols = sc.npay;
    if (sc.rows_out) {
        pc.pin[pc.ncols] = sc.rows_in;
        pc.pout[pc.ncols] = sc.rows_out;
        pc.pdt[pc.ncols] = TQP_INT32;
        pc.ncols++;
    }
    if (npass == 0) {
        const unsigned g = unsigned(ntiles > 4096 ? 4096 : ntiles);
        TQP_LAUNCH("copy_sorted", k_copy_sorted<K>, dim3(g), dim3(256), 0, s, key_in, key_out, pc, n, d_n);
        return check_launch("sort copy");
    }
    if (!pred && n <= kSortTile) {
        TQP_LAUNCH("sort_tile", (k_sort_tile<K, Ord>), dim3(1), dim3(kSortNT), 0, s, key_in, key_out, pc, n, d_n,
                   ord, npass, dbits);
        return check_launch("sort of one tile");
    }
    Carver cv(ws);
    K *tmp_keys = nullptr;
    int32_t *tmp_rows = nullptr;
    void *tmp_col[kMaxPassCols] = {};
    if (npass > 1) {
        tmp_keys = reinterpret_cast<K *>(cv.take<char>(size_t(n) * sizeof(K)));
        tmp_rows = cv.take<int32_t>(size_t(n));
        for (int p = 0; p < sc.npay; p++) tmp_col[p] = cv.take<char>(size_t(n) * dtype_size(sc.pdt[p]));
        if (sc.rows_out) tmp_col[sc.npay] = tmp_rows;
    }
    uint32_t *counts = cv.take<uint32_t>(size_t(ntiles + max_tile_groups(ntiles) + 1) * kBins);
    uint32_t *csum = counts + size_t(ntiles) * kBins;
    uint32_t *dtot = csum + size_t(max_tile_groups(ntiles)) * kBins;
    uint64_t *keep_bits = cv.take<uint64_t>(size_t(ceil_div(n > 0 ? n : 1, 64)));
    int rc;
    const K *src_k = key_in;
    PassCols cur = pc;
    const int64_t *pass_n = pred ? d_kept : d_n;   // item count of the passes after a filtered one
    for (int p = 0; p < npass; p++) {
        const bool to_out = ((npass - 1 - p) % 2) == 0;
        K *dk = to_out ? key_out : tmp_keys;
        PassCols x = cur;
        for (int q = 0; q < pc.ncols; q++) x.pout[q] = to_out ? pc.pout[q] : tmp_col[q];
        const int shift = p * dbits;
        const bool filt = pred && p == 0;
        const int64_t *cn = filt ? nullptr : pass_n;
        const unsigned grid_count = block_grid(max_tile_groups(ntiles), cn);
#define TQP_COUNT(ND, T, VEC, KEEP)                                                                  \
        TQP_LAUNCH("radix_count", (k_radix_count<K, Ord, ND>), dim3(grid_count), dim3(kCountNT), 0, s, src_k, n, \
                   cn, ord, shift, dbits, counts, csum, T, VEC, KEEP)
        if (filt) {
            int vec = 1;
            for (int q = 0; q < pred->ncol; q++)
                if (reinterpret_cast<uintptr_t>(pred->col[q]) % 16 != 0) vec = 0;
            uint8_t *kb = reinterpret_cast<uint8_t *>(keep_bits);
            if (pred->ncol <= 1) TQP_COUNT(1, *pred, vec, kb);
            else TQP_COUNT(kMaxSortPred, *pred, vec, kb);
        } else {
            TQP_COUNT(0, RowTests{}, 0, nullptr);
        }
#undef TQP_COUNT
        if ((rc = check_launch("radix tile counts"))) return rc;
        if (ntiles > kDirectTiles) {
            TQP_LAUNCH("radix_scan", k_radix_scan, dim3(unsigned(ceil_div(int64_t(1) << dbits, kScanDigits))),
                       dim3(kScanNT), 0, s, csum, dtot, n, cn);
            if ((rc = check_launch("radix tile scan"))) return rc;
        }
#define TQP_PASS(FILT)                                                                         \
        TQP_LAUNCH("onesweep", (k_onesweep<K, Ord, FILT>), dim3(grid_pass), dim3(kSortNT), 0, s, src_k, dk, \
                   x, n, cn, ord, shift, dbits, counts, csum, dtot, keep_bits, d_kept)
        // a workgroup per tile of the capacity; at most eight per compute unit and unit of the
        // knob, each looping, when the actual count is on the device and may be far smaller: a
        // workgroup without rows still costs its launch.  us at two units / one, capacity 30M,
        // int32 keys of 20 bits (and with 9 bytes of payload): 3000 rows 50/39 (51/46), 3M 92/80
        // (115/104), 15M 243/243 (438/438), 30M 508/499 (908/948).  From 2^25 rows of
        // capacity on always at least two units: the tiles that the longer loops leave uneven
        // weigh more there (256 queries of 633M rows in all, half of them kept: 23.8/24.6 ms).
        const int units = tune(kTuneSortPerCu) < 2 && n >= kSortLargeRows ? 2 : tune(kTuneSortPerCu);
        const int64_t most = int64_t(8) * kComputeUnits * units;
        const unsigned grid_pass = unsigned(cn && turns > most ? most : turns);
        if (filt) TQP_PASS(true);
        else TQP_PASS(false);
#undef TQP_PASS
        rc = check_launch("radix pass");
        if (rc) return rc;
        src_k = dk;
        for (int q = 0; q < pc.ncols; q++) cur.pin[q] = x.pout[q];
    }
    return TQP_OK;
}

}  // namespace tqp
