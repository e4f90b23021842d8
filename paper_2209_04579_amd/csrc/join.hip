// Sort-merge inner equi-join over two ascending key columns.
//
// Pairs.  In the canonical order (key, i, j) the pairs of one left row are
// consecutive and left rows follow each other, so the pairs of a tile of left
// rows are one run of the output.  A first kernel finds each tile's window of
// right rows and counts its pairs; a second one takes the tiles again, starts at
// the sum of the counts before its tile, finds every left row's right rows in the
// window (staged in LDS) and writes the pairs.  The pairs of a tile with many of them are
// left to a third kernel, which spreads them over the chip.
//
// Ranges (one per matched key).
//
//  1. Run-length encode each sorted side: one single-pass compaction of the
//     run heads gives (unique key, run start) and the number of runs.
//  2. Match: for each left run, find the right run with the same key
//     (binary search over the right run keys); a matched key becomes one range
//     (key, lstart, lcnt, rstart, rcnt).  Two decoupled look-backs in the same
//     kernel give each range its slot and its first output pair (the running
//     sum of lcnt * rcnt), so the pair total is known on the device.
//     It also records, for every tile of output pairs, the range holding the
//     tile's first pair.
//  3. Expand: output pairs are split into equal tiles, whatever the key skew;
//     a tile stages the pair offsets of its (at most tile-size) ranges in LDS,
//     each pair finds its range there and takes (i, j) = row-major position
//     within the range, which is the canonical (key, i, j) order.
#include "tqp_internal.hpp"

namespace tqp {

constexpr int kJoinNT = 256;
constexpr int kJoinIPT = 16;
constexpr int kExpandPer = 8;
constexpr int kExpandTile = kJoinNT * kExpandPer;   // output pairs per expand tile
// Consecutive runs of the match's first side per thread: 4 when either side is
// below 2^25 rows (each lane's ranges 32 bytes apart, so a store covers few
// cache lines when most runs match, as against a dimension), 16 when both
// sides are large (a quarter of the tiles, tickets and look-backs).  The
// tile count and the workspace are sized for the smaller tile.
constexpr int kMatchIPTSmall = 4;
constexpr int kMatchIPTLarge = 16;
constexpr int64_t kMatchLargeRows = int64_t(1) << 25;
constexpr int kMatchTile = kJoinNT * kMatchIPTSmall;
static int match_ipt(int64_t first) {
    return first >= kMatchLargeRows ? kMatchIPTLarge : kMatchIPTSmall;
}
constexpr int kMatchWindow = 4096;      // right keys staged in LDS per match tile
constexpr int kRleNT = 1024;
constexpr int kRleTile = kRleNT * kJoinIPT;

// Run heads of a sorted column -> (unique key, run start), count in *d_nu.
// Tiles of 1024 threads x 16 keys: the keys are only 4-8 bytes each, so a
// large tile keeps the per-tile ticket and look-back cost small next to the
// tile's own traffic.  A wave takes 16 rows of 64 consecutive keys, one key
// per lane and row, and compacts each row's heads by ballot, so the heads of
// a row are written by consecutive lanes to consecutive places (per-thread
// runs of 16 keys made each store touch 64 cache lines).
template <class K>
__global__ __launch_bounds__(kRleNT) void k_rle(const K *__restrict__ keys, int64_t n,
                                                const int64_t *d_n, K *__restrict__ ukey,
                                                int32_t *__restrict__ ustart, int64_t *d_nu,
                                                uint32_t *ticket, uint64_t *status) {
    __shared__ int64_t s_tile, s_prefix;
    __shared__ int32_t s_wcnt[kRleNT / kWave];
    const int64_t cnt = count_of(d_n, n);
    const int64_t ntiles = ceil_div(cnt, kRleTile);
    const int w = wave_id(), lane = lane_id();
    const uint64_t lt = lanemask_lt();
    for (;;) {
    const int64_t tile = take_tile(ticket, &s_tile);
    if (tile >= ntiles) {
        if (tile == 0 && threadIdx.x == 0) *d_nu = 0;
        break;
    }
    const int64_t wbase = tile * kRleTile + int64_t(w) * (kWave * kJoinIPT);
    K v[kJoinIPT], pv[kJoinIPT];
#pragma unroll
    for (int r = 0; r < kJoinIPT; r++) {
        const int64_t i = wbase + r * kWave + lane;
        v[r] = i < cnt ? keys[i] : K(0);
        pv[r] = i > 0 && i - 1 < cnt ? keys[i - 1] : K(0);
    }
    uint64_t hm[kJoinIPT];
    int32_t wc = 0;
#pragma unroll
    for (int r = 0; r < kJoinIPT; r++) {
        const int64_t i = wbase + r * kWave + lane;
        hm[r] = ballot(i < cnt && (i == 0 || v[r] != pv[r]));
        wc += __popcll(hm[r]);
    }
    if (lane == 0) s_wcnt[w] = wc;
    __syncthreads();
    int32_t wex = 0, total = 0;
#pragma unroll
    for (int ww = 0; ww < kRleNT / kWave; ww++) {
        const int32_t c = s_wcnt[ww];
        wex += ww < w ? c : 0;
        total += c;
    }
    if (w == 0) {
        int64_t pre = lookback_count(status, tile, total);
        if (lane == 0) s_prefix = pre;
    }
    __syncthreads();
    if (tile == ntiles - 1 && threadIdx.x == 0) *d_nu = s_prefix + total;
    int64_t q = s_prefix + wex;
#pragma unroll
    for (int r = 0; r < kJoinIPT; r++) {
        if ((hm[r] >> lane) & 1) {
            const int64_t pos = q + __popcll(hm[r] & lt);
            ukey[pos] = v[r];
            ustart[pos] = int32_t(wbase + r * kWave + lane);
        }
        q += __popcll(hm[r]);
    }
    __syncthreads();
    }
}

// Run heads of a sorted int32 column for other operators (the partition
// sort): ukey / ustart receive each run's value and first position, *d_nu
// the run count.  words: rle_words(n) zeroed-here uint64 words (ticket and
// look-back statuses).
size_t rle_words(int64_t n) { return size_t(1 + ceil_div(n > 0 ? n : 1, kRleTile)); }

int rle_i32(const int32_t *keys, int64_t n, int32_t *ukey, int32_t *ustart, int64_t *d_nu,
            uint64_t *words, hipStream_t s) {
    int rc = fill_u64(words, 0, int64_t(rle_words(n)), s);
    if (rc) return rc;
    const unsigned g = persistent_grid(ceil_div(n > 0 ? n : 1, kRleTile), tune(kTuneRlePerCu));
    TQP_LAUNCH("rle", k_rle<int32_t>, dim3(g), dim3(kRleNT), 0, s, keys, n, nullptr, ukey, ustart,
               d_nu, reinterpret_cast<uint32_t *>(words), words + 1);
    return check_launch("run-length encoding");
}

// The two sides (0 left, 1 right), the results by side.
struct MatchArgs {
    const void *uk[2];       // run keys
    const int32_t *us[2];    // run starts
    const int64_t *d_nu[2];  // runs
    const int64_t *d_n[2];   // rows (device), or null => n
    int64_t n[2];
    // ranges (workspace), capacity min(n): key, then start and count on each side
    int64_t *rkey, *rs[2], *rc[2];
    int64_t *off;                            // first pair of each range
    int64_t *ukey, *uss[2], *usc[2];         // user copies
    int64_t ucap;
    int64_t *d_nranges_ws;
    int64_t *d_nranges_user;
    int64_t *d_count;
    int64_t *tile_first;     // optional: range holding the first pair of each output tile
    int64_t ntiles_out;
    int64_t *bounds;         // per match tile: its window [bounds[2t], bounds[2t + 1]) of the other side's runs
    uint32_t *ticket;
    uint64_t *status_m;
    uint64_t *status_p;
};

// The match searches the other side for each run of its first one, so that is the side
// with fewer runs (both give the same ranges).  50M and 12.5M keys, 31M and 8M runs: 557 us the
// long way round, 354 this way; 50M keys in 1000 runs against 20M in 20M: 400 and 220 us
// with both run-length encodings.
__device__ __forceinline__ int match_first(const MatchArgs &a) { return *a.d_nu[1] < *a.d_nu[0] ? 1 : 0; }

// The other side's runs a match tile can meet lie in [lower_bound of its first
// key, upper_bound of its last): one thread per tile, all tiles at once, so no
// tile waits on a search over the whole other side.
template <class K>
__global__ __launch_bounds__(256) void k_match_bounds(MatchArgs a, int64_t tile_runs, int64_t cap_tiles) {
    const int f = match_first(a);
    const K *uL = static_cast<const K *>(a.uk[f]), *uR = static_cast<const K *>(a.uk[1 - f]);
    const int64_t nuL = *a.d_nu[f], nuR = *a.d_nu[1 - f];
    const int64_t ntiles = ceil_div(nuL, tile_runs);
    for (int64_t t = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; t < ntiles && t < cap_tiles;
         t += int64_t(gridDim.x) * blockDim.x) {
        const int64_t u0 = t * tile_runs;
        const int64_t u1 = (u0 + tile_runs < nuL ? u0 + tile_runs : nuL) - 1;
        const K k0 = uL[u0], k1 = uL[u1];
        int64_t lo = 0, hi = nuR;
        while (lo < hi) {
            const int64_t mid = (lo + hi) >> 1;
            if (uR[mid] < k0) lo = mid + 1;
            else hi = mid;
        }
        const int64_t wl = lo;
        hi = nuR;
        while (lo < hi) {
            const int64_t mid = (lo + hi) >> 1;
            if (!(k1 < uR[mid])) lo = mid + 1;
            else hi = mid;
        }
        a.bounds[2 * t] = wl;
        a.bounds[2 * t + 1] = lo;
    }
}

// Lower bound of k among wkeys[pos, wn), keys at or after pos: a gallop from
// pos, then a binary search inside the last step (a few reads when the two
// sides' keys interleave evenly).
template <class K, class P>
__device__ __forceinline__ int64_t gallop_lower(P wkeys, int64_t pos, int64_t wn, K k) {
    int64_t lo = pos, hi = pos, step = 1;
    while (hi < wn && wkeys[hi] < k) {
        lo = hi + 1;
        hi = lo + step;
        step <<= 1;
    }
    if (hi > wn) hi = wn;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (wkeys[mid] < k) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// Each thread takes IPT consecutive runs of the first side (called left here) and finds
// each one's key among the tile's right window (staged in LDS when it fits) by galloping
// from the previous key's position.  A first sweep counts the matched runs
// and their pairs; after the two look-backs, a second sweep writes the
// ranges of the matched runs from the window positions kept in registers.
template <class K, int IPT>
__global__ __launch_bounds__(kJoinNT) void k_join_match(MatchArgs a) {
    constexpr int kTileRuns = kJoinNT * IPT;
    __shared__ int64_t s_tile, s_pm, s_pp;
    __shared__ int64_t s_win[2];
    __shared__ K s_rkeys[kMatchWindow];
    __shared__ int32_t s_scan32[kJoinNT / kWave];
    __shared__ int64_t s_scan64[kJoinNT / kWave];
    const int f = match_first(a), o2 = 1 - f;
    const int64_t nuL = count_of(a.d_nu[f], a.n[f]);
    const int64_t nuR = count_of(a.d_nu[o2], a.n[o2]);
    const int64_t nl = count_of(a.d_n[f], a.n[f]);
    const int64_t nr = count_of(a.d_n[o2], a.n[o2]);
    const int64_t ntiles = ceil_div(nuL, kTileRuns);
    const K *uL = static_cast<const K *>(a.uk[f]);
    const K *uR = static_cast<const K *>(a.uk[o2]);
    const int32_t *sL = a.us[f], *sR = a.us[o2];
    int64_t *const rls = a.rs[f], *const rlc = a.rc[f], *const rrs = a.rs[o2], *const rrc = a.rc[o2];
    int64_t *const uls = a.uss[f], *const ulc = a.usc[f], *const urs = a.uss[o2], *const urc = a.usc[o2];
    for (;;) {
    const int64_t tile = take_tile(a.ticket, &s_tile);
    if (tile >= ntiles) {
        if (tile == 0 && threadIdx.x == 0) {
            *a.d_nranges_ws = 0;
            if (a.d_nranges_user) *a.d_nranges_user = 0;
            *a.d_count = 0;
        }
        break;
    }
    if (threadIdx.x < 2) s_win[threadIdx.x] = a.bounds[2 * tile + threadIdx.x];
    __syncthreads();
    const int64_t w_lo = s_win[0], w_hi = s_win[1];
    const int64_t wn = w_hi - w_lo;
    const bool in_lds = wn <= kMatchWindow;
    if (in_lds)
        for (int64_t i = threadIdx.x; i < wn; i += kJoinNT) s_rkeys[i] = uR[w_lo + i];
    // this thread's left runs: keys and starts (one more start for the counts)
    const int64_t u0 = tile * kTileRuns + int64_t(threadIdx.x) * IPT;
    K key[IPT];
    if (u0 + IPT <= nuL && reinterpret_cast<uintptr_t>(uL) % 16 == 0) {
        // u0 is a multiple of IPT, so whole 16-byte groups
        constexpr int kPer = 16 / sizeof(K);
        const int4 *q = reinterpret_cast<const int4 *>(uL + u0);
#pragma unroll
        for (int j = 0; j < IPT / kPer; j++) {
            const int4 x = q[j];
            const K *e = reinterpret_cast<const K *>(&x);
#pragma unroll
            for (int t = 0; t < kPer; t++) key[j * kPer + t] = e[t];
        }
    } else {
#pragma unroll
        for (int r = 0; r < IPT; r++) key[r] = u0 + r < nuL ? uL[u0 + r] : K(0);
    }
    int32_t st[IPT + 1];
#pragma unroll
    for (int r = 0; r <= IPT; r++) st[r] = u0 + r < nuL ? sL[u0 + r] : int32_t(nl);
    __syncthreads();
    uint32_t hit = 0;
    int32_t widx[IPT];
    int64_t pairs = 0;
    int64_t from = 0;
#pragma unroll
    for (int r = 0; r < IPT; r++) {
        widx[r] = 0;
        if (u0 + r < nuL) {
            const K k = key[r];
            const int64_t lo = in_lds ? gallop_lower(static_cast<const K *>(s_rkeys), from, wn, k)
                                      : gallop_lower(uR + w_lo, from, wn, k);
            from = lo;
            const K rk = lo < wn ? (in_lds ? s_rkeys[lo] : uR[w_lo + lo]) : k;
            if (lo < wn && rk == k) {
                hit |= 1u << r;
                widx[r] = int32_t(lo);
                const int64_t g = w_lo + lo;
                const int64_t rs = sR[g];
                const int64_t rc = (g + 1 < nuR ? int64_t(sR[g + 1]) : nr) - rs;
                pairs += int64_t(st[r + 1] - st[r]) * rc;
            }
        }
    }
    int32_t tot_m;
    int64_t tot_p;
    const int32_t ex_m = block_excl_scan<kJoinNT>(int32_t(__popc(hit)), &tot_m, s_scan32);
    const int64_t ex_p = block_excl_scan<kJoinNT>(pairs, &tot_p, s_scan64);
    if (wave_id() < 2) {                 // a wave each
        const int64_t pre = wave_id() == 0 ? lookback_count(a.status_m, tile, tot_m)
                                           : lookback_count(a.status_p, tile, tot_p);
        if (lane_id() == 0) (wave_id() == 0 ? s_pm : s_pp) = pre;
    }
    __syncthreads();
    if (tile == ntiles - 1 && threadIdx.x == 0) {
        *a.d_nranges_ws = s_pm + tot_m;
        if (a.d_nranges_user) *a.d_nranges_user = s_pm + tot_m;
        *a.d_count = s_pp + tot_p;
    }
    int64_t q = s_pm + ex_m;
    int64_t o = s_pp + ex_p;
#pragma unroll
    for (int r = 0; r < IPT; r++) {
        if (!(hit & (1u << r))) continue;
        const int64_t g = w_lo + widx[r];
        const int64_t rs = sR[g];
        const int64_t rc = (g + 1 < nuR ? int64_t(sR[g + 1]) : nr) - rs;
        const int64_t ls = st[r], lc = int64_t(st[r + 1]) - ls;
        if (a.rkey) {
            a.rkey[q] = int64_t(key[r]);
            rls[q] = ls;
            rlc[q] = lc;
            rrs[q] = rs;
            rrc[q] = rc;
            a.off[q] = o;
        }
        if (a.ukey && q < a.ucap) {
            a.ukey[q] = int64_t(key[r]);
            uls[q] = ls;
            ulc[q] = lc;
            urs[q] = rs;
            urc[q] = rc;
        }
        const int64_t p = lc * rc;
        if (a.tile_first) {
            // this range holds the first pair of every output tile starting in it
            for (int64_t t = ceil_div(o, kExpandTile); t * kExpandTile < o + p && t < a.ntiles_out; t++)
                a.tile_first[t] = q;
        }
        o += p;
        q++;
    }
    __syncthreads();
    }
}

// Output tile t (kExpandTile pairs) starts in range tile_first[t] and ends at
// most kExpandTile ranges later; those ranges' first-pair offsets are staged in
// LDS, and each output finds its range there by binary search.  Consecutive
// threads write consecutive pairs.
template <class K>
__global__ __launch_bounds__(kJoinNT) void k_join_expand(
    const int64_t *__restrict__ rkey, const int64_t *__restrict__ rls,
    const int64_t *__restrict__ rlc, const int64_t *__restrict__ rrs,
    const int64_t *__restrict__ rrc, const int64_t *__restrict__ off,
    const int64_t *__restrict__ tile_first, const int64_t *d_nranges, const int64_t *d_count,
    int64_t cap, const int32_t *__restrict__ lrows, const int32_t *__restrict__ rrows,
    int32_t *__restrict__ out_l, int32_t *__restrict__ out_r, K *__restrict__ out_key) {
    __shared__ int64_t s_off[kExpandTile + 1];
    const int64_t nranges = *d_nranges;
    const int64_t total = *d_count;
    const int64_t limit = total < cap ? total : cap;
    const int64_t ntiles = ceil_div(limit, kExpandTile);
    for (int64_t t = blockIdx.x; t < ntiles; t += gridDim.x) {
        const int64_t o_begin = t * kExpandTile;
        const int64_t o_end = o_begin + kExpandTile < limit ? o_begin + kExpandTile : limit;
        const int64_t m0 = tile_first[t];
        int64_t m1 = t + 1 < ntiles ? tile_first[t + 1] : nranges - 1;
        if (m1 > m0 + kExpandTile) m1 = m0 + kExpandTile;
        const int nm = int(m1 - m0 + 1);
        for (int i = threadIdx.x; i < nm; i += kJoinNT) s_off[i] = off[m0 + i];
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kExpandPer; k++) {
            const int64_t o = o_begin + k * kJoinNT + threadIdx.x;
            if (o < o_end) {
                int lo = 0, hi = nm;               // last local range with offset <= o
                while (hi - lo > 1) {
                    const int mid = (lo + hi) >> 1;
                    if (s_off[mid] <= o) lo = mid;
                    else hi = mid;
                }
                const int64_t m = m0 + lo;
                const uint64_t tt = uint64_t(o - s_off[lo]);
                const uint64_t rc = uint64_t(rrc[m]);
                uint64_t i, j;
                if (rc == 1) {
                    i = tt;
                    j = 0;
                } else if ((tt >> 32) == 0 && (rc >> 32) == 0) {
                    i = uint32_t(tt) / uint32_t(rc);
                    j = tt - i * rc;
                } else {
                    i = tt / rc;
                    j = tt - i * rc;
                }
                const int64_t li = rls[m] + int64_t(i), rj = rrs[m] + int64_t(j);
                if (out_l) out_l[o] = lrows ? lrows[li] : int32_t(li);
                if (out_r) out_r[o] = rrows ? rrows[rj] : int32_t(rj);
                if (out_key) out_key[o] = K(rkey[m]);
            }
        }
        __syncthreads();
    }
}

// ---- pairs ---------------------------------------------------------------------
//
// What bounds it: reading the left keys (twice) and writing the pairs.  A version of
// this through the runs of both sides (run-length encoding, a match of the runs with two
// look-backs, an expansion that searched each output's range) takes 345 us for 30M
// left rows against 2M right ones, 280 now; 20M against 1M unique ones 232 and 140; 1.5M
// against 400K in runs of two 86 and 57.  The searches are chains of LDS reads, so
// many small workgroups are kept resident.
//
// Where left rows meet many right ones, the pairs decide, not the rows: tiles with many are
// listed, and windows that cannot be staged are searched once only, with what the
// search found kept for the writing (12 bytes per left row).  us through the runs / with
// every tile's pairs found again and written by its own workgroup up to 16384 of
// them, in steps of 32768 beyond / now, int32 keys (slower than through the runs: few keys
// that are only counted, 20K x 20K rows of two keys 22/25, and 2M x 30M int64 rows of 1M keys
// counted 163/177):
//   500 x 10K, 20 right rows each 41/83/28          10K x 1M, 100 each     54/205/44
//   3M x 3M, 10 each             200/238/168        2M x 30M, 30 each      450/923/339
//   30K x 30K, 300 each          66/129/44          20K x 20K, 10K each    4330/720/500
constexpr int kPjNT = 256;
constexpr int kPjIPT = 8;
constexpr int kPjTile = kPjNT * kPjIPT;            // left rows per tile
constexpr int kPjNW = kPjNT / kWave;
constexpr int kPjWinBytes = 19456;                 // right keys of a tile's window staged in LDS (five workgroups per CU)
constexpr int kPjMaxSteps = 8;
constexpr uint32_t kPjSegments = 16;               // staged lengths of window that the count goes through one by one
constexpr int64_t kPjFewTiles = 2 * kComputeUnits; // ... unless there are fewer tiles
constexpr int kPjChunk = kPjNT * kPjIPT;           // pairs written at a time
constexpr int kPjSpread = 2 * kPjChunk;            // ... of listed tiles
constexpr uint32_t kPjRun = 32;                    // right rows per left one that a tile's own workgroup writes
constexpr int64_t kPjSmallCap = 8 * kPjChunk;      // capacity up to which it writes all of its pairs

// Pairs that a tile's own workgroup writes, a chunk after the other: where the tiles leave the
// chip idle, fewer.
__device__ __forceinline__ int64_t pj_direct(int64_t ntiles) { return (ntiles < kPjFewTiles ? 2 : 4) * kPjChunk; }

// Tiles per block for nl left rows: the widest of 8, 4, 2, 1 that still gives
// eight blocks per compute unit.  (A block's tiles share one search of the right
// side; the same rule on the device in every kernel.)
__host__ __device__ inline int pj_steps(int64_t nl) {
    int st = kPjMaxSteps;
    while (st > 1 && nl < int64_t(kPjTile) * st * 8 * kComputeUnits) st >>= 1;
    return st;
}

struct PairArgs {
    const void *lkey;
    const int64_t *d_nl;
    int64_t nl;
    const void *rkey;
    const int64_t *d_nr;
    int64_t nr;
    const int32_t *lrows, *rrows;
    int32_t *out_l, *out_r;
    void *out_key;
    int64_t cap;
    int64_t *d_count;
    int32_t *win;            // per tile: its window [win[2t], win[2t + 1]) of right rows
    int64_t *tpairs;         // per tile: its pairs, complemented if it is listed
    int64_t *bpairs;         // per block: its pairs
    // Where tiles may be listed or have windows that cannot be staged (else null): of
    // those that are or have, per left row its first pair in the tile and its first right row;
    // of the listed ones their first pair, and the list of their chunks.
    int64_t *toff;
    int64_t *roff;
    int32_t *rpos;
    int2 *list;              // tile, chunk in the tile
    uint32_t *nlist;
};
// A tile is listed if it has more than pj_direct pairs or a left row with more than kPjRun
// right rows: its pairs are then spread over the chip by a third launch.  With a capacity
// of kPjSmallCap (or as many pairs at most) no workgroup writes more than that anyway, so if
// every window can be staged, every tile is written at once and that launch (4 us of a
// 10,000-row query's 66) is left out.
static bool pj_lists(int64_t nl, int64_t nr, int64_t cap, int key_size) {
    const int64_t most = (nl < kPjTile ? nl : kPjTile) * nr;
    return nr > kPjWinBytes / key_size || (most > kPjSmallCap && cap > kPjSmallCap);
}

// Whether the windows are longer on average than can be staged.
static bool pj_long(int64_t nl, int64_t nr, int key_size) {
    const int64_t win = kPjWinBytes / key_size;
    return nr > win && nr * kPjTile > nl * win;
}

// The first position in [lo, n) whose key is not below k (not above k: UPPER),
// found by a whole wave: 64 probes per round trip, spread over [lo, n), then over
// ever narrower stretches.  NEAR: the position is likely close to lo, so the
// first stretches are short ones from lo, ever wider.
template <bool UPPER, class K>
__device__ __forceinline__ int64_t wave_bound(const K *p, int64_t lo, int64_t n, K k, bool near) {
    const int lane = lane_id();
    auto before = [&](int64_t i) { return UPPER ? !(k < p[i]) : p[i] < k; };
    int64_t at = lo, step = kWave, hi = n;
    while (near) {
        const int64_t i = at + (int64_t(lane) + 1) * step - 1;
        const bool b = i < n && before(i);
        const uint64_t m = ballot(b);                 // ones, then zeros
        const int c = __popcll(m);
        at += int64_t(c) * step;
        if (c < kWave) {
            hi = at + step - 1 < n ? at + step - 1 : n;
            break;
        }
        step *= kWave;
    }
    // the bound lies in [at, hi]
    while (at < hi) {
        const int64_t s = (hi - at + kWave - 1) / kWave;
        const int64_t i = at + (int64_t(lane) + 1) * s - 1;
        const bool b = i < hi && before(i);
        const int c = __popcll(ballot(b));
        at += int64_t(c) * s;
        const int64_t h = at + s - 1;
        hi = h < hi ? h : hi;
    }
    return at;
}

// The first position in p[0, n) that is not below k (above k: UPPER), at or after
// lo: steps of 1, 2, 4, ... from lo, then a binary search inside the last one.
template <bool UPPER, class K, class P>
__device__ __forceinline__ uint32_t gallop(P p, uint32_t lo, uint32_t n, K k) {
    uint32_t hi = lo, step = 1;
    while (hi < n && (UPPER ? !(k < p[hi]) : p[hi] < k)) {
        lo = hi + 1;
        hi = lo + step;
        step <<= 1;
    }
    if (hi > n) hi = n;
    while (lo < hi) {
        const uint32_t mid = (lo + hi) >> 1;
        if (UPPER ? !(k < p[mid]) : p[mid] < k) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// For a thread's ascending keys: the first position in p[0, n) not below each,
// and how many positions hold it.  The first key takes a binary search, each
// further one starts from the one before (most are equal to it or next to it).
// Returns how many positions hold the last key (valid or not).
template <class K, class P>
__device__ __forceinline__ uint32_t match_rows(P p, uint32_t n, const K (&key)[kPjIPT], uint32_t valid,
                                           uint32_t (&pos)[kPjIPT], uint32_t (&cnt)[kPjIPT]) {
    uint32_t at = 0, c = 0;
    for (uint32_t hi = n; at < hi;) {
        const uint32_t mid = (at + hi) >> 1;
        if (p[mid] < key[0]) at = mid + 1;
        else hi = mid;
    }
#pragma unroll
    for (int r = 0; r < kPjIPT; r++) {
        if (r == 0 || key[r] != key[r > 0 ? r - 1 : 0]) {
            if (r > 0) at = gallop<false>(p, at, n, key[r]);
            c = 0;
            if (at < n && p[at] == key[r])
                c = at + 1 < n && p[at + 1] == key[r] ? gallop<true>(p, at + 2, n, key[r]) - at : 1;
        }
        pos[r] = at;
        cnt[r] = (valid >> r) & 1 ? c : 0;
    }
    return c;
}

// A thread's rows: kPjIPT consecutive ones of the tile (past the end: the last
// row again, its valid bit clear).
template <class K>
__device__ __forceinline__ uint32_t load_left(const K *lk, int64_t tile0, int64_t nl, bool vec, K (&key)[kPjIPT]) {
    const int64_t row0 = tile0 + threadIdx.x * kPjIPT;
    if (vec && row0 + kPjIPT <= nl) {
        constexpr int kPer = 16 / sizeof(K);
        const int4 *q = reinterpret_cast<const int4 *>(lk + row0);
#pragma unroll
        for (int j = 0; j < kPjIPT / kPer; j++) {
            const int4 x = q[j];
            const K *e = reinterpret_cast<const K *>(&x);
#pragma unroll
            for (int t = 0; t < kPer; t++) key[j * kPer + t] = e[t];
        }
        return (1u << kPjIPT) - 1u;
    }
    uint32_t valid = 0;
#pragma unroll
    for (int r = 0; r < kPjIPT; r++) {
        key[r] = lk[row0 + r < nl ? row0 + r : nl - 1];
        valid |= (row0 + r < nl ? 1u : 0u) << r;
    }
    return valid;
}

// match_rows over a window p[0, n) too long to stage: every stride-th of its keys
// is staged instead (nc of them), and a key's search ends in one stretch of the
// window.  A thread's searches advance together, so a step is one round trip to
// memory for all of them, and there are log2(stride) steps.
template <class K>
__device__ __forceinline__ uint32_t match_rows_far(const K *p, uint32_t n, const K *s_win, uint32_t nc,
                                                   uint32_t stride, const K (&key)[kPjIPT], uint32_t valid,
                                                   uint32_t (&pos)[kPjIPT], uint32_t (&cnt)[kPjIPT]) {
    constexpr int R = kPjIPT;
    uint32_t len[R];                                   // the position lies in [pos, pos + len]
#pragma unroll
    for (int r = 0; r < R; r++) {
        pos[r] = 0;
        len[r] = nc;
    }
    for (uint32_t left = nc; left > 0; left >>= 1) {
#pragma unroll
        for (int r = 0; r < R; r++) {
            const uint32_t half = (len[r] + 1) >> 1;
            const bool up = len[r] > 0 && s_win[pos[r] + half - 1] < key[r];
            pos[r] += up ? half : 0;
            len[r] = up ? len[r] - half : len[r] > 0 ? half - 1 : 0;
        }
    }
#pragma unroll
    for (int r = 0; r < R; r++) {
        const bool in = pos[r] < nc;
        pos[r] *= stride;
        len[r] = in ? stride - 1 : n - pos[r];
    }
    for (uint32_t left = stride; left > 0; left >>= 1) {
#pragma unroll
        for (int r = 0; r < R; r++) {
            const uint32_t half = (len[r] + 1) >> 1;
            const bool up = len[r] > 0 && p[pos[r] + half - 1] < key[r];
            pos[r] += up ? half : 0;
            len[r] = up ? len[r] - half : len[r] > 0 ? half - 1 : 0;
        }
    }
    uint32_t c = 0;
    bool hit[R], more[R];
#pragma unroll
    for (int r = 0; r < R; r++) {
        hit[r] = pos[r] < n && p[pos[r]] == key[r];
        more[r] = hit[r] && pos[r] + 1 < n && p[pos[r] + 1] == key[r];
    }
#pragma unroll
    for (int r = 0; r < R; r++) {
        if (r == 0 || key[r] != key[r > 0 ? r - 1 : 0])
            c = more[r] ? gallop<true>(p, pos[r] + 2, n, key[r]) - pos[r] : hit[r] ? 1 : 0;
        cnt[r] = (valid >> r) & 1 ? c : 0;
    }
    return c;
}

// match_rows by binary searches for all the thread's keys, and for both ends of their
// positions, side by side: one read's latency per step instead of a chain of them, but
// more reads where the keys lie close together.
template <class K, class P>
__device__ __forceinline__ uint32_t search_rows(P p, uint32_t n, const K (&key)[kPjIPT], uint32_t valid,
                                                uint32_t (&pos)[kPjIPT], uint32_t (&cnt)[kPjIPT]) {
    uint32_t end[kPjIPT];
#pragma unroll
    for (int r = 0; r < kPjIPT; r++) pos[r] = end[r] = 0;
    for (uint32_t st = n ? 1u << (31 - __builtin_clz(n)) : 0u; st > 0; st >>= 1) {
#pragma unroll
        for (int r = 0; r < kPjIPT; r++) {
            const uint32_t a = pos[r] + st, b = end[r] + st;
            const K x = p[a <= n ? a - 1 : 0], y = p[b <= n ? b - 1 : 0];
            pos[r] = a <= n && x < key[r] ? a : pos[r];
            end[r] = b <= n && !(key[r] < y) ? b : end[r];
        }
    }
#pragma unroll
    for (int r = 0; r < kPjIPT; r++) cnt[r] = (valid >> r) & 1 ? end[r] - pos[r] : 0;
    return end[kPjIPT - 1] - pos[kPjIPT - 1];
}

// The same over a window p[0, n) too long to stage: every stride-th of its keys is staged in
// s_win instead (nc of them), and a search there ends in one stretch of the window, so
// that there are log2(stride) steps of one round trip to memory each.
template <class K>
__device__ __forceinline__ uint32_t search_rows_far(const K *p, uint32_t n, const K *s_win, uint32_t nc,
                                                    uint32_t stride, const K (&key)[kPjIPT], uint32_t valid,
                                                    uint32_t (&pos)[kPjIPT], uint32_t (&cnt)[kPjIPT]) {
    search_rows(s_win, nc, key, ~0u, pos, cnt);
    uint32_t pb[kPjIPT], end[kPjIPT], eb[kPjIPT];      // the stretches, and the positions inside
#pragma unroll
    for (int r = 0; r < kPjIPT; r++) {
        pb[r] = pos[r] * stride;
        eb[r] = (pos[r] + cnt[r]) * stride;
        pos[r] = end[r] = 0;
    }
    for (uint32_t st = 1u << (31 - __builtin_clz(stride)); st > 0; st >>= 1) {
#pragma unroll
        for (int r = 0; r < kPjIPT; r++) {
            // (a stretch has stride - 1 unstaged keys, the last one what is left of the window)
            const uint32_t a = pos[r] + st, b = end[r] + st;
            const bool ina = a < stride && pb[r] + a <= n, inb = b < stride && eb[r] + b <= n;
            const K x = p[ina ? pb[r] + a - 1 : 0], y = p[inb ? eb[r] + b - 1 : 0];
            pos[r] = ina && x < key[r] ? a : pos[r];
            end[r] = inb && !(key[r] < y) ? b : end[r];
        }
    }
#pragma unroll
    for (int r = 0; r < kPjIPT; r++) {
        pos[r] += pb[r];
        end[r] += eb[r];
        cnt[r] = (valid >> r) & 1 ? end[r] - pos[r] : 0;
    }
    return end[kPjIPT - 1] - pos[kPjIPT - 1];
}

// Stages len (at most kWin) right keys, every stride-th from p on, all loads in flight at once.
template <class K>
__device__ __forceinline__ void stage_keys(const K *p, uint32_t len, uint32_t stride, K *s_win) {
    constexpr int kPer = (kPjWinBytes / int(sizeof(K)) + kPjNT - 1) / kPjNT;
    K x[kPer];
#pragma unroll
    for (int u = 0; u < kPer; u++) {
        const uint32_t i = threadIdx.x + u * kPjNT;
        x[u] = p[int64_t(i < len ? i : len - 1) * stride];
    }
#pragma unroll
    for (int u = 0; u < kPer; u++)
        if (threadIdx.x + u * kPjNT < len) s_win[threadIdx.x + u * kPjNT] = x[u];
}

// The right rows of a tile's left rows in a window [wlo, wlo + wn) of any length, by searches:
// staged in turn, a segment at a time, or, beyond kPjSegments of them, every stride-th
// key staged.  (The second way has fewer steps in a row, but its reads of the window are
// scattered: so few tiles, which leave the chip idle, always take it.)
template <class K>
__device__ __forceinline__ uint32_t match_long(const K *rk, int64_t wlo, uint32_t wn, int64_t ntiles, K *s_win,
                                               const K (&key)[kPjIPT], uint32_t valid,
                                               uint32_t (&pos)[kPjIPT], uint32_t (&cnt)[kPjIPT]) {
    constexpr uint32_t kWin = kPjWinBytes / sizeof(K);
    if (wn > (ntiles < kPjFewTiles ? 1 : kPjSegments) * kWin) {
        const uint32_t stride = (wn + kWin - 1) / kWin, nc = wn / stride;
        __syncthreads();
        stage_keys(rk + wlo + stride - 1, nc, stride, s_win);
        __syncthreads();
        return search_rows_far(rk + wlo, wn, static_cast<const K *>(s_win), nc, stride, key, valid, pos, cnt);
    }
    uint32_t after = 0;
#pragma unroll
    for (int r = 0; r < kPjIPT; r++) pos[r] = cnt[r] = 0;
    for (uint32_t s0 = 0; s0 < wn; s0 += kWin) {
        const uint32_t len = wn - s0 < kWin ? wn - s0 : kWin;
        __syncthreads();
        stage_keys(rk + wlo + s0, len, 1, s_win);
        __syncthreads();
        if (s_win[len - 1] < key[0]) {
#pragma unroll
            for (int r = 0; r < kPjIPT; r++) pos[r] += len;
        } else if (!(key[kPjIPT - 1] < s_win[0])) {
            uint32_t p[kPjIPT], c[kPjIPT];
            after += search_rows(static_cast<const K *>(s_win), len, key, valid, p, c);
#pragma unroll
            for (int r = 0; r < kPjIPT; r++) {
                pos[r] += p[r];
                cnt[r] += c[r];
            }
        }
    }
    return after;
}

// The right rows of a tile's left rows in the window [wlo, wlo + wn), staged in
// s_win whole or in part (the caller's barrier must have freed s_win).
template <class K>
__device__ __forceinline__ uint32_t match_tile(const K *rk, int64_t wlo, uint32_t wn, K *s_win,
                                           const K (&key)[kPjIPT], uint32_t valid,
                                           uint32_t (&pos)[kPjIPT], uint32_t (&cnt)[kPjIPT]) {
    constexpr uint32_t kWin = kPjWinBytes / sizeof(K);
    const uint32_t stride = (wn + kWin - 1) / kWin;
    if (stride <= 1) {
        for (uint32_t i = threadIdx.x; i < wn; i += kPjNT) s_win[i] = rk[wlo + i];
        __syncthreads();
        return match_rows(static_cast<const K *>(s_win), wn, key, valid, pos, cnt);
    }
    const uint32_t nc = wn / stride;
    for (uint32_t i = threadIdx.x; i < nc; i += kPjNT) s_win[i] = rk[wlo + int64_t(i + 1) * stride - 1];
    __syncthreads();
    return match_rows_far(rk + wlo, wn, static_cast<const K *>(s_win), nc, stride, key, valid, pos, cnt);
}

// Windows and pair counts.  The tiles of a block are taken in order, the next
// one's keys loading meanwhile; a tile's window starts where the one before found
// its last key (a block's first tile searches the right side), and kPjAhead right
// keys from there are staged at once: only a tile whose keys reach further
// searches for its window's end.
template <class K> constexpr uint32_t pj_ahead() { return 4096 / sizeof(K); }
template <class K, bool LONG>
__global__ __launch_bounds__(kPjNT, LONG ? 3 : sizeof(K) == 4 ? 6 : 5) void k_pair_count(PairArgs a) {
    __shared__ K s_win[kPjWinBytes / sizeof(K)];
    __shared__ K s_last;
    __shared__ int64_t s_bound, s_upper;
    __shared__ uint32_t s_end[2];                      // the last row's position and count
    __shared__ int64_t s_sum[kPjNW];
    __shared__ uint32_t s_long[kPjNW];                 // whether a row has more than kPjRun right rows
    const int64_t nl = count_of(a.d_nl, a.nl), nr = count_of(a.d_nr, a.nr);
    const K *lk = static_cast<const K *>(a.lkey), *rk = static_cast<const K *>(a.rkey);
    const bool vec = reinterpret_cast<uintptr_t>(lk) % 16 == 0;
    const int steps = pj_steps(nl);
    const int64_t ntiles = ceil_div(nl, kPjTile), nblocks = ceil_div(ntiles, steps);
    if (blockIdx.x == 0 && threadIdx.x == 0) *a.nlist = 0;
    for (int64_t b = blockIdx.x; b < nblocks; b += gridDim.x) {
        const int64_t t0 = b * steps, t1 = t0 + steps < ntiles ? t0 + steps : ntiles;
        K key[kPjIPT];
        uint32_t valid = load_left(lk, t0 * kPjTile, nl, vec, key);
        if constexpr (LONG) {
            if (threadIdx.x == kPjNT - 1) s_last = key[kPjIPT - 1];
            __syncthreads();
        }
        if (wave_id() == 0) {
            const int64_t x = wave_bound<false>(rk, 0, nr, shfl(key[0], 0), false);
            if (lane_id() == 0) s_bound = x;
        } else if (LONG && wave_id() == 1) {
            const int64_t x = wave_bound<true>(rk, 0, nr, s_last, false);
            if (lane_id() == 0) s_upper = x;
        }
        __syncthreads();
        int64_t from = s_bound, bsum = 0;
        for (int64_t t = t0; t < t1; t++) {
            K next[kPjIPT];
            uint32_t nvalid = 0;
            uint32_t pos[kPjIPT], cnt[kPjIPT], after;  // after: positions holding the thread's last key
            if constexpr (LONG) {
                if (t > t0) {
                    if (threadIdx.x == kPjNT - 1) s_last = key[kPjIPT - 1];
                    __syncthreads();
                    if (wave_id() == 0) {
                        const int64_t x = wave_bound<true>(rk, from, nr, s_last, true);
                        if (lane_id() == 0) s_upper = x;
                    }
                    __syncthreads();
                }
                after = match_long(rk, from, uint32_t(s_upper - from), ntiles, s_win, key, valid, pos, cnt);
                if (t + 1 < t1) nvalid = load_left(lk, (t + 1) * kPjTile, nl, vec, next);
            } else {
                const uint32_t left = uint32_t(nr - from);
                uint32_t wn = left < pj_ahead<K>() ? left : pj_ahead<K>();
                for (uint32_t i = threadIdx.x; i < wn; i += kPjNT) s_win[i] = rk[from + i];
                if (threadIdx.x == kPjNT - 1) s_last = key[kPjIPT - 1];
                if (t + 1 < t1) nvalid = load_left(lk, (t + 1) * kPjTile, nl, vec, next);
                __syncthreads();
                if (wn == left || s_last < s_win[wn - 1]) {
                    after = match_rows(static_cast<const K *>(s_win), wn, key, valid, pos, cnt);
                } else {
                    if (wave_id() == 0) {
                        const int64_t x = wave_bound<true>(rk, from + wn, nr, s_last, true);
                        if (lane_id() == 0) s_bound = x;
                    }
                    __syncthreads();
                    wn = uint32_t(s_bound - from);
                    after = match_tile(rk, from, wn, s_win, key, valid, pos, cnt);
                }
            }
            if (threadIdx.x == kPjNT - 1) {
                s_end[0] = pos[kPjIPT - 1];
                s_end[1] = after;
            }
            int64_t sum = 0;
            bool longrun = false;
#pragma unroll
            for (int r = 0; r < kPjIPT; r++) {
                sum += cnt[r];
                longrun = longrun || cnt[r] > kPjRun;
            }
            longrun = __any(longrun);
            const int64_t upto = wave_incl_scan(sum);
            if (lane_id() == kWave - 1) {
                s_sum[wave_id()] = upto;
                s_long[wave_id()] = longrun;
            }
            __syncthreads();
            int64_t ex = upto - sum, total = 0;
            const bool stored = a.roff && s_end[0] + s_end[1] > kPjWinBytes / sizeof(K);
            bool listed = false;
#pragma unroll
            for (int w = 0; w < kPjNW; w++) {
                if (w < wave_id()) ex += s_sum[w];
                total += s_sum[w];
                listed = listed || s_long[w];
            }
            listed = (listed || total > pj_direct(ntiles)) && a.roff;
            if (threadIdx.x == 0) {
                a.tpairs[t] = listed ? ~total : total;
                a.win[2 * t] = int32_t(from);
                a.win[2 * t + 1] = int32_t(from + s_end[0] + s_end[1]);
                bsum += total;
            }
            if (listed || stored) {
                // (the arrays hold whole tiles)
                const int64_t row0 = t * kPjTile + threadIdx.x * kPjIPT;
#pragma unroll
                for (int r = 0; r < kPjIPT; r += 4) {
                    const int64_t e1 = ex + cnt[r], e2 = e1 + cnt[r + 1], e3 = e2 + cnt[r + 2];
                    const int32_t f = int32_t(from);
                    longlong2 *off = reinterpret_cast<longlong2 *>(a.roff + row0 + r);
                    off[0] = {ex, e1};
                    off[1] = {e2, e3};
                    *reinterpret_cast<int4 *>(a.rpos + row0 + r) = {f + int32_t(pos[r]), f + int32_t(pos[r + 1]),
                                                                    f + int32_t(pos[r + 2]), f + int32_t(pos[r + 3])};
                    ex = e3 + cnt[r + 3];
                }
            }
            from += s_end[0];
#pragma unroll
            for (int r = 0; r < kPjIPT; r++) key[r] = next[r];
            valid = nvalid;
        }
        if (threadIdx.x == 0) a.bpairs[b] = bsum;
        __syncthreads();
    }
}

// Inclusive maximum over the lanes of a wave (values >= 0), as wave_incl_scan_u32.
template <int Ctrl, int RowMask> __device__ __forceinline__ uint32_t dpp_max(uint32_t v) {
    const uint32_t u = uint32_t(__builtin_amdgcn_update_dpp(0, int(v), Ctrl, RowMask, 0xf, false));
    return u > v ? u : v;
}
__device__ __forceinline__ uint32_t wave_incl_max(uint32_t v) {
    v = dpp_max<0x111, 0xf>(v);
    v = dpp_max<0x112, 0xf>(v);
    v = dpp_max<0x114, 0xf>(v);
    v = dpp_max<0x118, 0xf>(v);
    v = dpp_max<0x142, 0xa>(v);
    v = dpp_max<0x143, 0xc>(v);
    return v;
}

// The left row of each pair of a chunk, in place: s_mark holds a row at the chunk's first
// pair and at the first pair of every further row, 0 elsewhere; rows ascend, so that a
// running maximum fills it.  The marks must be visible; a barrier is left to the caller.
template <int N>
__device__ __forceinline__ void fill_marks(uint16_t *s_mark, uint32_t *s_max) {
    constexpr int R = N / kPjNT;                       // pairs per thread
    static_assert(R % 8 == 0, "16-byte accesses");
    uint4 x[R / 8];
    uint32_t v[R];
#pragma unroll
    for (int q = 0; q < R / 8; q++) {
        x[q] = reinterpret_cast<const uint4 *>(s_mark)[threadIdx.x * (R / 8) + q];
        v[8 * q] = x[q].x & 0xffff; v[8 * q + 1] = x[q].x >> 16; v[8 * q + 2] = x[q].y & 0xffff; v[8 * q + 3] = x[q].y >> 16;
        v[8 * q + 4] = x[q].z & 0xffff; v[8 * q + 5] = x[q].z >> 16; v[8 * q + 6] = x[q].w & 0xffff; v[8 * q + 7] = x[q].w >> 16;
    }
#pragma unroll
    for (int k = 1; k < R; k++) v[k] = v[k] > v[k - 1] ? v[k] : v[k - 1];
    const uint32_t inc = wave_incl_max(v[R - 1]);
    if (lane_id() == kWave - 1) s_max[wave_id()] = inc;
    const uint32_t up = uint32_t(__shfl_up(int(inc), 1, kWave));
    uint32_t pre = lane_id() > 0 ? up : 0;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kPjNW; w++)
        if (w < wave_id()) pre = s_max[w] > pre ? s_max[w] : pre;
#pragma unroll
    for (int k = 0; k < R; k++) v[k] = v[k] > pre ? v[k] : pre;
#pragma unroll
    for (int q = 0; q < R / 8; q++)
        reinterpret_cast<uint4 *>(s_mark)[threadIdx.x * (R / 8) + q] =
            uint4{v[8 * q] | v[8 * q + 1] << 16, v[8 * q + 2] | v[8 * q + 3] << 16,
                  v[8 * q + 4] | v[8 * q + 5] << 16, v[8 * q + 6] | v[8 * q + 7] << 16};
}

// Pairs [o0, o0 + n) of a tile whose first pair is slot base, from the filled marks
// (rows counted from left row row0): consecutive threads take consecutive pairs.  The right
// row of pair o is s_d[its left row] + o (modulo 2^32).
template <class K, int N, int R>
__device__ __forceinline__ void write_chunk(const PairArgs &a, const uint16_t *s_mark, const uint32_t *s_d,
                                            int64_t row0, int64_t base, int64_t o0, int n) {
    const K *lk = static_cast<const K *>(a.lkey);
    const int64_t slot = base + o0;
    // (past the end: the last pair again, so that no load waits for a branch)
#pragma unroll 1
    for (int k0 = 0; k0 < N / kPjNT; k0 += R) {
        uint32_t row[R];
        int32_t j[R], left[R];
        K key[R];
#pragma unroll
        for (int k = 0; k < R; k++) {
            const int o = (k0 + k) * kPjNT + int(threadIdx.x), at = o < n ? o : n - 1;
            row[k] = s_mark[at];
            j[k] = int32_t(s_d[row[k]] + uint32_t(o0) + uint32_t(at));
            left[k] = int32_t(row0) + int32_t(row[k]);
        }
        if (a.out_key) {
#pragma unroll
            for (int k = 0; k < R; k++) key[k] = lk[row0 + row[k]];
        }
        if (a.lrows) {
#pragma unroll
            for (int k = 0; k < R; k++) left[k] = a.lrows[row0 + row[k]];
        }
        if (a.rrows) {
#pragma unroll
            for (int k = 0; k < R; k++) j[k] = a.rrows[j[k]];
        }
#pragma unroll
        for (int k = 0; k < R; k++) {
            const int o = (k0 + k) * kPjNT + int(threadIdx.x);
            if (o >= n) break;
            if (a.out_l) a.out_l[slot + o] = left[k];
            if (a.out_r) a.out_r[slot + o] = j[k];
            if (a.out_key) static_cast<K *>(a.out_key)[slot + o] = key[k];
        }
    }
}

// LIST: tiles that are listed are left out.
template <class K, bool LIST>
__global__ __launch_bounds__(kPjNT, LIST ? 5 : 3) void k_pair_write(PairArgs a) {
    __shared__ K s_win[kPjWinBytes / sizeof(K)];
    // the left and right rows of a chunk's pairs (or, of long runs, the chunk's marks)
    __shared__ uint32_t s_pos[kPjTile];
    __shared__ __attribute__((aligned(16))) uint16_t s_off[kPjTile];
    __shared__ uint32_t s_scan[kPjNW];
    __shared__ int64_t s_sum[kPjNW];
    __shared__ uint32_t s_slot;
    const int64_t nl = count_of(a.d_nl, a.nl);
    const K *lk = static_cast<const K *>(a.lkey), *rk = static_cast<const K *>(a.rkey);
    const bool vec = reinterpret_cast<uintptr_t>(lk) % 16 == 0;
    const int steps = pj_steps(nl);
    const int64_t ntiles = ceil_div(nl, kPjTile), nblocks = ceil_div(ntiles, steps);
    const bool want = a.out_l || a.out_r || a.out_key;
    const int w = wave_id(), lane = lane_id();
    if (nblocks == 0 && blockIdx.x == 0 && threadIdx.x == 0) *a.d_count = 0;
    int64_t base = 0, from = 0;                        // pairs of the blocks before `from`
    for (int64_t b = blockIdx.x; b < nblocks; b += gridDim.x) {
        int64_t part = 0;
#pragma unroll 4
        for (int64_t i = from + threadIdx.x; i < b; i += kPjNT) part += a.bpairs[i];
        part = wave_sum(part);
        __syncthreads();
        if (lane == 0) s_sum[w] = part;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kPjNW; i++) base += s_sum[i];
        from = b;
        const int64_t t0 = b * steps, t1 = t0 + steps < ntiles ? t0 + steps : ntiles;
        // the block's tiles, one per lane: pairs, window
        int64_t tp = 0;
        int32_t tlo = 0, thi = 0;
        bool listed = false;
        if (lane < t1 - t0) {
            tp = a.tpairs[t0 + lane];
            listed = tp < 0;
            if (listed) tp = ~tp;
            tlo = a.win[2 * (t0 + lane)];
            thi = a.win[2 * (t0 + lane) + 1];
        }
        if (LIST && __any(listed)) {                   // (the same for the workgroup)
            // the chunks, below the capacity, of the listed tiles go on the list
            const int64_t end = base + wave_incl_scan(tp), tbase = end - tp;
            const int64_t room = a.cap - tbase < tp ? a.cap - tbase : tp;
            const uint32_t n = listed && room > 0 ? uint32_t((room + kPjSpread - 1) / kPjSpread) : 0u;
            const uint32_t upto = wave_incl_scan(n);
            const uint32_t all = uint32_t(__builtin_amdgcn_readlane(int(upto), kWave - 1));
            if (all) {
                if (threadIdx.x == 0) s_slot = atomicAdd(a.nlist, all);
                if (w == 0 && n) a.toff[t0 + lane] = tbase;
                __syncthreads();
                const uint32_t at = s_slot;
                for (int l = 0; l < int(t1 - t0); l++) {
                    const uint32_t nt = uint32_t(__builtin_amdgcn_readlane(int(n), l));
                    const uint32_t to = at + uint32_t(__builtin_amdgcn_readlane(int(upto), l)) - nt;
                    for (uint32_t c = threadIdx.x; c < nt; c += kPjNT) a.list[to + c] = make_int2(int(t0) + l, int(c));
                }
            }
        }
        int64_t first = base;                          // the tile's first pair
        for (int64_t t = t0; t < t1; t++) {
            const int l = int(t - t0);
            const int64_t total = shfl(tp, l), tbase = first, row0 = t * kPjTile, wlo = shfl(tlo, l);
            const uint32_t wn = uint32_t(shfl(thi, l) - int32_t(wlo));
            first += total;
            if (total == 0 || !want || tbase >= a.cap) continue;
            if (LIST && shfl(int(listed), l)) continue;
            const uint32_t lim = uint32_t(a.cap - tbase < total ? a.cap - tbase : total);
            K key[kPjIPT];
            const uint32_t valid = load_left(lk, row0, nl, vec, key);
            uint32_t pos[kPjIPT], cnt[kPjIPT];
            if (LIST && wn > kPjWinBytes / sizeof(K)) {
                // the count has left the rows' positions and offsets
                const int64_t at = row0 + threadIdx.x * kPjIPT;
#pragma unroll
                for (int r = 0; r < kPjIPT; r++) pos[r] = uint32_t(a.rpos[at + r] - int32_t(wlo));
                uint32_t off = uint32_t(a.roff[at]);
#pragma unroll
                for (int r = 0; r < kPjIPT; r++) {
                    const uint32_t end = r + 1 < kPjIPT || threadIdx.x < kPjNT - 1 ? uint32_t(a.roff[at + r + 1]) : uint32_t(total);
                    cnt[r] = end - off;
                    off = end;
                }
            } else {
                for (uint32_t i = threadIdx.x; i < wn; i += kPjNT) s_win[i] = rk[wlo + i];
                __syncthreads();
                match_rows(static_cast<const K *>(s_win), wn, key, valid, pos, cnt);
            }
            uint32_t sum = 0, tot;
            bool longrun = false;
#pragma unroll
            for (int r = 0; r < kPjIPT; r++) {
                sum += cnt[r];
                longrun = longrun || cnt[r] > kPjRun;
            }
            uint32_t off = block_excl_scan<kPjNT>(sum, &tot, s_scan);
            bool marks = false;
            if constexpr (!LIST) marks = __syncthreads_or(longrun);
            if (!marks) {
                // the left and right rows of a chunk's pairs are listed in LDS,
                // consecutive threads write them
                for (uint32_t o0 = 0; o0 < lim; o0 += kPjChunk) {
                    uint32_t at = off;
#pragma unroll
                    for (int r = 0; r < kPjIPT; r++) {
                        const uint32_t end = at + cnt[r];
                        for (uint32_t q = at > o0 ? at : o0; q < end && q < o0 + kPjChunk; q++) {
                            s_off[q - o0] = uint16_t(threadIdx.x * kPjIPT + r);
                            s_pos[q - o0] = pos[r] + (q - at);
                        }
                        at = end;
                    }
                    __syncthreads();
                    const uint32_t n = lim - o0 < kPjChunk ? lim - o0 : kPjChunk;
                    const int64_t slot = tbase + o0;
                    // (one loop for each place of the keys: a choice inside makes the reads flat)
                    const auto write = [&](const auto &key_of) {
#pragma unroll 4
                        for (uint32_t o = threadIdx.x; o < n; o += kPjNT) {
                            const int64_t i = row0 + s_off[o], j = wlo + s_pos[o];
                            if (a.out_l) a.out_l[slot + o] = a.lrows ? a.lrows[i] : int32_t(i);
                            if (a.out_r) a.out_r[slot + o] = a.rrows ? a.rrows[j] : int32_t(j);
                            if (a.out_key) static_cast<K *>(a.out_key)[slot + o] = key_of(i, s_pos[o]);
                        }
                    };
                    if (LIST && wn > kPjWinBytes / sizeof(K)) write([&](int64_t i, uint32_t) { return lk[i]; });
                    else write([&](int64_t, uint32_t x) { return s_win[x]; });
                    if (o0 + kPjChunk < lim) __syncthreads();
                }
            }
            if constexpr (!LIST) if (marks) {
                // long runs: the first pair of every left row is marked, chunk by chunk
#pragma unroll
                for (int r = 0; r < kPjIPT; r++) {
                    s_pos[threadIdx.x * kPjIPT + r] = uint32_t(wlo) + pos[r] - off;
                    off += cnt[r];
                }
                off -= sum;
                for (uint32_t o0 = 0; o0 < lim; o0 += kPjChunk) {
                    reinterpret_cast<uint4 *>(s_off)[threadIdx.x] = uint4{0, 0, 0, 0};
                    __syncthreads();
                    uint32_t at = off;
#pragma unroll
                    for (int r = 0; r < kPjIPT; r++) {
                        if (cnt[r] && at + cnt[r] > o0 && at < o0 + kPjChunk)
                            s_off[at > o0 ? at - o0 : 0] = uint16_t(threadIdx.x * kPjIPT + r);
                        at += cnt[r];
                    }
                    __syncthreads();
                    fill_marks<kPjChunk>(s_off, s_scan);
                    __syncthreads();
                    write_chunk<K, kPjChunk, 4>(a, s_off, s_pos, row0, tbase, o0, int(lim - o0 < kPjChunk ? lim - o0 : kPjChunk));
                    __syncthreads();
                }
            }
            __syncthreads();                           // LDS is reused by the next tile
        }
        if (b == nblocks - 1 && threadIdx.x == 0) *a.d_count = first;
    }
}

// The chunks on the list, one per workgroup at a time: the rows that a chunk's pairs
// belong to are found in the offsets that the count has left, and filled in as above.  What
// bounds it: the round trips to memory of a chunk, one after another (the next chunk's
// entry is read ahead).
template <class K>
__global__ __launch_bounds__(kPjNT) void k_pair_spread(PairArgs a) {
    __shared__ uint32_t s_d[kPjTile];
    __shared__ __attribute__((aligned(16))) uint16_t s_mark[kPjSpread];
    __shared__ uint32_t s_max[kPjNW];
    __shared__ int32_t s_rows[2];
    const uint32_t n = *a.nlist;
    const int64_t nl = count_of(a.d_nl, a.nl);
    if (blockIdx.x >= n) return;
    int2 e = a.list[blockIdx.x];
    int64_t base = a.toff[e.x], total = ~a.tpairs[e.x];
    for (uint32_t c = blockIdx.x; c < n; c += gridDim.x) {
        const int2 ne = a.list[c + gridDim.x < n ? c + gridDim.x : c];
        const int64_t row0 = int64_t(e.x) * kPjTile, o0 = int64_t(e.y) * kPjSpread;
        const int rows = int(nl - row0 < kPjTile ? nl - row0 : kPjTile);
        int64_t o1 = o0 + kPjSpread < total ? o0 + kPjSpread : total;
        if (base + o1 > a.cap) o1 = a.cap - base;
        const int64_t *off = a.roff + row0;
#pragma unroll
        for (int q = 0; q < kPjSpread / kPjChunk; q++)
            reinterpret_cast<uint4 *>(s_mark)[threadIdx.x + q * kPjNT] = uint4{0, 0, 0, 0};
        // the last row that begins at or before the first pair, and the first past the last one
        if (wave_id() == 0) {
            const int64_t x = wave_bound<true>(off, 0, rows, o0, false) - 1;
            if (lane_id() == 0) s_rows[0] = int32_t(x);
        } else if (wave_id() == 1) {
            const int64_t x = wave_bound<false>(off, 0, rows, o1, false);
            if (lane_id() == 0) s_rows[1] = int32_t(x);
        }
        const int64_t nbase = a.toff[ne.x], ntotal = ~a.tpairs[ne.x];
        __syncthreads();
        const int ra = s_rows[0], rb = s_rows[1];
        for (int r = ra + int(threadIdx.x); r < rb; r += kPjNT) {
            const int64_t at = off[r], next = r + 1 < rows ? off[r + 1] : total;
            s_d[r - ra] = uint32_t(a.rpos[row0 + r]) - uint32_t(at);
            if (next > at && next > o0) s_mark[at > o0 ? at - o0 : 0] = uint16_t(r - ra);
        }
        __syncthreads();
        fill_marks<kPjSpread>(s_mark, s_max);
        __syncthreads();
        write_chunk<K, kPjSpread, 8>(a, s_mark, s_d, row0 + ra, base, o0, int(o1 - o0));
        __syncthreads();
        e = ne;
        base = nbase;
        total = ntotal;
    }
}

struct JoinLayout {
    void *sl_key, *sr_key;
    int32_t *sl_rows, *sr_rows;
    void *sort_ws;
    size_t sort_ws_bytes;
    void *uL, *uR;
    int32_t *sL, *sR;
    int64_t *rng[5];
    int64_t *off;
    int64_t *tile_first;     // per output tile of the expand: its first range
    int64_t ntiles_out;
    int64_t *bounds;         // per match tile: its window of right runs
    int64_t ntiles_match;
    int64_t *counters;       // nuL, nuR, nranges
    uint64_t *words;         // tickets + statuses
    int64_t nwords;
    uint64_t *stL, *stR, *stM, *stP;
    // pairs without ranges
    int32_t *win;
    int64_t *tpairs, *bpairs, *toff, *roff;
    int32_t *rpos;
    int2 *list;
    uint32_t *nlist;
    size_t bytes;
};

static JoinLayout join_layout(void *ws, int64_t nl, int64_t nr, int dtype, uint32_t flags,
                              int64_t cap) {
    JoinLayout L = {};
    Carver c(ws);
    const int ks = dtype_size(dtype);
    if (!(flags & TQP_JOIN_SORTED)) {
        L.sl_key = c.take<char>(size_t(nl) * ks);
        L.sl_rows = c.take<int32_t>(size_t(nl));
        L.sr_key = c.take<char>(size_t(nr) * ks);
        L.sr_rows = c.take<int32_t>(size_t(nr));
        const int64_t nmax = nl > nr ? nl : nr;
        L.sort_ws_bytes = sort_ws_bytes(nmax, dtype, ks * 8);
        L.sort_ws = c.take<char>(L.sort_ws_bytes);
    }
    if (!(flags & TQP_JOIN_RANGES)) {
        const size_t nt = size_t(ceil_div(nl > 0 ? nl : 1, kPjTile));
        L.win = c.take<int32_t>(2 * nt);
        L.tpairs = c.take<int64_t>(nt);
        L.bpairs = c.take<int64_t>(nt);
        L.nlist = c.take<uint32_t>(1);
        if (cap > 0 && pj_lists(nl, nr, cap, ks)) {
            L.toff = c.take<int64_t>(nt);
            L.roff = c.take<int64_t>(nt * kPjTile);
            L.rpos = c.take<int32_t>(nt * kPjTile);
            L.list = c.take<int2>(size_t(cap / kPjSpread) + nt);
        }
        L.bytes = c.bytes();
        return L;
    }
    L.uL = c.take<char>(size_t(nl > 0 ? nl : 1) * ks);
    L.sL = c.take<int32_t>(size_t(nl > 0 ? nl : 1));
    L.uR = c.take<char>(size_t(nr > 0 ? nr : 1) * ks);
    L.sR = c.take<int32_t>(size_t(nr > 0 ? nr : 1));
    const int64_t nm = (nl < nr ? nl : nr) > 0 ? (nl < nr ? nl : nr) : 1;
    for (int k = 0; k < 5; k++) L.rng[k] = c.take<int64_t>(size_t(nm));
    L.off = c.take<int64_t>(size_t(nm));
    L.ntiles_out = ceil_div(cap > 0 ? cap : 1, kExpandTile);
    L.tile_first = c.take<int64_t>(size_t(L.ntiles_out));
    L.ntiles_match = ceil_div(nl > 0 ? nl : 1, kMatchTile);
    L.bounds = c.take<int64_t>(size_t(2 * L.ntiles_match));
    L.counters = c.take<int64_t>(4);
    const int64_t tl = ceil_div(nl > 0 ? nl : 1, kRleTile);
    const int64_t tr = ceil_div(nr > 0 ? nr : 1, kRleTile);
    const int64_t tm = ceil_div(nl > 0 ? nl : 1, kMatchTile);
    L.nwords = 4 + tl + tr + 2 * tm;
    L.words = c.take<uint64_t>(size_t(L.nwords));
    if (L.words) {
        L.stL = L.words + 4;
        L.stR = L.stL + tl;
        L.stM = L.stR + tr;
        L.stP = L.stM + tm;
    }
    L.bytes = c.bytes();
    return L;
}

template <class K>
static int join_typed(const tqp_col *lkey, const int32_t *lrows, const int64_t *d_nl,
                      const tqp_col *rkey, const int32_t *rrows, const int64_t *d_nr,
                      uint32_t flags, int32_t *out_l, int32_t *out_r, void *out_pair_key,
                      int64_t cap, int64_t *d_count, const tqp_ranges *ranges, int64_t range_cap,
                      int64_t *d_nranges, void *ws, hipStream_t s) {
    const int64_t nl = lkey->len, nr = rkey->len;
    const bool want_pairs = (out_l || out_r || out_pair_key) && cap > 0;
    JoinLayout L = join_layout(ws, nl, nr, lkey->dtype, flags, want_pairs ? cap : 0);
    const K *lk = static_cast<const K *>(lkey->data);
    const K *rk = static_cast<const K *>(rkey->data);
    int rc;
    if (!(flags & TQP_JOIN_SORTED)) {
        int64_t kmin[2];
        int kbits[2];
        const void *keys[2] = {lk, rk};
        const int64_t ns[2] = {nl, nr};
        const int64_t *const d_ns[2] = {d_nl, d_nr};
        rc = derive_key_ranges(keys, lkey->dtype, ns, d_ns, L.sort_ws, L.sort_ws_bytes, s, kmin,
                               kbits);
        if (rc) return rc;
        rc = sort_impl(lk, lkey->dtype, lrows, nl, d_nl, kbits[0], kmin[0], L.sl_key, L.sl_rows,
                       L.sort_ws, L.sort_ws_bytes, s);
        if (rc) return rc;
        rc = sort_impl(rk, rkey->dtype, rrows, nr, d_nr, kbits[1], kmin[1], L.sr_key, L.sr_rows,
                       L.sort_ws, L.sort_ws_bytes, s);
        if (rc) return rc;
        lk = static_cast<const K *>(L.sl_key);
        rk = static_cast<const K *>(L.sr_key);
        lrows = L.sl_rows;
        rrows = L.sr_rows;
    }
    if (!(flags & TQP_JOIN_RANGES)) {
        PairArgs p = {};
        p.lkey = lk;
        p.d_nl = d_nl;
        p.nl = nl;
        p.rkey = rk;
        p.d_nr = d_nr;
        p.nr = nr;
        p.lrows = lrows;
        p.rrows = rrows;
        p.cap = cap;
        if (want_pairs) {
            p.out_l = out_l;
            p.out_r = out_r;
            p.out_key = out_pair_key;
        }
        p.d_count = d_count;
        p.win = L.win;
        p.tpairs = L.tpairs;
        p.bpairs = L.bpairs;
        p.toff = L.toff;
        p.list = L.list;
        p.nlist = L.nlist;
        p.roff = L.roff;
        p.rpos = L.rpos;
        const int64_t nt = ceil_div(nl, kPjTile);
        if (pj_long(nl, nr, sizeof(K)))
            TQP_LAUNCH("pair_count", (k_pair_count<K, true>), dim3(block_grid(nt, d_nl)), dim3(kPjNT), 0, s, p);
        else
            TQP_LAUNCH("pair_count", (k_pair_count<K, false>), dim3(block_grid(nt, d_nl)), dim3(kPjNT), 0, s, p);
        if ((rc = check_launch("join pair counts"))) return rc;
        if (L.roff || !want_pairs)
            TQP_LAUNCH("pair_write", (k_pair_write<K, true>), dim3(block_grid(nt, d_nl)), dim3(kPjNT), 0, s, p);
        else
            TQP_LAUNCH("pair_write", (k_pair_write<K, false>), dim3(block_grid(nt, d_nl)), dim3(kPjNT), 0, s, p);
        if ((rc = check_launch("join pairs")) || !L.roff) return rc;
        TQP_LAUNCH("pair_spread", k_pair_spread<K>, dim3(unsigned(kComputeUnits * 8)), dim3(kPjNT), 0, s, p);
        return check_launch("join pairs of large tiles");
    }
    rc = fill_u64(L.words, 0, L.nwords, s);
    if (rc) return rc;
    uint32_t *tickets = reinterpret_cast<uint32_t *>(L.words);
    const unsigned gl = persistent_grid(ceil_div(nl > 0 ? nl : 1, kRleTile), tune(kTuneRlePerCu));
    const unsigned gr = persistent_grid(ceil_div(nr > 0 ? nr : 1, kRleTile), tune(kTuneRlePerCu));
    TQP_LAUNCH("rle", k_rle<K>, dim3(gl), dim3(kRleNT), 0, s, lk, nl, d_nl,
                       static_cast<K *>(L.uL), L.sL, &L.counters[0], tickets + 0, L.stL);
    if ((rc = check_launch("join rle left"))) return rc;
    TQP_LAUNCH("rle", k_rle<K>, dim3(gr), dim3(kRleNT), 0, s, rk, nr, d_nr,
                       static_cast<K *>(L.uR), L.sR, &L.counters[1], tickets + 2, L.stR);
    if ((rc = check_launch("join rle right"))) return rc;
    MatchArgs a = {};
    const void *const uk[2] = {L.uL, L.uR};
    const int32_t *const us[2] = {L.sL, L.sR};
    const int64_t *const d_n[2] = {d_nl, d_nr};
    int64_t *const uss[2] = {ranges->lstart, ranges->rstart}, *const usc[2] = {ranges->lcnt, ranges->rcnt};
    for (int k = 0; k < 2; k++) {
        a.uk[k] = uk[k];
        a.us[k] = us[k];
        a.d_nu[k] = &L.counters[k];
        a.d_n[k] = d_n[k];
        a.rs[k] = L.rng[1 + 2 * k];
        a.rc[k] = L.rng[2 + 2 * k];
        a.uss[k] = uss[k];
        a.usc[k] = usc[k];
    }
    a.n[0] = nl;
    a.n[1] = nr;
    a.rkey = L.rng[0];
    a.off = L.off;
    a.ukey = ranges->key;
    a.ucap = range_cap;
    a.d_nranges_user = d_nranges;
    a.d_nranges_ws = &L.counters[2];
    a.d_count = d_count;
    if (want_pairs) {
        a.tile_first = L.tile_first;
        a.ntiles_out = L.ntiles_out;
    }
    if (!want_pairs) a.rkey = nullptr;      // only the expand reads the workspace copy
    a.ticket = tickets + 4;
    a.status_m = L.stM;
    a.status_p = L.stP;
    a.bounds = L.bounds;
    const int64_t most = nl < nr ? nl : nr;          // runs of the first side, whichever it is
    const int ipt = match_ipt(most);
    {
        int64_t g = ceil_div(L.ntiles_match, 256);
        if (g > 1024) g = 1024;
        TQP_LAUNCH("match_bounds", k_match_bounds<K>, dim3(unsigned(g)), dim3(256), 0, s, a,
                   int64_t(kJoinNT) * ipt, L.ntiles_match);
        if ((rc = check_launch("join match bounds"))) return rc;
    }
    const unsigned gm = persistent_grid(ceil_div(most > 0 ? most : 1, int64_t(kJoinNT) * ipt),
                                        tune(kTuneMatchPerCu));
    if (ipt == kMatchIPTLarge)
        TQP_LAUNCH("join_match", (k_join_match<K, kMatchIPTLarge>), dim3(gm), dim3(kJoinNT), 0, s, a);
    else
        TQP_LAUNCH("join_match", (k_join_match<K, kMatchIPTSmall>), dim3(gm), dim3(kJoinNT), 0, s, a);
    if ((rc = check_launch("join match"))) return rc;
    if (want_pairs) {
        int64_t g = L.ntiles_out;
        if (g > 16384) g = 16384;
        TQP_LAUNCH("join_expand", k_join_expand<K>, dim3(unsigned(g)), dim3(kJoinNT), 0, s,
                   L.rng[0], L.rng[1], L.rng[2], L.rng[3], L.rng[4], L.off, L.tile_first,
                   &L.counters[2], d_count, cap, lrows, rrows, out_l, out_r,
                   static_cast<K *>(out_pair_key));
        if ((rc = check_launch("join expand"))) return rc;
    }
    return TQP_OK;
}

}  // namespace tqp

using namespace tqp;

TQP_API size_t tqp_join_workspace_bytes(int64_t nl, int64_t nr, int dtype, uint32_t flags,
                                        int64_t cap) {
    if (nl < 0 || nr < 0 || cap < 0 || (dtype != TQP_INT32 && dtype != TQP_INT64)) return 0;
    return join_layout(nullptr, nl, nr, dtype, flags, cap).bytes;
}

TQP_API int tqp_join(const tqp_col *lkey, const int32_t *lrows, const int64_t *d_nl,
                     const tqp_col *rkey, const int32_t *rrows, const int64_t *d_nr,
                     uint32_t flags, int32_t *out_l, int32_t *out_r, void *out_pair_key,
                     int64_t cap, int64_t *d_count, const tqp_ranges *ranges, int64_t range_cap,
                     int64_t *d_nranges, void *ws, size_t ws_bytes, void *stream) {
    clear_error();
    if (!lkey || !rkey || !d_count) return set_error(TQP_EINVAL, "tqp_join: null argument");
    if (lkey->dtype != rkey->dtype || (lkey->dtype != TQP_INT32 && lkey->dtype != TQP_INT64))
        return set_error(TQP_EINVAL, "tqp_join: keys must share dtype int32 or int64");
    if (flags & ~(TQP_JOIN_SORTED | TQP_JOIN_RANGES))
        return set_error(TQP_EINVAL, "tqp_join: unknown flag bits");
    const int64_t nl = lkey->len, nr = rkey->len;
    if (nl < 0 || nr < 0 || nl > (int64_t(1) << 30) - 1 || nr > (int64_t(1) << 30) - 1)
        return set_error(TQP_EINVAL, "tqp_join: sides must hold [0, 2^30 - 1] rows");
    if ((nl > 0 && !lkey->data) || (nr > 0 && !rkey->data))
        return set_error(TQP_EINVAL, "tqp_join: null key data");
    if (cap < 0) return set_error(TQP_EINVAL, "tqp_join: negative cap");
    if ((flags & TQP_JOIN_RANGES) &&
        (!ranges || !d_nranges || range_cap < 0 ||
         (range_cap > 0 && (!ranges->key || !ranges->lstart || !ranges->lcnt || !ranges->rstart ||
                            !ranges->rcnt))))
        return set_error(TQP_EINVAL, "tqp_join: ranges mode needs five arrays and d_nranges");
    const bool want_pairs = (out_l || out_r || out_pair_key) && cap > 0;
    const size_t need = tqp_join_workspace_bytes(nl, nr, lkey->dtype, flags, want_pairs ? cap : 0);
    if (!ws || ws_bytes < need)
        return set_error(TQP_ECAPACITY, "tqp_join: workspace needs %zu bytes", need);
    hipStream_t s = as_stream(stream);
    if (lkey->dtype == TQP_INT32)
        return join_typed<int32_t>(lkey, lrows, d_nl, rkey, rrows, d_nr, flags, out_l, out_r,
                                   out_pair_key, cap, d_count, ranges, range_cap, d_nranges, ws, s);
    return join_typed<int64_t>(lkey, lrows, d_nl, rkey, rrows, d_nr, flags, out_l, out_r,
                               out_pair_key, cap, d_count, ranges, range_cap, d_nranges, ws, s);
}
