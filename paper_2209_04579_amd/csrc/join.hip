// Sort-merge inner equi-join over two ascending key columns.
//
// Pairs.  In the canonical order (key, i, j) the pairs of one left row are
// consecutive and left rows follow each other, so the pairs of a tile of left
// rows are one run of the output.  A first kernel finds each tile's window of
// right rows and counts its pairs; a second one takes the tiles again, starts at
// the sum of the counts before its tile, finds every left row's right rows in the
// window (staged in LDS) and writes the pairs.  A tile with very many pairs is
// left to a third kernel, which spreads its pairs over the chip.
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
constexpr int kJoinTile = kJoinNT * kJoinIPT;
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

template <class K>
__device__ __forceinline__ void load_keys16(const K *p, int64_t row0, int64_t cnt, K (&v)[16]) {
    if (row0 + 16 <= cnt) {
        if (sizeof(K) == 4) {
            const int4 *q = reinterpret_cast<const int4 *>(p + row0);
#pragma unroll
            for (int k = 0; k < 4; k++) {
                int4 x = q[k];
                v[4 * k + 0] = K(x.x);
                v[4 * k + 1] = K(x.y);
                v[4 * k + 2] = K(x.z);
                v[4 * k + 3] = K(x.w);
            }
        } else {
            const longlong2 *q = reinterpret_cast<const longlong2 *>(p + row0);
#pragma unroll
            for (int k = 0; k < 8; k++) {
                longlong2 x = q[k];
                v[2 * k + 0] = K(x.x);
                v[2 * k + 1] = K(x.y);
            }
        }
    } else {
#pragma unroll
        for (int r = 0; r < 16; r++) v[r] = row0 + r < cnt ? p[row0 + r] : K(0);
    }
}

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

struct MatchArgs {
    const void *uL;
    const int32_t *sL;
    const int64_t *d_nuL;
    const int64_t *d_nl;     // left row count (device), or null => nl
    int64_t nl;
    const void *uR;
    const int32_t *sR;
    const int64_t *d_nuR;
    const int64_t *d_nr;
    int64_t nr;
    int64_t *rkey, *rls, *rlc, *rrs, *rrc;   // ranges (workspace), capacity min(nl, nr)
    int64_t *off;                            // first pair of each range
    int64_t *ukey, *uls, *ulc, *urs, *urc;   // optional user copies
    int64_t ucap;
    int64_t *d_nranges_ws;
    int64_t *d_nranges_user;
    int64_t *d_count;
    int64_t *tile_first;     // optional: range holding the first pair of each output tile
    int64_t ntiles_out;
    const int64_t *bounds;   // per match tile: its window [bounds[2t], bounds[2t + 1]) of right runs
    uint32_t *ticket;
    uint64_t *status_m;
    uint64_t *status_p;
};

// The right runs a match tile can meet lie in [lower_bound of its first left
// key, upper_bound of its last): one thread per tile, all tiles at once, so no
// tile waits on a search over the whole right side.
template <class K>
__global__ __launch_bounds__(256) void k_match_bounds(const K *__restrict__ uL,
                                                      const int64_t *d_nuL, const K *__restrict__ uR,
                                                      const int64_t *d_nuR, int64_t tile_runs,
                                                      int64_t cap_tiles, int64_t *bounds) {
    const int64_t nuL = *d_nuL, nuR = *d_nuR;
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
        bounds[2 * t] = wl;
        bounds[2 * t + 1] = lo;
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

// Each thread takes IPT consecutive left runs and finds each one's key
// among the tile's right window (staged in LDS when it fits) by galloping
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
    const int64_t nuL = count_of(a.d_nuL, a.nl);
    const int64_t nuR = count_of(a.d_nuR, a.nr);
    const int64_t nl = count_of(a.d_nl, a.nl);
    const int64_t nr = count_of(a.d_nr, a.nr);
    const int64_t ntiles = ceil_div(nuL, kTileRuns);
    const K *uL = static_cast<const K *>(a.uL);
    const K *uR = static_cast<const K *>(a.uR);
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
    for (int r = 0; r <= IPT; r++) st[r] = u0 + r < nuL ? a.sL[u0 + r] : int32_t(nl);
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
                const int64_t rs = a.sR[g];
                const int64_t rc = (g + 1 < nuR ? int64_t(a.sR[g + 1]) : nr) - rs;
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
        const int64_t rs = a.sR[g];
        const int64_t rc = (g + 1 < nuR ? int64_t(a.sR[g + 1]) : nr) - rs;
        const int64_t ls = st[r], lc = int64_t(st[r + 1]) - ls;
        if (a.rkey) {
            a.rkey[q] = int64_t(key[r]);
            a.rls[q] = ls;
            a.rlc[q] = lc;
            a.rrs[q] = rs;
            a.rrc[q] = rc;
            a.off[q] = o;
        }
        if (a.ukey && q < a.ucap) {
            a.ukey[q] = int64_t(key[r]);
            a.uls[q] = ls;
            a.ulc[q] = lc;
            a.urs[q] = rs;
            a.urc[q] = rc;
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
// What bounds it: reading the left keys (twice) and writing the pairs.  The
// version before this went through the runs of both sides (run-length encoding,
// a match of the runs with two look-backs, an expansion that searched each
// output's range): 30M left rows against 2M unique right ones 365 -> 257 us,
// 500K against 10K 60 -> 24, 1.5M against 400K in runs of two 86 -> 57.  The
// searches are chains of LDS reads, so many small workgroups are kept resident.
constexpr int kPjNT = 256;
constexpr int kPjIPT = 8;
constexpr int kPjTile = kPjNT * kPjIPT;            // left rows per tile
constexpr int kPjNW = kPjNT / kWave;
constexpr int kPjWinBytes = 15360;                 // right keys of a tile's window staged in LDS (five workgroups per CU)
constexpr int kPjMaxSteps = 8;
constexpr int64_t kPjDirect = 8 * kPjTile;         // pairs a tile's own workgroup writes
constexpr int64_t kPjChunk = 32768;                // pairs per step of a larger tile

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
    int64_t *tpairs;         // per tile: its pairs
    int64_t *bpairs;         // per block: its pairs
    int64_t *toff;           // first pair of each tile on the list
    int64_t direct;          // pairs up to which a tile's own workgroup writes them
    int32_t *list;           // tiles with more
    uint32_t *nlist;
};

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
template <class K>
__global__ __launch_bounds__(kPjNT) void k_pair_count(PairArgs a) {
    __shared__ K s_win[kPjWinBytes / sizeof(K)];
    __shared__ K s_last;
    __shared__ int64_t s_bound;
    __shared__ uint32_t s_end[2];                      // the last row's position and count
    __shared__ int64_t s_sum[kPjNW];
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
        if (wave_id() == 0) {
            const int64_t x = wave_bound<false>(rk, 0, nr, shfl(key[0], 0), false);
            if (lane_id() == 0) s_bound = x;
        }
        __syncthreads();
        int64_t from = s_bound, bsum = 0;
        for (int64_t t = t0; t < t1; t++) {
            const uint32_t left = uint32_t(nr - from);
            uint32_t wn = left < pj_ahead<K>() ? left : pj_ahead<K>();
            for (uint32_t i = threadIdx.x; i < wn; i += kPjNT) s_win[i] = rk[from + i];
            if (threadIdx.x == kPjNT - 1) s_last = key[kPjIPT - 1];
            K next[kPjIPT];
            uint32_t nvalid = 0;
            if (t + 1 < t1) nvalid = load_left(lk, (t + 1) * kPjTile, nl, vec, next);
            __syncthreads();
            uint32_t pos[kPjIPT], cnt[kPjIPT], after;  // after: positions holding the thread's last key
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
            if (threadIdx.x == kPjNT - 1) {
                s_end[0] = pos[kPjIPT - 1];
                s_end[1] = after;
            }
            int64_t sum = 0;
#pragma unroll
            for (int r = 0; r < kPjIPT; r++) sum += cnt[r];
            sum = wave_sum(sum);
            if (lane_id() == 0) s_sum[wave_id()] = sum;
            __syncthreads();
            if (threadIdx.x == 0) {
                int64_t x = 0;
#pragma unroll
                for (int w = 0; w < kPjNW; w++) x += s_sum[w];
                a.tpairs[t] = x;
                a.win[2 * t] = int32_t(from);
                a.win[2 * t + 1] = int32_t(from + s_end[0] + s_end[1]);
                bsum += x;
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

struct PairOut {
    int64_t base;            // the tile's first pair
    int64_t row0, wlo;
};

// Writes pairs [o0, o1) of a tile, whose rows' first pairs are s_off[]: consecutive threads take consecutive pairs, each finding
// its left row by a binary search.
template <class K, class O>
__device__ __forceinline__ void expand_tile(const PairArgs &a, const PairOut &t, const uint32_t *s_pos,
                                            const O *s_off, int64_t o0, int64_t o1) {
    const K *lk = static_cast<const K *>(a.lkey);
    for (int64_t o = o0 + threadIdx.x; o < o1; o += kPjNT) {
        if (t.base + o >= a.cap) return;
        int row = 0;                                   // the last row with s_off[row] <= o
#pragma unroll
        for (int st = kPjTile / 2; st > 0; st >>= 1) row += int64_t(s_off[row + st]) <= o ? st : 0;
        const int64_t i = t.row0 + row, j = t.wlo + s_pos[row] + (o - int64_t(s_off[row]));
        if (a.out_l) a.out_l[t.base + o] = a.lrows ? a.lrows[i] : int32_t(i);
        if (a.out_r) a.out_r[t.base + o] = a.rrows ? a.rrows[j] : int32_t(j);
        if (a.out_key) static_cast<K *>(a.out_key)[t.base + o] = lk[i];
    }
}

// Fills s_pos and s_off (the exclusive sums of the counts) for a tile.
template <class O>
__device__ __forceinline__ void tile_offsets(const uint32_t (&pos)[kPjIPT], const uint32_t (&cnt)[kPjIPT],
                                             uint32_t *s_pos, O *s_off, O *s_scan) {
    O sum = 0, tot;
#pragma unroll
    for (int r = 0; r < kPjIPT; r++) {
        s_pos[threadIdx.x * kPjIPT + r] = pos[r];
        sum += cnt[r];
    }
    O ex = block_excl_scan<kPjNT>(sum, &tot, s_scan);
#pragma unroll
    for (int r = 0; r < kPjIPT; r++) {
        s_off[threadIdx.x * kPjIPT + r] = ex;
        ex += cnt[r];
    }
    __syncthreads();
}

template <class K>
__global__ __launch_bounds__(kPjNT, 5) void k_pair_write(PairArgs a) {
    __shared__ K s_win[kPjWinBytes / sizeof(K)];
    __shared__ uint32_t s_pos[kPjTile];
    __shared__ uint32_t s_off[kPjTile];          // at most a.direct pairs here
    __shared__ uint32_t s_scan[kPjNW];
    __shared__ int64_t s_sum[kPjNW];
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
        if (lane < t1 - t0) {
            tp = a.tpairs[t0 + lane];
            tlo = a.win[2 * (t0 + lane)];
            thi = a.win[2 * (t0 + lane) + 1];
        }
        int64_t first = base;                          // the tile's first pair
        for (int64_t t = t0; t < t1; t++) {
            const int l = int(t - t0);
            const int64_t total = shfl(tp, l);
            const PairOut po = {first, t * kPjTile, shfl(tlo, l)};
            const uint32_t wn = uint32_t(shfl(thi, l) - int32_t(po.wlo));
            first += total;
            if (total == 0 || !want || po.base >= a.cap) continue;
            if (total > a.direct) {
                if (threadIdx.x == 0) {
                    a.toff[t] = po.base;
                    a.list[atomicAdd(a.nlist, 1u)] = int32_t(t);
                }
                continue;
            }
            K key[kPjIPT];
            const uint32_t valid = load_left(lk, po.row0, nl, vec, key);
            uint32_t pos[kPjIPT], cnt[kPjIPT];
            match_tile(rk, po.wlo, wn, s_win, key, valid, pos, cnt);
            bool single = true;
            uint32_t hits = 0;
#pragma unroll
            for (int r = 0; r < kPjIPT; r++) {
                single = single && cnt[r] <= 1;
                hits += cnt[r] ? 1 : 0;
            }
            if (__syncthreads_and(single)) {
                // at most one right row each: the matched rows and their right
                // rows are listed in LDS, consecutive threads write them
                uint32_t tot;
                uint32_t q = block_excl_scan<kPjNT>(hits, &tot, s_scan);
#pragma unroll
                for (int r = 0; r < kPjIPT; r++) {
                    if (cnt[r]) {
                        s_off[q] = threadIdx.x * kPjIPT + r;
                        s_pos[q++] = pos[r];
                    }
                }
                __syncthreads();
                const uint32_t lim = uint32_t(a.cap - po.base < total ? a.cap - po.base : total);
                const bool staged = wn <= kPjWinBytes / sizeof(K);
#pragma unroll 4
                for (uint32_t o = threadIdx.x; o < lim; o += kPjNT) {
                    const int64_t i = po.row0 + s_off[o], j = po.wlo + s_pos[o];
                    if (a.out_l) a.out_l[po.base + o] = a.lrows ? a.lrows[i] : int32_t(i);
                    if (a.out_r) a.out_r[po.base + o] = a.rrows ? a.rrows[j] : int32_t(j);
                    if (a.out_key)
                        static_cast<K *>(a.out_key)[po.base + o] = staged ? s_win[s_pos[o]] : rk[j];
                }
            } else {
                tile_offsets(pos, cnt, s_pos, s_off, s_scan);
                expand_tile<K>(a, po, s_pos, s_off, 0, total);
            }
            __syncthreads();                           // LDS is reused by the next tile
        }
        if (b == nblocks - 1 && threadIdx.x == 0) *a.d_count = first;
    }
}

// The tiles on the list, their pairs cut into chunks that are dealt to all the
// workgroups in turn.
template <class K>
__global__ __launch_bounds__(kPjNT) void k_pair_large(PairArgs a) {
    __shared__ K s_win[kPjWinBytes / sizeof(K)];
    __shared__ uint32_t s_pos[kPjTile];
    __shared__ int64_t s_off[kPjTile];
    __shared__ int64_t s_scan[kPjNW];
    __shared__ int64_t s_chunk[kPjNT + 1];             // first chunk of each of kPjNT list entries
    const uint32_t nlist = *a.nlist;
    if (nlist == 0) return;
    const int64_t nl = count_of(a.d_nl, a.nl);
    const K *lk = static_cast<const K *>(a.lkey), *rk = static_cast<const K *>(a.rkey);
    const bool vec = reinterpret_cast<uintptr_t>(lk) % 16 == 0;
    int64_t carry = 0;                                 // chunks of the entries before
    for (uint32_t e0 = 0; e0 < nlist; e0 += kPjNT) {
        const uint32_t e = e0 + threadIdx.x;
        const int64_t n = e < nlist ? ceil_div(a.tpairs[a.list[e]], kPjChunk) : 0;
        int64_t tot;
        const int64_t ex = block_excl_scan<kPjNT>(n, &tot, s_scan);
        s_chunk[threadIdx.x] = ex;
        if (threadIdx.x == 0) s_chunk[kPjNT] = tot;
        __syncthreads();
        // this workgroup's chunks: those with (carry + c) % gridDim.x == blockIdx.x
        int64_t c = int64_t(blockIdx.x) - carry % gridDim.x;
        if (c < 0) c += gridDim.x;
        for (; c < tot; c += gridDim.x) {
            int x = 0;                                 // the last entry with s_chunk[x] <= c
#pragma unroll
            for (int st = kPjNT / 2; st > 0; st >>= 1) x += s_chunk[x + st] <= c ? st : 0;
            const int64_t t = a.list[e0 + x];
            const int64_t o0 = (c - s_chunk[x]) * kPjChunk, total = a.tpairs[t];
            const PairOut po = {a.toff[t], t * kPjTile, a.win[2 * t]};
            if (po.base + o0 >= a.cap) continue;       // (the same for the workgroup)
            K key[kPjIPT];
            const uint32_t valid = load_left(lk, po.row0, nl, vec, key);
            uint32_t pos[kPjIPT], cnt[kPjIPT];
            match_tile(rk, po.wlo, uint32_t(a.win[2 * t + 1] - po.wlo), s_win, key, valid, pos, cnt);
            tile_offsets(pos, cnt, s_pos, s_off, s_scan);
            expand_tile<K>(a, po, s_pos, s_off, o0, o0 + kPjChunk < total ? o0 + kPjChunk : total);
            __syncthreads();
        }
        carry += tot;
        __syncthreads();
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
    int64_t *tpairs, *bpairs, *toff;
    int32_t *list;
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
        L.toff = c.take<int64_t>(nt);
        L.list = c.take<int32_t>(nt);
        L.nlist = c.take<uint32_t>(1);
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
        // A tile has at most `most` pairs, and with a capacity of kPjDirect none of them
        // writes more than that: then every tile is written at once and the third
        // launch (4 us of a 10,000-row query's 66) is left out.
        const int64_t most = (nl < kPjTile ? nl : kPjTile) * nr;
        p.direct = cap <= kPjDirect && most <= INT32_MAX ? most : kPjDirect;
        const int64_t nt = ceil_div(nl, kPjTile);
        TQP_LAUNCH("pair_count", k_pair_count<K>, dim3(block_grid(nt, d_nl)), dim3(kPjNT), 0, s, p);
        if ((rc = check_launch("join pair counts"))) return rc;
        TQP_LAUNCH("pair_write", k_pair_write<K>, dim3(block_grid(nt, d_nl)), dim3(kPjNT), 0, s, p);
        if ((rc = check_launch("join pairs"))) return rc;
        if (!want_pairs || most <= p.direct) return TQP_OK;
        TQP_LAUNCH("pair_large", k_pair_large<K>, dim3(unsigned(kComputeUnits * 4)), dim3(kPjNT), 0, s, p);
        return check_launch("join large tiles");
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
    // The match searches the other side for each run of its first one, so that is the
    // shorter side (both give the same ranges).  50M and 12.5M keys, 31M and 8M runs:
    // 557 us the long way round, 354 this way.
    const int f = nr < nl ? 1 : 0, o = 1 - f;        // the sides as first and other: 0 left, 1 right
    const K *uk[2] = {static_cast<const K *>(L.uL), static_cast<const K *>(L.uR)};
    const int32_t *us[2] = {L.sL, L.sR};
    const int64_t *const d_len[2] = {d_nl, d_nr};
    const int64_t len[2] = {nl, nr};
    MatchArgs a = {};
    a.uL = uk[f];
    a.sL = us[f];
    a.d_nuL = &L.counters[f];
    a.d_nl = d_len[f];
    a.nl = len[f];
    a.uR = uk[o];
    a.sR = us[o];
    a.d_nuR = &L.counters[o];
    a.d_nr = d_len[o];
    a.nr = len[o];
    a.rkey = L.rng[0];
    a.rls = L.rng[f ? 3 : 1];
    a.rlc = L.rng[f ? 4 : 2];
    a.rrs = L.rng[f ? 1 : 3];
    a.rrc = L.rng[f ? 2 : 4];
    a.off = L.off;
    if (flags & TQP_JOIN_RANGES) {
        a.ukey = ranges->key;
        a.uls = f ? ranges->rstart : ranges->lstart;
        a.ulc = f ? ranges->rcnt : ranges->lcnt;
        a.urs = f ? ranges->lstart : ranges->rstart;
        a.urc = f ? ranges->lcnt : ranges->rcnt;
        a.ucap = range_cap;
        a.d_nranges_user = d_nranges;
    }
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
    const int ipt = match_ipt(len[f]);
    {
        int64_t g = ceil_div(L.ntiles_match, 256);
        if (g > 1024) g = 1024;
        TQP_LAUNCH("match_bounds", k_match_bounds<K>, dim3(unsigned(g)), dim3(256), 0, s,
                   uk[f], &L.counters[f], uk[o], &L.counters[o], int64_t(kJoinNT) * ipt, L.ntiles_match,
                   L.bounds);
        if ((rc = check_launch("join match bounds"))) return rc;
    }
    const unsigned gm = persistent_grid(ceil_div(len[f] > 0 ? len[f] : 1, int64_t(kJoinNT) * ipt),
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
