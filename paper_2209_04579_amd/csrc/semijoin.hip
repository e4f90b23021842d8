// Semi-join reduction in front of a star join.
//
// An inner join of a fact row with a dimension can only produce output when
// the row's foreign key occurs among the dimension's (filtered) keys, so the
// fact rows that fail that test for any dimension can be dropped before the
// sort-merge joins without changing their result (the relational semi-join
// of the fact table with each dimension side).
//
// A dimension side is reduced to a key set: a bitmap over its key range
// (tqp_keyset_build).  Two kernels then take the fact table.  k_semi_mask streams the
// key columns and writes one keep bit per row, a kept count per block and, of a large
// table, the kept rows' keys where they are few; k_semi_write writes the kept rows out.
// Where the sets keep many rows of several columns, k_semi_direct does both in one pass.
//
// k_semi_mask: a workgroup stages the sets that belong in LDS once.  Each wave then takes
// chunks of 512 rows by itself, 8 consecutive rows per lane: the next chunk's keys are
// loaded before this one's are tested, and the only barrier is where a block's
// count is written.  The other sets are read from memory (they stay in L2) for the rows
// still alive after the LDS tests.
//
// What bounds it: the read of the key columns (4.7 TB/s with the slabs' writes
// between them, 5.5 without), and close behind it the instructions per key: so a
// position is 32-bit for int32 keys, and one past the set is moved to a zero bit
// beside it instead of tested.
//
// us, k_semi_direct's form of 512-thread workgroups for every table / now:
//   kept, of 300M rows and 3 int32 sets  1% 903/877   5% 1207/999  14% 1326/1310  22% 1433/1292
//   of 60M rows and 3 int64 sets         1% 356/347   5% 449/398   14% 473/473    22% 512/491
//   of 3M rows, sets of 1M, 100K, 25 and 1000 positions   1%       22%       60%
//     1 int32 set                                      30.3/15.6 33.8/19.7 36.4/24.0
//     3 int32 sets                                     26.6/19.3 31.6/25.6 38.5/31.9
//     3 int64 sets                                     36.5/25.9 43.7/37.9 48.7/45.9
// Slower than that form: four int64 sets of 3M to 6M rows by up to 12% where many rows are
// kept (4M rows, 14% 59.8/67.9) and of 60M rows with all kept (925/990), and tables taken
// in parts by up to 5% (300M rows, three int32 sets, 0.2% kept 988/1043).
#include <mutex>
#include <type_traits>

#include "keepbits.hpp"
#include "semirows.hpp"

namespace tqp {

constexpr int kSjNT = 256;
constexpr int kSjMaxSets = 4;
constexpr int kSjMaxPay = 4;
static_assert(kSjIPT == kFilterIPT && kSjChunk == kWave * kSjIPT, "a lane's keep bits are a byte");
// Words of key sets staged in LDS per 256 threads of workgroup (36 KiB): a
// 1024-thread workgroup, alone on its compute unit, stages up to 144 KiB.
constexpr int kSjLdsWordsPer256 = 9216;
// Every workgroup stages the sets, so a table of few rows reads a large set from L2 instead.
// us, staged / from L2, of sets of 1M, 100K, 25 and 1000 positions: one int32 set 13.7/12.6 at 1M
// rows, 15.6/19.8 at 3M; two int64 sets 17.5/15.1 at 400K, 21.2/14.8 at 1M, 27.9/20.5 at 3M; four
// 27.9/19.3 at 1M, 43.9/35.3 at 3M (at 60% kept 64.5/59.8).  A set of a few words is staged
// at once: 10K to 200K rows of three int64 sets of 100K, 30K and 10K positions, all kept, 18.0/20.0
// (all with workgroups of 1024).
static bool sj_staged(int64_t n, int nsets, int64_t words) {
    return words <= 4096 || n >= (nsets == 1 ? 64 : 128) * words;
}
// A chunk that keeps at most this many rows leaves their keys, row by row, in
// its slab of the workspace.  The columns would be read again a 128-byte line per
// kept row and set (three int32 sets, 300M rows, without slabs / with: 0.8% kept 926/882 us, 5%
// 1345/1004, 14% 1587/1317); above a quarter kept every line is used anyway, and
// columns of at most kSjCached bytes are still in the last-level cache (256 MiB).
constexpr int kSjSlab = 128;
constexpr int64_t kSjCached = 200'000'000;

struct SemiArgs {
    const void *key[kSjMaxSets];
    const uint32_t *bits[kSjMaxSets];
    int64_t lo[kSjMaxSets];
    uint64_t nbits[kSjMaxSets];
    int32_t lds_off[kSjMaxSets];     // word offset of a set staged in LDS; -1: read from memory
    int32_t lds_len[kSjMaxSets];
    uint32_t sh[kSjMaxSets];         // int32 keys: position 0 is bit sh of the first word
    int64_t n;
    int32_t lg_block;                // log2 of the chunks per block
    int32_t lg_group;                // log2 of the chunks that a workgroup takes together: at
                                     // least a block, and at least one per wave
    int64_t nchunks;                 // chunks of all blocks
    uint8_t *keep;                   // one byte per lane
    int32_t *bcnt;
    void *slab;                      // kSjSlab kept rows' keys per chunk (null: none)
    // where the device chooses (else null): 1, the single pass, or 0, the two kernels
    int32_t *pick;
    uint64_t *words;                 // the single pass's ticket, then a look-back status per tile
    int64_t nwords;
};

// The keys of a whole chunk of aligned columns, 8 consecutive rows per lane; of the first
// one where `row0` starts no whole chunk (so a.n >= kSjChunk: sj_whole_chunks).  There is
// no second way to load them here: a register that another branch had written would
// make the compiler wait for every load in flight before this one's are issued.
template <class K, int NS>
__device__ __forceinline__ void sj_load(const SemiArgs &a, int64_t row0, K (&v)[NS][kSjIPT]) {
    constexpr int V = 16 / int(sizeof(K));     // keys per 16-byte load
    row0 = sj_chunk_row(row0, a.n);
#pragma unroll
    for (int s = 0; s < NS; s++) {
        const K *p = static_cast<const K *>(a.key[s]) + row0;
#pragma unroll
        for (int k = 0; k < kSjIPT / V; k++) {
            const uint32_t q = sj_lane_key<V>(threadIdx.x % kWave, k);
            if constexpr (sizeof(K) == 4) {
                const int4 x = *reinterpret_cast<const int4 *>(p + q);
                v[s][k * V + 0] = x.x; v[s][k * V + 1] = x.y;
                v[s][k * V + 2] = x.z; v[s][k * V + 3] = x.w;
            } else {
                const longlong2 x = *reinterpret_cast<const longlong2 *>(p + q);
                v[s][k * V + 0] = x.x; v[s][k * V + 1] = x.y;
            }
        }
    }
}

// The keys of any chunk that begins inside the table; past its end, the last row's again.
template <class K, int NS>
__device__ __forceinline__ void sj_load_any(const SemiArgs &a, int64_t row0, K (&v)[NS][kSjIPT]) {
#pragma unroll
    for (int s = 0; s < NS; s++) {
        const K *p = static_cast<const K *>(a.key[s]) + row0;
#pragma unroll
        for (int r = 0; r < kSjIPT; r++) v[s][r] = p[sj_any_row(row0, a.n, lane_id(), r)];
    }
}

// The position of a key in a set that starts at lo, 2^32 - 1 if it does not fit 32
// bits.  int32 keys: modulo 2^32.
__device__ __forceinline__ uint32_t sj_pos(int32_t v, int64_t lo) { return uint32_t(v) - uint32_t(lo); }
__device__ __forceinline__ uint32_t sj_pos(int64_t v, int64_t lo) {
    const uint64_t i = uint64_t(v) - uint64_t(lo);
    return i >> 32 ? ~0u : uint32_t(i);
}

// A set in LDS: every row is tested, without a branch.  The set's words lie there in
// descending order between two zero words, so that with d = 31 - position
// (plus 32 times where word 0 lies) d >> 5 is the word, a shift by d (modulo
// 32) brings the bit to the top, and a d on either side of the set is moved to
// a zero bit: six instructions and a read per key.
template <class K, int R>
__device__ __forceinline__ uint32_t sj_test_lds(const SemiArgs &a, int s, const uint32_t *sets, const K (&v)[R]) {
    const uint32_t off = uint32_t(a.lds_off[s]), len = uint32_t(a.lds_len[s]);
    const uint32_t zero = 32 * (off + len) + 31, least = 32 * off + 31, most = zero + 1;
    uint32_t m = 0;
#pragma unroll
    for (int r = R - 1; r >= 0; r--) {
        uint32_t d = zero - sj_pos(v[r], a.lo[s]);
        d = d < least ? least : d;
        d = d > most ? most : d;
        m = __builtin_amdgcn_alignbit(m, sets[d >> 5] << (d & 31), 31);
    }
    return m;
}
// A set of less than 32 positions, its bits in a scalar register.
template <class K, int R>
__device__ __forceinline__ uint32_t sj_test_reg(const SemiArgs &a, int s, uint32_t bits, const K (&v)[R]) {
    uint32_t m = 0;
#pragma unroll
    for (int r = R - 1; r >= 0; r--) {
        uint32_t d = ~sj_pos(v[r], a.lo[s]);
        d = d > ~31u ? d : ~31u;
        m = __builtin_amdgcn_alignbit(m, bits << (d & 31), 31);
    }
    return m;
}

// A set in memory: only the rows still alive read their word.
template <class K, int R>
__device__ __forceinline__ uint32_t sj_test_mem(const SemiArgs &a, int s, const K (&v)[R], uint32_t alive) {
    using Pos = std::conditional_t<sizeof(K) == 4, uint32_t, uint64_t>;
    if (a.nbits[s] == 0) return 0;
    const uint32_t *w = a.bits[s];
    const Pos lo = Pos(a.lo[s]), last = Pos(a.nbits[s] - 1);
    const uint32_t sh = sizeof(K) == 4 ? a.sh[s] : 0;
    uint32_t word[R];
#pragma unroll
    for (int r = 0; r < R; r++) {
        const Pos idx = Pos(v[r]) - lo;
        const bool in = ((alive >> r) & 1u) && idx <= last;
        word[r] = in ? w[(idx >> 5) + ((uint32_t(idx & 31) + sh) >> 5)] : 0u;
    }
    uint32_t m = 0;
#pragma unroll
    for (int r = 0; r < R; r++)
        m |= ((word[r] >> ((uint32_t(Pos(v[r]) - lo) + sh) & 31)) & 1u) << r;
    return m;
}

// Copies the sets that belong in LDS there (see sj_test_lds), those of less than 32
// positions also to small.  COUNT: returns the product of the sets' shares of members, the share of
// rows kept if keys were spread evenly; 0 if a set is not in LDS.
template <int NS, bool COUNT>
__device__ __forceinline__ float sj_stage(const SemiArgs &a, uint32_t *s_sets, uint32_t (&small)[NS]) {
    __shared__ uint32_t s_pop[NS];
    if constexpr (COUNT) {
        if (threadIdx.x < NS) s_pop[threadIdx.x] = 0;
        __syncthreads();
    }
    for (int s = 0; s < NS; s++) {
        if (a.lds_off[s] < 0) continue;
        uint32_t *dst = s_sets + a.lds_off[s];
        const int len = a.lds_len[s];
        uint32_t pop = 0;
        for (int i = threadIdx.x; i <= len + 1; i += blockDim.x) {
            uint32_t x = i > 0 && i <= len ? a.bits[s][len - i] : 0u;
            if (i == 1 && (a.nbits[s] & 31)) x &= (1u << (a.nbits[s] & 31)) - 1u;
            dst[i] = x;
            pop += __popc(x);
        }
        if constexpr (COUNT) {
            pop = wave_sum(pop);
            if (lane_id() == 0 && pop) atomicAdd(&s_pop[s], pop);
        }
    }
    __syncthreads();
    float share = 1.0f;
#pragma unroll
    for (int s = 0; s < NS; s++) {
        small[s] = a.lds_off[s] >= 0 && a.nbits[s] < 32 ? __builtin_amdgcn_readfirstlane(s_sets[a.lds_off[s] + 1]) : 0u;
        if constexpr (COUNT) share *= a.lds_off[s] >= 0 ? float(s_pop[s]) / float(a.nbits[s]) : 0.0f;
    }
    return share;
}

// The rows of R keys that are in every set, of those in alive.
template <class K, int NS, int R>
__device__ __forceinline__ uint32_t sj_test(const SemiArgs &a, const uint32_t *s_sets, const uint32_t (&small)[NS],
                                            const K (&v)[NS][R], uint32_t alive) {
#pragma unroll
    for (int s = 0; s < NS; s++) {
        if (a.lds_off[s] < 0) continue;
        alive &= a.nbits[s] < 32 ? sj_test_reg(a, s, small[s], v[s]) : sj_test_lds(a, s, s_sets, v[s]);
    }
#pragma unroll
    for (int s = 0; s < NS; s++)
        if (a.lds_off[s] < 0) alive &= sj_test_mem(a, s, v[s], alive);
    return alive;
}

// The two kernels read the kept rows' keys twice, the single pass of k_semi_direct once; but
// there each tile waits for the counts of those before it.  So the single pass is taken
// where many rows are kept: where the sets' shares of members multiply to sj_dense, which is
// the share kept if keys are spread evenly, known before a key is read, and only for columns
// wide and long enough (above kSjCached) that the second read counts.  us, two kernels /
// single pass, by share kept:
//   rows                1%        5%       14%       22%       30%       50%       100%
//   60M  2 int64     254/345   279/355   340/366   383/382   489/393   545/437   664/540
//        3 int64     347/438   404/452   479/473   552/494   681/513   764/565   920/736
//        4 int64     446/532   537/572   668/587   729/621   896/639   990/711  1190/981
//   300M 2 int32     615/856   691/874   888/907  1041/978 1181/1060 1332/1274 1837/1833
//        3 int32    883/1081  996/1139 1309/1197 1549/1301 1730/1407 1943/1721 2448/2495
//        4 int32   1146/1342 1301/1417 1705/1488 2066/1610 2267/1764 2529/2145 3120/3165
//   8M   4 int64     78/93 (1%), 115/106 (14%), 132/119 (30%), 167/143 (60%)
// The choice costs 2-4 us, and the single pass 5-7 more where it follows (the sets are staged
// twice): at 8M rows of 3 int64 sets, 192 MB, it would be 88/95 at 30%, 110/113 at 60%.
// Two int32 sets gain too little.
__host__ __device__ constexpr float sj_dense(int nsets) { return nsets == 2 ? 0.22f : 0.12f; }
__host__ __device__ constexpr bool sj_picks(int key_bytes, int nsets) { return nsets >= (key_bytes == 8 ? 2 : 3); }

// VEC: every key column is 16-byte aligned, and there is a whole chunk of rows at least.
template <class K, int NS, bool VEC>
__global__ __launch_bounds__(4 * kSjNT) void k_semi_mask(SemiArgs a) {
    // two chunks' keys in registers, where they take at most half of them
    constexpr bool kAhead = VEC && NS * int(sizeof(K)) * kSjIPT * 2 <= 64 * 4;
    extern __shared__ uint32_t s_sets[];
    __shared__ uint32_t s_cnt[2][4 * kSjNT / kWave];         // by turn: one may still be read
    const int nw = blockDim.x / kWave;
    const int wave = __builtin_amdgcn_readfirstlane(wave_id());
    if (threadIdx.x < 2 * 4 * kSjNT / kWave) (&s_cnt[0][0])[threadIdx.x] = 0;
    uint32_t small[NS];
    const float share = sj_stage<NS, sj_picks(sizeof(K), NS)>(a, s_sets, small);
    if (sj_picks(sizeof(K), NS) && a.pick) {                       // (the same for every workgroup)
        const bool dense = share >= sj_dense(NS);
        if (blockIdx.x == 0 && threadIdx.x == 0) *a.pick = dense ? 1 : 0;
        if (dense) {
            for (int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; i < a.nwords; i += int64_t(gridDim.x) * blockDim.x)
                a.words[i] = 0;
            return;
        }
    }

    const int ngroups = int((a.nchunks + (1 << a.lg_group) - 1) >> a.lg_group);
    const int last_j = (1 << a.lg_group) / nw - 1;           // a wave takes every nw-th chunk of a group
    int g = blockIdx.x, j = 0, turn = 0;
    K va[NS][kSjIPT], vb[NS][kSjIPT];
    if constexpr (VEC) sj_load<K, NS>(a, ((int64_t(g) << a.lg_group) + wave) * kSjChunk, va);
    auto step = [&](K (&v)[NS][kSjIPT], K (&next)[NS][kSjIPT]) {
        const int in_group = j * nw + wave;
        const int64_t chunk = (int64_t(g) << a.lg_group) + in_group;
        const int64_t row0 = chunk * kSjChunk;
        const bool ends = j == last_j;
        const int g0 = g;
        j = ends ? 0 : j + 1;
        if (ends) g += gridDim.x;
        const int64_t next_row = ((int64_t(g) << a.lg_group) + j * nw + wave) * kSjChunk;
        // v has arrived once only the loads of `next` are still out.  Waiting for it here, on
        // every path, lets its registers be written again without another wait.
        if constexpr (kAhead) {
            sj_load<K, NS>(a, next_row, next);
            __builtin_amdgcn_s_waitcnt(0x0f70 | NS * kSjIPT * int(sizeof(K)) / 16);
        } else if constexpr (VEC) {
            __builtin_amdgcn_s_waitcnt(0x0f70);
        }
        uint32_t alive = 0xff;
        if (!VEC || row0 + kSjChunk > a.n) {
            const int64_t left = a.n - row0 - lane_id() * kSjIPT;    // rows from this lane's on
            alive = left >= kSjIPT ? 0xffu : left > 0 ? (1u << int(left)) - 1u : 0u;
            if (row0 < a.n) {
                sj_load_any<K, NS>(a, row0, v);
                __builtin_amdgcn_s_waitcnt(0x0f70);
            }
        }
        alive = sj_test(a, s_sets, small, v, alive);
        if (chunk < a.nchunks) a.keep[chunk * kWave + lane_id()] = uint8_t(alive);
        const uint32_t upto = wave_incl_scan(uint32_t(__popc(alive)));
        const int kept = __builtin_amdgcn_readlane(int(upto), kWave - 1);
        if (a.slab && kept && kept <= kSjSlab) {
            K *slab = static_cast<K *>(a.slab) + chunk * (kSjSlab * NS);
            uint32_t at = (upto - __popc(alive)) * NS;
#pragma unroll
            for (int r = 0; r < kSjIPT; r++) {
                if (!((alive >> r) & 1u)) continue;
#pragma unroll
                for (int s = 0; s < NS; s++) slab[at + s] = v[s][r];
                at += NS;
            }
        }
        if constexpr (VEC && !kAhead) sj_load<K, NS>(a, next_row, next);
        if (lane_id() == 0 && kept) atomicAdd(&s_cnt[turn][in_group >> a.lg_block], uint32_t(kept));
        if (ends) {
            __syncthreads();
            if (int(threadIdx.x) < 1 << (a.lg_group - a.lg_block)) {
                const int64_t b = (int64_t(g0) << (a.lg_group - a.lg_block)) + threadIdx.x;
                if (b << a.lg_block < a.nchunks) a.bcnt[b] = int32_t(s_cnt[turn][threadIdx.x]);
                s_cnt[turn][threadIdx.x] = 0;                // in use again after the next barrier
            }
            turn ^= 1;
        }
    };
    if (g >= ngroups) return;
    if constexpr (kAhead) {
        for (;;) {
            step(va, vb);
            if (g >= ngroups) break;
            step(vb, va);
            if (g >= ngroups) break;
        }
    } else {
        while (g < ngroups) step(va, va);
    }
}

// The rows that the keep bits name, in ascending order: the block's offset is the sum of the
// counts before it, its rows become a list in LDS, and consecutive threads write
// consecutive slots.  (k_filter_write with the keys out of the slabs.)
struct SemiOut {
    void *key_out[kSjMaxSets];
    const void *pin[kSjMaxPay];
    void *pout[kSjMaxPay];
    int32_t paylg[kSjMaxPay];
    int32_t npay;
    int32_t steps;
    int64_t nblocks;
    int32_t *out_rows;
    int64_t *d_count;
    // a table taken in parts: the id of this part's first row, the kept rows of the
    // parts before (null: none) and where the next part finds its own (null: nowhere)
    int32_t row0;
    const int64_t *d_prev;
    int64_t *d_next;
};

// Stores element value v of a payload column of element size 1 << lg.
__device__ __forceinline__ void sj_store(void *out, int lg, int64_t i, uint64_t v) {
    if (lg == 0) static_cast<uint8_t *>(out)[i] = uint8_t(v);
    else if (lg == 2) static_cast<uint32_t *>(out)[i] = uint32_t(v);
    else static_cast<uint64_t *>(out)[i] = v;
}

template <class K, int NS>
__global__ __launch_bounds__(kFilterNT) void k_semi_write(SemiArgs a, SemiOut o) {
    constexpr int kU = 4;                        // rows per thread and pass
    extern __shared__ uint16_t s_list[];         // steps * kFilterTile entries
    __shared__ int32_t s_scan[kFilterNT / kWave];
    __shared__ int64_t s_sum[kFilterNT / kWave];
    __shared__ int32_t s_chunk[kFilterMaxSteps * kFilterTile / kSjChunk + 1];   // first list entry
    if (sj_picks(sizeof(K), NS) && a.pick && *a.pick) return;
    if (o.nblocks == 0 && threadIdx.x == 0) *o.d_count = 0;
    const int steps = o.steps;
    int64_t base = o.d_prev ? *o.d_prev : 0;     // kept rows of the blocks before `from`
    int64_t from = 0;
    for (int64_t b = blockIdx.x; b < o.nblocks; b += gridDim.x) {
        uint64_t bits = keep_word(a.keep, b * kFilterNT + threadIdx.x, steps);
        int64_t part = 0;
#pragma unroll 4
        for (int64_t i = from + threadIdx.x; i < b; i += kFilterNT) part += a.bcnt[i];
        part = wave_sum(part);
        if (lane_id() == 0) s_sum[wave_id()] = part;
        int32_t total;
        int q = block_excl_scan<kFilterNT>(int32_t(__popcll(bits)), &total, s_scan);
#pragma unroll
        for (int w = 0; w < kFilterNT / kWave; w++) base += s_sum[w];
        from = b;
        if (b == o.nblocks - 1 && threadIdx.x == 0) {
            *o.d_count = base + total;
            if (o.d_next) *o.d_next = base + total;
        }
        const int per_chunk = kWave / steps;     // threads whose bits are one chunk
        if (threadIdx.x % per_chunk == 0) s_chunk[threadIdx.x / per_chunk] = q;
        if (threadIdx.x == 0) s_chunk[(1 << a.lg_block)] = total;
        const int first = int(threadIdx.x) * steps * kFilterIPT;
        while (bits) {
            s_list[q++] = uint16_t(first + __builtin_ctzll(bits));
            bits &= bits - 1;
        }
        __syncthreads();
        const int64_t row0 = b * steps * kFilterTile;
        for (int i0 = threadIdx.x; i0 < total; i0 += kU * kFilterNT) {
            const int64_t slot = base + i0;
            int32_t row[kU];
            const K *at[kU];                     // in a slab, or null
#pragma unroll
            for (int u = 0; u < kU; u++) {
                const int i = i0 + u * kFilterNT;
                const int r = s_list[i < total ? i : i0];
                const int c = r / kSjChunk;
                const int beg = s_chunk[c], cnt = s_chunk[c + 1] - beg;
                row[u] = int32_t(row0 + r);
                at[u] = a.slab && cnt <= kSjSlab ? static_cast<const K *>(a.slab) +
                            ((b * (1 << a.lg_block) + c) * kSjSlab + (i < total ? i : i0) - beg) * NS
                                                 : nullptr;
            }
            K key[kU][NS];
#pragma unroll
            for (int u = 0; u < kU; u++) {
                if (at[u]) {
#pragma unroll
                    for (int s = 0; s < NS; s++)
                        if (o.key_out[s]) key[u][s] = at[u][s];
                } else {
#pragma unroll
                    for (int s = 0; s < NS; s++)
                        if (o.key_out[s]) key[u][s] = static_cast<const K *>(a.key[s])[row[u]];
                }
            }
#pragma unroll
            for (int u = 0; u < kU; u++) {
                if (i0 + u * kFilterNT >= total) break;
                if (o.out_rows) o.out_rows[slot + u * kFilterNT] = o.row0 + row[u];
#pragma unroll
                for (int s = 0; s < NS; s++)
                    if (o.key_out[s]) static_cast<K *>(o.key_out[s])[slot + u * kFilterNT] = key[u][s];
            }
            for (int c = 0; c < o.npay; c++) {
                const int lg = o.paylg[c];
                const void *in = o.pin[c];
                uint64_t w[kU];
#pragma unroll
                for (int u = 0; u < kU; u++) w[u] = word_of(in, lg, row[u]);
#pragma unroll
                for (int u = 0; u < kU; u++)
                    if (i0 + u * kFilterNT < total)
                        sj_store(o.pout[c], lg, slot + u * kFilterNT, from_word(w[u], in, lg, row[u]));
            }
        }
        __syncthreads();                         // the lists are reused
    }
}

// The single pass (see sj_picks): tiles handed out by a ticket, each tile's first slot from a
// look-back over the counts of the tiles before it, its rows written straight from registers.
// Bounded by the same reads and writes, then by what a tile waits for: so a tile is as long as
// the registers hold (three 16-byte loads per thread and set), and a compute unit's threads
// are one workgroup.
constexpr int kSjDirectNT = 1024;
constexpr int kSjDirectSteps = 3;                // 16-byte loads per set
template <class K> constexpr int64_t sj_direct_tile() { return int64_t(kSjDirectNT) * (16 / sizeof(K)) * kSjDirectSteps; }
// (a word or status per tile, in place of its keep bits)
static_assert(sj_direct_tile<int64_t>() >= 8 * 8 * 2, "the words fit the keep bits");

template <class K, int NS>
__global__ __launch_bounds__(kSjDirectNT) void k_semi_direct(SemiArgs a, SemiOut o, int vec) {
    constexpr int V = 16 / int(sizeof(K)), Steps = kSjDirectSteps, R = V * Steps;
    constexpr int64_t Step = int64_t(kSjDirectNT) * V, Tile = Step * Steps;
    __shared__ int64_t s_tile, s_prefix;
    __shared__ uint64_t s_scan[kSjDirectNT / kWave];
    extern __shared__ uint32_t s_sets[];
    if (a.pick && !*a.pick) return;
    const int64_t n = a.n, ntiles = ceil_div(n, Tile);
    const int64_t before = o.d_prev ? *o.d_prev : 0;
    const int tid = threadIdx.x;
    uint32_t small[NS];
    sj_stage<NS, false>(a, s_sets, small);
    for (;;) {
        const int64_t tile = take_tile(reinterpret_cast<uint32_t *>(a.words), &s_tile);
        if (tile >= ntiles) break;
        // item r = k * V + j of this thread is row trow + k * Step + j
        const int64_t trow = tile * Tile + int64_t(tid) * V;
        K v[NS][R];
        uint32_t alive = (1u << R) - 1u;
        if (vec && tile * Tile + Tile <= n) {            // (the same for the workgroup)
#pragma unroll
            for (int s = 0; s < NS; s++) {
                const K *p = static_cast<const K *>(a.key[s]) + trow;
#pragma unroll
                for (int k = 0; k < Steps; k++) {
                    const int4 x = *reinterpret_cast<const int4 *>(p + k * Step);
                    const K *e = reinterpret_cast<const K *>(&x);
#pragma unroll
                    for (int j = 0; j < V; j++) v[s][k * V + j] = e[j];
                }
            }
        } else {
            alive = 0;
#pragma unroll
            for (int r = 0; r < R; r++) {
                const int64_t row = trow + (r / V) * Step + r % V;
                alive |= (row < n ? 1u : 0u) << r;
#pragma unroll
                for (int s = 0; s < NS; s++) v[s][r] = row < n ? static_cast<const K *>(a.key[s])[row] : K(0);
            }
        }
        alive = sj_test(a, s_sets, small, v, alive);
        // kept rows are ordered by (step, thread, j): per-step counts, 16 bits apiece (a step
        // keeps at most 4096 rows)
        static_assert(Steps <= 4 && kSjDirectNT * V < 1 << 16, "packed counts");
        uint64_t packed = 0, tot;
#pragma unroll
        for (int k = 0; k < Steps; k++) packed |= uint64_t(__popc((alive >> (k * V)) & ((1u << V) - 1u))) << (16 * k);
        const uint64_t ex = block_excl_scan<kSjDirectNT>(packed, &tot, s_scan);
        int total = 0, first[Steps];                 // the thread's first kept row of each step
#pragma unroll
        for (int k = 0; k < Steps; k++) {
            first[k] = total + int((ex >> (16 * k)) & 0xffff);
            total += int((tot >> (16 * k)) & 0xffff);
        }
        if (wave_id() == 0) {
            const int64_t pre = lookback_count(a.words + 1, tile, total);
            if (lane_id() == 0) s_prefix = pre;
        }
        __syncthreads();
        const int64_t base = before + s_prefix;
        if (tile == ntiles - 1 && tid == 0) {
            *o.d_count = base + total;
            if (o.d_next) *o.d_next = base + total;
        }
        const auto slot_of = [&](int r) {
            const uint32_t mk = (alive >> (r / V * V)) & ((1u << V) - 1u);
            return base + first[r / V] + __popc(mk & ((1u << (r % V)) - 1u));
        };
#pragma unroll
        for (int r = 0; r < R; r++) {
            if (!((alive >> r) & 1u)) continue;
            const int64_t slot = slot_of(r);
            if (o.out_rows) o.out_rows[slot] = o.row0 + int32_t(trow + (r / V) * Step + r % V);
#pragma unroll
            for (int s = 0; s < NS; s++)
                if (o.key_out[s]) static_cast<K *>(o.key_out[s])[slot] = v[s][r];
        }
        for (int c = 0; c < o.npay; c++) {
            const int lg = o.paylg[c];
            const void *in = o.pin[c];
            uint64_t w[R];
#pragma unroll
            for (int r = 0; r < R; r++)
                w[r] = (alive >> r) & 1u ? word_of(in, lg, trow + (r / V) * Step + r % V) : 0;
#pragma unroll
            for (int r = 0; r < R; r++)
                if ((alive >> r) & 1u)
                    sj_store(o.pout[c], lg, slot_of(r), from_word(w[r], in, lg, trow + (r / V) * Step + r % V));
        }
    }
}

// Sets the bit of every key (of the first count) that falls in the set's
// range [lo, lo + nbits).
__global__ __launch_bounds__(256) void k_keyset_set(const void *key, int dt, int64_t n,
                                                    const int64_t *d_n, int64_t lo,
                                                    uint64_t nbits, uint32_t *bits) {
    const int64_t cnt = count_of(d_n, n);
    const int lg = dtype_lg(dt);
    for (int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; i < cnt;
         i += int64_t(gridDim.x) * blockDim.x) {
        const int64_t v = sext_of(load_word(key, lg, i), dt);
        const uint64_t idx = uint64_t(v) - uint64_t(lo);
        if (idx < nbits) atomicOr(&bits[idx >> 5], 1u << (idx & 31));
    }
}

struct SemiLaunch {
    int per_cu, nt;
    size_t lds;
    bool vec;                        // the key columns are 16-byte aligned
};

template <class F> static int sj_allow_lds(F kern, size_t lds) {
    if (lds <= 65536) return TQP_OK;             // more has to be allowed per kernel
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, int(lds));
    return e == hipSuccess ? TQP_OK
                           : set_error(TQP_EHIP, "tqp_semijoin: LDS of %zu bytes: %s", lds, hipGetErrorString(e));
}

template <class K, int NS>
static int launch_semi_direct(const SemiArgs &a, const SemiOut &o, const SemiLaunch &l, hipStream_t s) {
    int rc = sj_allow_lds(k_semi_direct<K, NS>, l.lds);
    if (rc) return rc;
    const unsigned grid = persistent_grid(ceil_div(a.n, sj_direct_tile<K>()), l.lds > 65536 ? 1 : 2);
    TQP_LAUNCH("semijoin_direct", (k_semi_direct<K, NS>), dim3(grid), dim3(kSjDirectNT), l.lds, s, a, o, l.vec ? 1 : 0);
    return check_launch("tqp_semijoin");
}

template <class K, int NS, bool VEC>
static int launch_semijoin(const SemiArgs &a, const SemiOut &o, const SemiLaunch &l, hipStream_t s) {
    int rc;
    if (a.n > 0) {
        if ((rc = sj_allow_lds(k_semi_mask<K, NS, VEC>, l.lds))) return rc;
        const unsigned grid = persistent_grid(ceil_div(a.nchunks, int64_t(1) << a.lg_group), l.per_cu);
        TQP_LAUNCH("semijoin", (k_semi_mask<K, NS, VEC>), dim3(grid), dim3(unsigned(l.nt)), l.lds, s, a);
        if ((rc = check_launch("tqp_semijoin"))) return rc;
    }
    TQP_LAUNCH("semijoin_write", (k_semi_write<K, NS>), dim3(block_grid(o.nblocks)), dim3(kFilterNT),
               size_t(o.steps) * kFilterTile * sizeof(uint16_t), s, a, o);
    if ((rc = check_launch("tqp_semijoin"))) return rc;
    if constexpr (sj_picks(sizeof(K), NS)) {
        if (a.pick) return launch_semi_direct<K, NS>(a, o, l, s);
    }
    return TQP_OK;
}

template <class K, bool VEC>
static int launch_semijoin(int ns, const SemiArgs &a, const SemiOut &o, const SemiLaunch &l, hipStream_t s) {
    switch (ns) {
    case 1: return launch_semijoin<K, 1, VEC>(a, o, l, s);
    case 2: return launch_semijoin<K, 2, VEC>(a, o, l, s);
    case 3: return launch_semijoin<K, 3, VEC>(a, o, l, s);
    default: return launch_semijoin<K, 4, VEC>(a, o, l, s);
    }
}

struct SemiLayout {
    KeepLayout keep;
    void *slab;
    int64_t *d_sum;                  // two, for a table taken in parts
    int32_t *pick;
    size_t bytes;
};

static SemiLayout semi_layout(void *ws, int64_t n, int dtype, bool slabs) {
    SemiLayout L = {};
    Carver c(ws);
    L.d_sum = c.take<int64_t>(3);
    L.pick = reinterpret_cast<int32_t *>(L.d_sum ? L.d_sum + 2 : nullptr);
    const size_t bits = keep_layout(nullptr, n).bytes;
    char *at = c.take<char>(bits);
    L.keep = keep_layout(at, n);
    if (slabs)
        L.slab = c.take<char>(size_t(ceil_div(n, kSjChunk)) * kSjSlab * kSjMaxSets * dtype_size(dtype));
    L.bytes = c.bytes();
    return L;
}

}  // namespace tqp

using namespace tqp;

TQP_API int tqp_keyset_build(const tqp_col *key, const int64_t *d_n, int64_t lo, int64_t nbits,
                             uint32_t *bits, void *stream) {
    clear_error();
    if (!key || !dtype_ok(key->dtype) || key->len < 0 || (key->len > 0 && !key->data) ||
        !col_aligned(key->data, key->dtype))
        return set_error(TQP_EINVAL, "tqp_keyset_build: bad key column");
    if (nbits < 0 || nbits > TQP_KEYSET_MAX_BITS)
        return set_error(TQP_EINVAL, "tqp_keyset_build: nbits must be in [0, 2^36]");
    if (nbits > 0 && !bits) return set_error(TQP_EINVAL, "tqp_keyset_build: bits is required");
    if (nbits > 0 && lo > INT64_MAX - nbits + 1)
        return set_error(TQP_EINVAL, "tqp_keyset_build: lo + nbits - 1 exceeds the int64 range");
    if (nbits == 0) return TQP_OK;
    hipStream_t s = as_stream(stream);
    int rc = fill_u32(bits, 0, ceil_div(nbits, 32), s);
    if (rc || key->len == 0) return rc;
    int64_t blocks = ceil_div(key->len, 256 * 8);
    if (blocks > 2048) blocks = 2048;
    TQP_LAUNCH("keyset_set", k_keyset_set, dim3(unsigned(blocks)), dim3(256), 0, s, key->data,
               key->dtype, key->len, d_n, lo, uint64_t(nbits), bits);
    return check_launch("tqp_keyset_build");
}

TQP_API size_t tqp_semijoin_workspace_bytes(int64_t n, int dtype) {
    return semi_layout(nullptr, n < 0 ? 0 : n, dtype, true).bytes;
}

// Validates the arguments and runs the kernels, over the whole table with slabs (if it is
// large) or, with `part` rows > 0, over parts of that many rows one after another without.
static int semijoin_run(const char *who, const tqp_col *keys, const tqp_keyset *sets, int nsets,
                        const tqp_col *keys_out, const tqp_col *pay_in, const tqp_col *pay_out,
                        int npay, int32_t *out_rows, int64_t *d_count, void *ws, size_t ws_bytes,
                        int64_t part, void *stream) {
    if (!keys || !sets || nsets < 1 || nsets > kSjMaxSets)
        return set_error(TQP_EINVAL, "%s: nsets must be in [1, %d] with keys and sets", who,
                         kSjMaxSets);
    if (npay < 0 || npay > kSjMaxPay || (npay > 0 && (!pay_in || !pay_out)))
        return set_error(TQP_EINVAL, "%s: npay must be in [0, %d] with both arrays", who,
                         kSjMaxPay);
    if (!d_count) return set_error(TQP_EINVAL, "%s: d_count is required", who);
    const int64_t n = keys[0].len;
    const int dt = keys[0].dtype;
    if (n < 0 || n > INT32_MAX)
        return set_error(TQP_EINVAL, "%s: bad row count %lld", who, (long long)n);
    if (dt != TQP_INT32 && dt != TQP_INT64)
        return set_error(TQP_EINVAL, "%s: key columns must be int32 or int64", who);
    SemiArgs a = {};
    SemiOut out = {};
    bool vec = true;
    int lds_words = 0;
    const int knob = tune(kTuneSemiWg);
    const int wg = knob >= 4 ? 4 : knob >= 2 ? 2 : 1;
    const int lds_budget = kSjLdsWordsPer256 * wg;
    for (int s = 0; s < nsets; s++) {
        if (keys[s].dtype != dt || keys[s].len != n || (n > 0 && !keys[s].data) ||
            !col_aligned(keys[s].data, dt))
            return set_error(TQP_EINVAL,
                             "%s: key column %d differs in dtype or length, or is unaligned", who, s);
        if (sets[s].nbits < 0 || sets[s].nbits > TQP_KEYSET_MAX_BITS || (sets[s].nbits > 0 && !sets[s].bits) ||
            (sets[s].nbits > 0 && sets[s].lo > INT64_MAX - sets[s].nbits + 1))
            return set_error(TQP_EINVAL, "%s: key set %d is invalid", who, s);
        vec = vec && reinterpret_cast<uintptr_t>(keys[s].data) % 16 == 0;
        a.key[s] = keys[s].data;
        a.bits[s] = sets[s].bits;
        a.lo[s] = sets[s].lo;
        a.nbits[s] = uint64_t(sets[s].nbits);
        // int32 keys: positions are computed modulo 2^32, over the part of the
        // range that int32 can hold
        if (dt == TQP_INT32 && sets[s].nbits > 0) {
            int64_t lo = sets[s].lo, hi = lo + (sets[s].nbits - 1);
            if (hi < INT32_MIN || lo > INT32_MAX) {
                a.nbits[s] = 0;
            } else {
                if (hi > INT32_MAX) hi = INT32_MAX;
                if (lo < INT32_MIN) {
                    const uint64_t skip = uint64_t(INT32_MIN) - uint64_t(lo);
                    a.bits[s] += skip / 32;
                    a.sh[s] = uint32_t(skip % 32);
                    lo = INT32_MIN;
                }
                a.lo[s] = lo;
                a.nbits[s] = uint64_t(hi - lo) + 1;
            }
        }
        const int64_t words_s = ceil_div(int64_t(a.nbits[s]), 32);
        if (words_s > 0 && a.sh[s] == 0 && lds_words + words_s <= lds_budget && sj_staged(n, nsets, words_s)) {
            a.lds_off[s] = lds_words;
            a.lds_len[s] = int32_t(words_s);
            lds_words += int(words_s) + 2;       // between two zero words
        } else {
            a.lds_off[s] = -1;
            a.lds_len[s] = 0;
        }
        if (keys_out && keys_out[s].data) {
            if (keys_out[s].dtype != dt || keys_out[s].len < n)
                return set_error(TQP_EINVAL, "%s: keys_out[%d] has a bad dtype or length", who, s);
            out.key_out[s] = keys_out[s].data;
        }
    }
    for (int c = 0; c < npay; c++) {
        if (!dtype_ok(pay_in[c].dtype) || pay_in[c].dtype != pay_out[c].dtype ||
            pay_in[c].len < n || pay_out[c].len < n ||
            (n > 0 && (!pay_in[c].data || !pay_out[c].data)) ||
            !col_aligned(pay_in[c].data, pay_in[c].dtype) ||
            !col_aligned(pay_out[c].data, pay_out[c].dtype))
            return set_error(TQP_EINVAL, "%s: payload %d has a bad dtype, length or pointer", who, c);
        out.pin[c] = pay_in[c].data;
        out.pout[c] = pay_out[c].data;
        out.paylg[c] = pay_in[c].dtype == TQP_INT8 ? 0 : pay_in[c].dtype == TQP_INT32 ? 2 : 3;
    }
    out.npay = npay;
    const int64_t most = part > 0 && part < n ? part : n;
    const size_t need = semi_layout(nullptr, most, dt, part == 0).bytes;
    if (!ws || ws_bytes < need)
        return set_error(TQP_ECAPACITY, "%s: scratch needs %zu bytes", who, need);
    hipStream_t s = as_stream(stream);
    out.out_rows = out_rows;
    out.d_count = d_count;
    const int ks = dtype_size(dt);
    int64_t row0 = 0;
    for (int turn = 0; row0 < n || row0 == 0; turn ^= 1) {
        const int64_t rows = sj_part_rows(n, row0, most);
        const SemiLayout L = semi_layout(ws, rows, dt, part == 0);
        a.n = rows;
        // smaller workgroups where larger ones would leave compute units without one and
        // the sets leave room (100K rows of four int64 columns, 60% kept: 21.6 -> 17.5 us)
        int units = wg;                          // 256-thread units per workgroup
        while (units > 1 && rows < int64_t(kComputeUnits) * kSjChunk * (kSjNT / kWave) * units &&
               lds_words <= kSjLdsWordsPer256 * (units / 2))
            units /= 2;
        const int nw = kSjNT * units / kWave;
        const int per_cu = tune(kTuneSemiPerCu) / units > 0 ? tune(kTuneSemiPerCu) / units : 1;
        const int per_block = L.keep.steps * kFilterTile / kSjChunk;        // powers of two
        a.lg_block = __builtin_ctz(per_block);
        a.lg_group = __builtin_ctz(per_block > nw ? per_block : nw);
        a.nchunks = L.keep.nblocks << a.lg_block;
        a.keep = L.keep.keep;
        a.bcnt = L.keep.bcnt;
        const bool large = rows * ks * nsets > kSjCached;
        a.slab = large ? L.slab : nullptr;
        out.steps = L.keep.steps;
        out.nblocks = L.keep.nblocks;
        out.row0 = int32_t(row0);
        out.d_prev = row0 > 0 ? L.d_sum + turn : nullptr;
        out.d_next = row0 + rows < n ? L.d_sum + (turn ^ 1) : nullptr;
        // the single pass leaves the keep bits unwritten: its words take their place
        a.pick = sj_picks(ks, nsets) && large ? L.pick : nullptr;
        a.words = reinterpret_cast<uint64_t *>(L.keep.keep);
        a.nwords = 1 + ceil_div(rows, ks == 4 ? sj_direct_tile<int32_t>() : sj_direct_tile<int64_t>());
        const SemiLaunch l = {per_cu, kSjNT * units, size_t(lds_words) * 4, vec};
        const bool whole = sj_whole_chunks(vec, rows);
        const auto run = dt == TQP_INT32 ? (whole ? launch_semijoin<int32_t, true> : launch_semijoin<int32_t, false>)
                                         : (whole ? launch_semijoin<int64_t, true> : launch_semijoin<int64_t, false>);
        const int rc = run(nsets, a, out, l, s);
        if (rc || n == 0) return rc;
        row0 += rows;
        for (int k = 0; k < nsets; k++) a.key[k] = static_cast<const char *>(a.key[k]) + rows * ks;
        for (int c = 0; c < npay; c++)
            out.pin[c] = static_cast<const char *>(out.pin[c]) + (rows << out.paylg[c]);
    }
    return TQP_OK;
}

TQP_API int tqp_semijoin(const tqp_col *keys, const tqp_keyset *sets, int nsets,
                         const tqp_col *keys_out, const tqp_col *pay_in, const tqp_col *pay_out,
                         int npay, int32_t *out_rows, int64_t *d_count, void *ws, size_t ws_bytes,
                         void *stream) {
    clear_error();
    if (reinterpret_cast<uintptr_t>(ws) % 8 != 0)
        return set_error(TQP_EINVAL, "tqp_semijoin: the workspace must be 8-byte aligned");
    return semijoin_run("tqp_semijoin", keys, sets, nsets, keys_out, pay_in, pay_out, npay,
                        out_rows, d_count, ws, ws_bytes, 0, stream);
}

// ---- the same with library-held scratch -----------------------------------
// For callers that cannot allocate device memory (code under graph capture,
// serving loops, harnesses that forbid allocation): the keep bits and counts
// live in a file-scope device array instead of a caller's workspace, of one part of
// the table at a time.  Each device the library runs on holds its own copy until
// the process ends.
constexpr size_t kSjScratchBytes = size_t(8) << 20;
static_assert(size_t(kSjPartRows) / 8 < kSjScratchBytes, "a part's keep bits");
// The longest table with int64 keys that is accepted (of int32: any).  The parts would
// take more; the limit of an earlier layout of the scratch is kept, for callers that rely on
// what is refused.
constexpr int64_t kSjMaxRows64 = ((int64_t(1) << 20) - 4) * 1536;
static __device__ __align__(256) uint64_t scratch[kSjScratchBytes / 8];
constexpr int kSjMaxDevices = 64;
static std::mutex g_scratch_mu;
static uint64_t *g_scratch_ptr[kSjMaxDevices];

// The device address of this device's scratch (the host-side name of the
// array is not one), looked up on the first call on each device.
static int sj_scratch(uint64_t **out) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess)
        return set_error(TQP_EHIP, "tqp_semijoin_noalloc: hipGetDevice: %s", hipGetErrorString(e));
    if (dev < 0 || dev >= kSjMaxDevices)
        return set_error(TQP_EINVAL, "tqp_semijoin_noalloc: device %d beyond the %d supported", dev,
                         kSjMaxDevices);
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p)
            return set_error(TQP_EHIP, "tqp_semijoin_noalloc: scratch address: %s",
                             hipGetErrorString(e));
        g_scratch_ptr[dev] = static_cast<uint64_t *>(p);
    }
    *out = g_scratch_ptr[dev];
    return TQP_OK;
}

TQP_API int64_t tqp_semijoin_noalloc_max_rows(int dtype) {
    if (dtype != TQP_INT32 && dtype != TQP_INT64) return 0;
    return dtype == TQP_INT32 ? INT32_MAX : kSjMaxRows64;
}

TQP_API int tqp_semijoin_noalloc(const tqp_col *keys, const tqp_keyset *sets, int nsets,
                                 const tqp_col *keys_out, const tqp_col *pay_in,
                                 const tqp_col *pay_out, int npay, int32_t *out_rows,
                                 int64_t *d_count, void *stream) {
    clear_error();
    if (keys && (keys[0].dtype == TQP_INT32 || keys[0].dtype == TQP_INT64) &&
        keys[0].len > tqp_semijoin_noalloc_max_rows(keys[0].dtype))
        return set_error(TQP_ECAPACITY,
                         "tqp_semijoin_noalloc: %lld rows exceed the static scratch's %lld",
                         (long long)keys[0].len,
                         (long long)tqp_semijoin_noalloc_max_rows(keys[0].dtype));
    uint64_t *words = nullptr;
    int rc = sj_scratch(&words);
    if (rc) return rc;
    return semijoin_run("tqp_semijoin_noalloc", keys, sets, nsets, keys_out, pay_in, pay_out,
                        npay, out_rows, d_count, words, kSjScratchBytes, kSjPartRows, stream);
}
