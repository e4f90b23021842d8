// WHERE with stream compaction, in two kernels and no hand-off between
// workgroups.
//
// k_filter_mask streams the predicate columns: 8 consecutive rows per thread,
// every column's loads issued before the first test, one keep bit per row
// written (1/8 byte) and one kept count per block of rows.  k_filter_write
// takes the blocks again: a block's output offset is the sum of the counts
// before it (a few kilobytes, read from the caches), its kept rows are expanded
// from the keep bits into a row list in LDS, in ascending order, and consecutive
// threads write consecutive slots, reading the payload columns through the list.
//
// What bounds it: the read of the predicate columns, then the payload lines that
// hold kept rows.  The version before this one was a single pass with a
// decoupled look-back per 4096-row tile: every tile waited for a ticket, a
// block scan and the look-back before its writes, and the next tile's loads
// behind them.  20M int32 rows keeping 57%, row ids and one byte of payload:
// 92 -> 20 + 45 us.  60M int64 rows keeping one in 84 with 13 bytes of payload
// (beside another stream's work): 244 -> 112 + 64 us.  Slower than that pass: five and
// more int8 payload columns of which more than two thirds are kept, whose bytes go out one per
// store (60M rows, eight columns: 55% kept 448/421 us, 70% 469/498, 100% 506/635).
#include "keepbits.hpp"
#include "rowtest.hpp"

namespace tqp {

constexpr int kMaxPred = 8;
constexpr int kMaxPay = 8;

// Steps (tiles) per block: the widest of 8, 4, 2, 1 that still gives sixteen
// blocks per compute unit, so that both kernels have enough workgroups to hide
// their memory latency and large tables keep the list of block counts short.
static int filter_steps(int64_t n) {
    int st = kFilterMaxSteps;
    while (st > 1 && n < int64_t(kFilterTile) * st * 16 * kComputeUnits) st >>= 1;
    return st;
}

// The kept-row masks of ND columns loaded together (ND = 0: one column after
// another, for more than kMaxTogether).
constexpr int kMaxTogether = 4;
template <int ND>
__device__ __forceinline__ void load_tile(const RowTests &t, int64_t row0, int64_t n, bool vec,
                                          RawRows<kFilterIPT> (&v)[ND > 0 ? ND : 1]) {
#pragma unroll
    for (int c = 0; c < ND; c++) load_rawrows<kFilterIPT>(t.col[c], t.dt[c], row0, n, vec, v[c]);
}
template <int ND>
__device__ __forceinline__ uint32_t test_tile(const RowTests &t, uint32_t mask,
                                              const RawRows<kFilterIPT> (&v)[ND > 0 ? ND : 1]) {
#pragma unroll
    for (int c = 0; c < ND; c++) mask &= test_rows<kFilterIPT>(t, t.beg[c], t.beg[c + 1], t.dt[c], v[c]);
    return mask;
}
template <int ND>
__device__ __forceinline__ uint32_t keep_rows(const RowTests &t, int64_t row0, int64_t n, bool vec,
                                              RawRows<kFilterIPT> (&v)[ND > 0 ? ND : 1]) {
    uint32_t mask = row0 + kFilterIPT <= n ? 0xffu : row0 < n ? (1u << int(n - row0)) - 1u : 0u;
    if constexpr (ND > 0) {
        load_tile<ND>(t, row0, n, vec, v);
        return test_tile<ND>(t, mask, v);
    } else {
        for (int c = 0; c < t.ncol; c++) {
            load_rawrows<kFilterIPT>(t.col[c], t.dt[c], row0, n, vec, v[0]);
            mask &= test_rows<kFilterIPT>(t, t.beg[c], t.beg[c + 1], t.dt[c], v[0]);
        }
        return mask;
    }
}

// keep[row / 8] bit row % 8 and bcnt[block]; a block is `steps` tiles.  Rows
// past n clear their bits, so every byte of a block is written.
template <int ND>
__global__ __launch_bounds__(kFilterNT) void k_filter_mask(RowTests t, int64_t n, int steps, int vec,
                                                           int64_t nblocks, uint8_t *__restrict__ keep,
                                                           int32_t *__restrict__ bcnt) {
    constexpr int U = ND == 1 ? 2 : 1;          // tiles in flight per step
    __shared__ int32_t s_cnt[kFilterNT / kWave];
    for (int64_t b = blockIdx.x; b < nblocks; b += gridDim.x) {
        int32_t kept = 0;
        for (int st = 0; st < steps; st += U) {
            const int64_t unit = (b * steps + st) * kFilterNT + threadIdx.x;   // 8 rows each
            RawRows<kFilterIPT> v[U][ND > 0 ? ND : 1];
            if (U == 2 && st + 1 < steps && vec && (b * steps + st + 2) * kFilterTile <= n) {
                // two whole tiles: both tiles' loads go out before the first test
                uint32_t m[U];
                load_tile<ND>(t, unit * kFilterIPT, n, true, v[0]);
                load_tile<ND>(t, (unit + kFilterNT) * kFilterIPT, n, true, v[U - 1]);
#pragma unroll
                for (int u = 0; u < U; u++) {
                    m[u] = test_tile<ND>(t, 0xffu, v[u]);
                    keep[unit + u * kFilterNT] = uint8_t(m[u]);
                    kept += __popc(m[u]);
                }
            } else {
#pragma unroll
                for (int u = 0; u < U; u++) {
                    if (st + u >= steps) break;
                    const int64_t x = unit + u * kFilterNT;
                    const uint32_t m = keep_rows<ND>(t, x * kFilterIPT, n, vec != 0, v[u]);
                    keep[x] = uint8_t(m);
                    kept += __popc(m);
                }
            }
        }
        kept = wave_sum(kept);
        if (lane_id() == 0) s_cnt[wave_id()] = kept;
        __syncthreads();
        if (threadIdx.x == 0) {
            int32_t tot = 0;
#pragma unroll
            for (int w = 0; w < kFilterNT / kWave; w++) tot += s_cnt[w];
            bcnt[b] = tot;
        }
        __syncthreads();
    }
}

struct FilterOut {
    const void *pin[kMaxPay];
    void *pout[kMaxPay];
    int32_t paydt[kMaxPay];
    int32_t npay;
    int32_t *out_rows;
    int64_t *d_count;
};

// Each thread expands steps * 8 keep bits; then kWriteU list entries per thread
// and pass.  The payload goes out in groups of NP columns (all of them when
// there are at most four): a group's loads, aligned words whatever the dtype, are
// all issued before its first store.
constexpr int kWriteU = 4;
template <class T, int NP>
__device__ __forceinline__ void write_col(void *out, const void *in, int lg, int64_t slot, int c,
                                          const int32_t (&row)[kWriteU],
                                          const uint64_t (&w)[kWriteU][NP > 0 ? NP : 1]) {
    T *o = static_cast<T *>(out) + slot;
#pragma unroll
    for (int u = 0; u < kWriteU; u++)
        if (row[u] >= 0) o[u * kFilterNT] = T(from_word(w[u][c], in, lg, row[u]));
}

template <int NP>
__global__ __launch_bounds__(kFilterNT) void k_filter_write(FilterOut a, int steps, int64_t nblocks,
                                                            const uint8_t *__restrict__ keep,
                                                            const int32_t *__restrict__ bcnt) {
    extern __shared__ uint16_t s_list[];         // steps * kFilterTile entries
    __shared__ int32_t s_scan[kFilterNT / kWave];
    __shared__ int64_t s_sum[kFilterNT / kWave];
    if (nblocks == 0 && threadIdx.x == 0) *a.d_count = 0;
    int64_t base = 0, from = 0;                  // kept rows of the blocks before `from`
    for (int64_t b = blockIdx.x; b < nblocks; b += gridDim.x) {
        const int64_t unit = b * kFilterNT + threadIdx.x;
        uint64_t bits = keep_word(keep, unit, steps);
        int64_t part = 0;
#pragma unroll 4
        for (int64_t i = from + threadIdx.x; i < b; i += kFilterNT) part += bcnt[i];
        part = wave_sum(part);
        if (lane_id() == 0) s_sum[wave_id()] = part;
        int32_t total;
        int q = block_excl_scan<kFilterNT>(int32_t(__popcll(bits)), &total, s_scan);
#pragma unroll
        for (int w = 0; w < kFilterNT / kWave; w++) base += s_sum[w];
        from = b;
        if (b == nblocks - 1 && threadIdx.x == 0) *a.d_count = base + total;
        const int first = int(threadIdx.x) * steps * kFilterIPT;
        while (bits) {
            s_list[q++] = uint16_t(first + __builtin_ctzll(bits));
            bits &= bits - 1;
        }
        __syncthreads();
        const int64_t row0 = b * steps * kFilterTile;
        for (int i0 = threadIdx.x; i0 < total; i0 += kWriteU * kFilterNT) {
            const int64_t slot = base + i0;
            int32_t row[kWriteU];
#pragma unroll
            for (int u = 0; u < kWriteU; u++) {
                const int i = i0 + u * kFilterNT;
                row[u] = i < total ? int32_t(row0 + s_list[i]) : -1;
            }
            if (a.out_rows) {
#pragma unroll
                for (int u = 0; u < kWriteU; u++)
                    if (row[u] >= 0) a.out_rows[slot + u * kFilterNT] = row[u];
            }
            if constexpr (NP > 0) {
                for (int g = 0; g < a.npay; g += NP) {
                    uint64_t w[kWriteU][NP];
#pragma unroll
                    for (int c = 0; c < NP; c++) {
                        if (g + c >= a.npay) break;
                        const int lg = dtype_lg(a.paydt[g + c]);
#pragma unroll
                        for (int u = 0; u < kWriteU; u++)
                            w[u][c] = word_of(a.pin[g + c], lg, row[u] >= 0 ? row[u] : row[0]);
                    }
#pragma unroll
                    for (int c = 0; c < NP; c++) {
                        if (g + c >= a.npay) break;
                        const int lg = dtype_lg(a.paydt[g + c]);
                        void *out = a.pout[g + c];
                        const void *in = a.pin[g + c];
                        if (lg == 0) write_col<uint8_t, NP>(out, in, 0, slot, c, row, w);
                        else if (lg == 2) write_col<uint32_t, NP>(out, in, 2, slot, c, row, w);
                        else write_col<uint64_t, NP>(out, in, 3, slot, c, row, w);
                    }
                }
            }
        }
        __syncthreads();                         // the list is reused
    }
}

// WHERE + aggregate without compaction: the predicate pass of k_filter_mask, then
// SUM(a * b) and COUNT over the kept rows.  A value operand that is also one of
// the (at most kMaxTogether) columns loaded together is taken from those loads;
// other value columns are read only by threads holding a kept row, so at low
// selectivity most of their cache lines are never fetched.  Partial sums are
// reduced per workgroup and added with one device atomic each; int64 addition
// wraps modulo 2^64, so every order gives the same bytes.
//
// What bounds it: the read of the predicate columns.  60M rows of 8 + 4 + 1 bytes
// keeping 1.8%: 241 -> 168 us (4.7 TB/s of those bytes; a plain read of them takes
// 125 us) against the version that converted each column to 64 bits as it was
// loaded, which made every column wait for the one before it.
struct FilterSumArgs {
    RowTests t;
    int32_t vec;
    int32_t aslot, bslot;            // the distinct column that a / b is, or -1
    const void *a;        // null: the sum is 0
    const void *b;        // null: SUM(a)
    int32_t adt, bdt;
    int64_t n;
    unsigned long long *d_sum;
    unsigned long long *d_count;
};

__global__ void k_zero2(unsigned long long *p, unsigned long long *q) {
    if (threadIdx.x == 0) {
        *p = 0;
        *q = 0;
    }
}

// ND distinct predicate columns (1 .. kMaxTogether) loaded together; ND = 0:
// one after another (or none).
template <int ND>
__device__ __forceinline__ void sum_operand(const FilterSumArgs &f, int slot, const void *p, int dt,
                                            int64_t row0, const RawRows<kFilterIPT> (&v)[ND > 0 ? ND : 1],
                                            int64_t (&x)[kFilterIPT]) {
    if constexpr (ND > 0) {
        if (slot >= 0) {
#pragma unroll
            for (int c = 0; c < ND; c++)
                if (c == slot) raw_values<kFilterIPT>(v[c], dt, x);
            return;
        }
    }
    RawRows<kFilterIPT> r;
    load_rawrows<kFilterIPT>(p, dt, row0, f.n, f.vec != 0, r);
    raw_values<kFilterIPT>(r, dt, x);
}

template <int ND>
__global__ __launch_bounds__(kFilterNT) void k_filter_sum(FilterSumArgs f) {
    __shared__ unsigned long long s_red[2][kFilterNT / kWave];
    const int64_t ntiles = ceil_div(f.n, kFilterTile);
    uint64_t sum = 0, cnt = 0;
    for (int64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        const int64_t row0 = tile * kFilterTile + int64_t(threadIdx.x) * kFilterIPT;
        RawRows<kFilterIPT> v[ND > 0 ? ND : 1];
        const uint32_t mask = keep_rows<ND>(f.t, row0, f.n, f.vec != 0, v);
        cnt += __popc(mask);
        if (mask && f.a) {
            int64_t x[kFilterIPT];
            sum_operand<ND>(f, f.aslot, f.a, f.adt, row0, v, x);
            if (f.b) {
                int64_t y[kFilterIPT];
                sum_operand<ND>(f, f.bslot, f.b, f.bdt, row0, v, y);
#pragma unroll
                for (int r = 0; r < kFilterIPT; r++)
                    sum += mask & (1u << r) ? uint64_t(x[r]) * uint64_t(y[r]) : 0;
            } else {
#pragma unroll
                for (int r = 0; r < kFilterIPT; r++) sum += mask & (1u << r) ? uint64_t(x[r]) : 0;
            }
        }
    }
    const uint64_t ws = uint64_t(wave_sum(int64_t(sum)));
    const uint64_t wc = uint64_t(wave_sum(int64_t(cnt)));
    if (lane_id() == 0) {
        s_red[0][wave_id()] = ws;
        s_red[1][wave_id()] = wc;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long ts = 0, tc = 0;
#pragma unroll
        for (int w = 0; w < kFilterNT / kWave; w++) {
            ts += s_red[0][w];
            tc += s_red[1][w];
        }
        if (ts) atomicAdd(f.d_sum, ts);
        if (tc) atomicAdd(f.d_count, tc);
    }
}

// Tiles are dealt to workgroups statically, so the grid holds no more
// workgroups than can be resident at once (their count depends on the
// variant's registers; looked up once per variant): a second round of
// late-starting workgroups would each still take a full share of tiles.
template <class Kern>
static int launch_filter_sum(Kern kern, int nd, int64_t n, hipStream_t s, const FilterSumArgs &f) {
    static int resident[kMaxTogether + 1] = {};
    if (resident[nd] == 0) {
        int per_cu = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void *>(kern),
                                                         kFilterNT, 0) != hipSuccess || per_cu < 1)
            per_cu = 1;
        resident[nd] = per_cu;
    }
    int per_cu = 2 * tune(kTuneFilterPerCu);
    if (per_cu > resident[nd]) per_cu = resident[nd];
    const unsigned grid = persistent_grid(ceil_div(n, kFilterTile), per_cu);
    TQP_LAUNCH("filter_sum", kern, dim3(grid), dim3(kFilterNT), 0, s, f);
    return check_launch("tqp_filter_sum");
}

KeepLayout keep_layout(void *ws, int64_t n) {
    KeepLayout L = {};
    Carver c(ws);
    L.steps = filter_steps(n);
    L.nblocks = ceil_div(n, int64_t(kFilterTile) * L.steps);
    L.keep = c.take<uint8_t>(size_t(L.nblocks) * kFilterNT * L.steps);
    L.bcnt = c.take<int32_t>(size_t(L.nblocks > 0 ? L.nblocks : 1));
    L.bytes = c.bytes();
    return L;
}

template <int ND>
static void launch_filter_mask(unsigned grid, hipStream_t s, const RowTests &t, int64_t n, bool vec,
                               const KeepLayout &L) {
    TQP_LAUNCH("filter_mask", k_filter_mask<ND>, dim3(grid), dim3(kFilterNT), 0, s, t, n, L.steps,
               vec ? 1 : 0, L.nblocks, L.keep, L.bcnt);
}

template <int NP>
static void launch_filter_write(unsigned grid, hipStream_t s, const FilterOut &a, const KeepLayout &L) {
    TQP_LAUNCH("filter", k_filter_write<NP>, dim3(grid), dim3(kFilterNT),
               size_t(L.steps) * kFilterTile * sizeof(uint16_t), s, a, L.steps, L.nblocks, L.keep, L.bcnt);
}

}  // namespace tqp

using namespace tqp;

TQP_API size_t tqp_filter_workspace_bytes(int64_t n) { return keep_layout(nullptr, n < 0 ? 0 : n).bytes; }

TQP_API int tqp_filter(const tqp_col *cols, int ncols, const tqp_pred *preds, int npred,
                       const tqp_col *pay_in, const tqp_col *pay_out, int npay,
                       int32_t *out_rows, int64_t *d_count, void *ws, size_t ws_bytes,
                       void *stream) {
    clear_error();
    if (!cols || ncols < 1 || ncols > kMaxPred)
        return set_error(TQP_EINVAL, "tqp_filter: ncols must be in [1, %d]", kMaxPred);
    if (!preds || npred < 1 || npred > kMaxPred)
        return set_error(TQP_EINVAL, "tqp_filter: npred must be in [1, %d]", kMaxPred);
    if (npay < 0 || npay > kMaxPay || (npay > 0 && (!pay_in || !pay_out)))
        return set_error(TQP_EINVAL, "tqp_filter: npay must be in [0, %d] with both arrays", kMaxPay);
    if (!d_count) return set_error(TQP_EINVAL, "tqp_filter: d_count is required");
    const int64_t n = cols[0].len;
    if (n < 0 || n > INT32_MAX) return set_error(TQP_EINVAL, "tqp_filter: bad row count %lld", (long long)n);
    FilterOut a = {};
    bool vec = true;
    for (int c = 0; c < ncols; c++) {
        if (!dtype_ok(cols[c].dtype) || cols[c].len != n || (n > 0 && !cols[c].data))
            return set_error(TQP_EINVAL, "tqp_filter: column %d has a bad dtype, length or pointer", c);
        if (!col_aligned(cols[c].data, cols[c].dtype))
            return set_error(TQP_EINVAL, "tqp_filter: column %d is unaligned", c);
        vec = vec && (reinterpret_cast<uintptr_t>(cols[c].data) % 16 == 0);
    }
    for (int p = 0; p < npred; p++)
        if (preds[p].col < 0 || preds[p].col >= ncols || preds[p].op < TQP_LT || preds[p].op > TQP_NE)
            return set_error(TQP_EINVAL, "tqp_filter: predicate %d is invalid", p);
    for (int c = 0; c < npay; c++) {
        if (!dtype_ok(pay_in[c].dtype) || pay_in[c].dtype != pay_out[c].dtype ||
            pay_in[c].len != n || pay_out[c].len < n || (n > 0 && (!pay_in[c].data || !pay_out[c].data)))
            return set_error(TQP_EINVAL, "tqp_filter: payload %d has a bad dtype, length or pointer", c);
        // (kept rows' payload is read as the aligned 8-byte word holding it)
        if (!col_aligned(pay_in[c].data, pay_in[c].dtype) || !col_aligned(pay_out[c].data, pay_out[c].dtype))
            return set_error(TQP_EINVAL, "tqp_filter: payload %d is unaligned", c);
        a.pin[c] = pay_in[c].data;
        a.pout[c] = pay_out[c].data;
        a.paydt[c] = pay_in[c].dtype;
    }
    KeepLayout L = keep_layout(nullptr, n);
    if (!ws || ws_bytes < L.bytes)
        return set_error(TQP_ECAPACITY, "tqp_filter: workspace needs %zu bytes", L.bytes);
    L = keep_layout(ws, n);
    RowTests t;
    build_tests(cols, preds, npred, &t);
    a.npay = npay;
    a.out_rows = out_rows;
    a.d_count = d_count;
    hipStream_t s = as_stream(stream);
    if (n > 0) {
        const unsigned grid = block_grid(L.nblocks);
        switch (t.ncol <= kMaxTogether ? t.ncol : 0) {
        case 1: launch_filter_mask<1>(grid, s, t, n, vec, L); break;
        case 2: launch_filter_mask<2>(grid, s, t, n, vec, L); break;
        case 3: launch_filter_mask<3>(grid, s, t, n, vec, L); break;
        case 4: launch_filter_mask<4>(grid, s, t, n, vec, L); break;
        default: launch_filter_mask<0>(grid, s, t, n, vec, L); break;
        }
        const int rc = check_launch("tqp_filter");
        if (rc) return rc;
    }
    const unsigned grid = block_grid(L.nblocks);
    switch (npay < 4 ? npay : 4) {
    case 0: launch_filter_write<0>(grid, s, a, L); break;
    case 1: launch_filter_write<1>(grid, s, a, L); break;
    case 2: launch_filter_write<2>(grid, s, a, L); break;
    case 3: launch_filter_write<3>(grid, s, a, L); break;
    default: launch_filter_write<4>(grid, s, a, L); break;
    }
    return check_launch("tqp_filter");
}

TQP_API int tqp_filter_sum(const tqp_col *cols, int ncols, const tqp_pred *preds, int npred,
                           const tqp_col *a, const tqp_col *b, int64_t *d_sum, int64_t *d_count,
                           void *stream) {
    clear_error();
    if (!cols || ncols < 1 || ncols > kMaxPred)
        return set_error(TQP_EINVAL, "tqp_filter_sum: ncols must be in [1, %d]", kMaxPred);
    if (npred < 0 || npred > kMaxPred || (npred > 0 && !preds))
        return set_error(TQP_EINVAL, "tqp_filter_sum: npred must be in [0, %d]", kMaxPred);
    if (!d_sum || !d_count) return set_error(TQP_EINVAL, "tqp_filter_sum: d_sum and d_count are required");
    if (b && !a) return set_error(TQP_EINVAL, "tqp_filter_sum: b needs a");
    const int64_t n = cols[0].len;
    if (n < 0 || n > INT32_MAX) return set_error(TQP_EINVAL, "tqp_filter_sum: bad row count %lld", (long long)n);
    FilterSumArgs f = {};
    bool vec = true;
    for (int c = 0; c < ncols; c++) {
        if (!dtype_ok(cols[c].dtype) || cols[c].len != n || (n > 0 && !cols[c].data) ||
            !col_aligned(cols[c].data, cols[c].dtype))
            return set_error(TQP_EINVAL, "tqp_filter_sum: column %d has a bad dtype, length or pointer", c);
        vec = vec && (reinterpret_cast<uintptr_t>(cols[c].data) % 16 == 0);
    }
    for (int p = 0; p < npred; p++)
        if (preds[p].col < 0 || preds[p].col >= ncols || preds[p].op < TQP_LT || preds[p].op > TQP_NE)
            return set_error(TQP_EINVAL, "tqp_filter_sum: predicate %d is invalid", p);
    build_tests(cols, preds, npred, &f.t);
    const tqp_col *vals[2] = {a, b};
    for (int k = 0; k < 2; k++) {
        const tqp_col *v = vals[k];
        if (!v) continue;
        if (!dtype_ok(v->dtype) || v->len < n || (n > 0 && !v->data) || !col_aligned(v->data, v->dtype))
            return set_error(TQP_EINVAL, "tqp_filter_sum: value column %c has a bad dtype, length or pointer",
                             k ? 'b' : 'a');
        vec = vec && (reinterpret_cast<uintptr_t>(v->data) % 16 == 0);
    }
    f.vec = vec ? 1 : 0;
    f.a = a ? a->data : nullptr;
    f.b = b ? b->data : nullptr;
    f.adt = a ? a->dtype : 0;
    f.bdt = b ? b->dtype : 0;
    // a value operand that is one of the loaded predicate columns
    f.aslot = f.bslot = -1;
    for (int c = 0; c < f.t.ncol; c++) {
        if (a && f.aslot < 0 && f.t.col[c] == a->data && f.t.dt[c] == a->dtype) f.aslot = c;
        if (b && f.bslot < 0 && f.t.col[c] == b->data && f.t.dt[c] == b->dtype) f.bslot = c;
    }
    f.n = n;
    f.d_sum = reinterpret_cast<unsigned long long *>(d_sum);
    f.d_count = reinterpret_cast<unsigned long long *>(d_count);
    hipStream_t s = as_stream(stream);
    TQP_LAUNCH("filter_sum_init", k_zero2, dim3(1), dim3(64), 0, s, f.d_sum, f.d_count);
    int rc = check_launch("tqp_filter_sum");
    if (rc || n == 0) return rc;
    const int nd = f.t.ncol <= kMaxTogether ? f.t.ncol : 0;
    switch (nd) {
    case 1: return launch_filter_sum(k_filter_sum<1>, nd, n, s, f);
    case 2: return launch_filter_sum(k_filter_sum<2>, nd, n, s, f);
    case 3: return launch_filter_sum(k_filter_sum<3>, nd, n, s, f);
    case 4: return launch_filter_sum(k_filter_sum<4>, nd, n, s, f);
    default: return launch_filter_sum(k_filter_sum<0>, nd, n, s, f);
    }
}
