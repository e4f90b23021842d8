// Predicate conjunctions as range tests, shared by the operators that evaluate
// them over whole columns (filter, filter + aggregate, filter + sort).
//
// The host turns `column op literal` into `(value - lo) <= span`, unsigned:
// one subtraction and one compare for every operator, with no per-row switch.
// All the ordering and equality predicates of one column intersect into a
// single range; != is the same test negated.  Columns of 1 or 4 bytes test in
// 32 bits.
//
// Loading and testing are separate: a column's rows are first loaded as raw
// words, with no conversion, so the loads of several columns go out together
// (a conversion inside the branch that picks the dtype makes the compiler
// wait for that column before the next one's loads).
#pragma once

#include "tqp_internal.hpp"

namespace tqp {

constexpr int kMaxTests = 8;

struct RowTests {
    const void *col[kMaxTests];     // the distinct columns
    int32_t dt[kMaxTests];
    int32_t beg[kMaxTests + 1];     // column c's tests: beg[c] .. beg[c + 1] - 1
    int32_t ncol;
    int64_t lo[kMaxTests];
    uint64_t span[kMaxTests];
    int32_t neg[kMaxTests];         // 1: holds outside the range
};

// The tests of a conjunction over cols (arguments already validated), columns
// in order of first use.  A range no value of the column's dtype can be in
// becomes a test that never holds.
inline void build_tests(const tqp_col *cols, const tqp_pred *preds, int npred, RowTests *t) {
    *t = RowTests{};
    int nt = 0;
    for (int p = 0; p < npred; p++) {
        const int col = preds[p].col;
        bool seen = false;
        for (int q = 0; q < p; q++) seen = seen || preds[q].col == col;
        if (seen) continue;
        const int dt = cols[col].dtype;
        const int64_t tmin = dt == TQP_INT8 ? INT8_MIN : dt == TQP_INT32 ? INT32_MIN : INT64_MIN;
        const int64_t tmax = dt == TQP_INT8 ? INT8_MAX : dt == TQP_INT32 ? INT32_MAX : INT64_MAX;
        t->col[t->ncol] = cols[col].data;
        t->dt[t->ncol] = dt;
        t->beg[t->ncol] = nt;
        t->ncol++;
        int64_t lo = tmin, hi = tmax;
        bool never = false, ranged = false;
        for (int q = p; q < npred; q++) {
            if (preds[q].col != col) continue;
            const int64_t lit = preds[q].literal;
            switch (preds[q].op) {
            case TQP_LT:
                if (lit == INT64_MIN) never = true;
                else hi = lit - 1 < hi ? lit - 1 : hi;
                ranged = true;
                break;
            case TQP_LE: hi = lit < hi ? lit : hi; ranged = true; break;
            case TQP_GT:
                if (lit == INT64_MAX) never = true;
                else lo = lit + 1 > lo ? lit + 1 : lo;
                ranged = true;
                break;
            case TQP_GE: lo = lit > lo ? lit : lo; ranged = true; break;
            case TQP_EQ:
                lo = lit > lo ? lit : lo;
                hi = lit < hi ? lit : hi;
                ranged = true;
                break;
            default:
                if (lit >= tmin && lit <= tmax) {      // otherwise it always holds
                    t->lo[nt] = lit;
                    t->span[nt] = 0;
                    t->neg[nt] = 1;
                    nt++;
                }
                break;
            }
        }
        if (never || lo > hi) {
            t->lo[nt] = 0;                             // outside the whole range: never
            t->span[nt] = ~uint64_t(0);
            t->neg[nt] = 1;
            nt++;
        } else if (ranged) {
            t->lo[nt] = lo;
            t->span[nt] = uint64_t(hi) - uint64_t(lo);
            t->neg[nt] = 0;
            nt++;
        }
    }
    t->beg[t->ncol] = nt;
}

// N (a multiple of 8) consecutive rows of one column, as loaded: N 8-byte,
// N 4-byte or N 1-byte elements in the first 2 N, N or N / 4 words.
template <int N> struct RawRows {
    uint32_t w[2 * N];
};

// vec: the column is 16-byte aligned.  Rows at or past n read as 0.
template <int N>
__device__ __forceinline__ void load_rawrows(const void *p, int dt, int64_t row0, int64_t n, bool vec,
                                             RawRows<N> &v) {
    if (vec && row0 + N <= n) {
        if (dt == TQP_INT64) {
            const uint4 *q = reinterpret_cast<const uint4 *>(static_cast<const int64_t *>(p) + row0);
#pragma unroll
            for (int k = 0; k < N / 2; k++) {
                const uint4 x = q[k];
                v.w[4 * k] = x.x; v.w[4 * k + 1] = x.y; v.w[4 * k + 2] = x.z; v.w[4 * k + 3] = x.w;
            }
        } else if (dt == TQP_INT32) {
            const uint4 *q = reinterpret_cast<const uint4 *>(static_cast<const int32_t *>(p) + row0);
#pragma unroll
            for (int k = 0; k < N / 4; k++) {
                const uint4 x = q[k];
                v.w[4 * k] = x.x; v.w[4 * k + 1] = x.y; v.w[4 * k + 2] = x.z; v.w[4 * k + 3] = x.w;
            }
        } else {
            const uint2 *q = reinterpret_cast<const uint2 *>(static_cast<const int8_t *>(p) + row0);
#pragma unroll
            for (int k = 0; k < N / 8; k++) {
                const uint2 x = q[k];
                v.w[2 * k] = x.x; v.w[2 * k + 1] = x.y;
            }
        }
    } else if (dt == TQP_INT64) {
#pragma unroll
        for (int r = 0; r < N; r++) {
            const uint64_t x = row0 + r < n ? static_cast<const uint64_t *>(p)[row0 + r] : 0;
            v.w[2 * r] = uint32_t(x);
            v.w[2 * r + 1] = uint32_t(x >> 32);
        }
    } else if (dt == TQP_INT32) {
#pragma unroll
        for (int r = 0; r < N; r++)
            v.w[r] = row0 + r < n ? static_cast<const uint32_t *>(p)[row0 + r] : 0u;
    } else {
#pragma unroll
        for (int k = 0; k < N / 4; k++) {
            uint32_t x = 0;
#pragma unroll
            for (int j = 0; j < 4; j++) {
                const int64_t r = row0 + 4 * k + j;
                x |= (r < n ? uint32_t(static_cast<const uint8_t *>(p)[r]) : 0u) << (8 * j);
            }
            v.w[k] = x;
        }
    }
}

// Row r's element of a raw 1- or 4-byte column, sign-extended to 32 bits.
template <int N> __device__ __forceinline__ int32_t raw_i32(const RawRows<N> &v, int dt, int r) {
    return dt == TQP_INT32 ? int32_t(v.w[r]) : int32_t(int8_t(v.w[r / 4] >> (8 * (r % 4))));
}
template <int N> __device__ __forceinline__ int64_t raw_i64(const RawRows<N> &v, int r) {
    return int64_t(uint64_t(v.w[2 * r]) | uint64_t(v.w[2 * r + 1]) << 32);
}

// All N elements of a raw column, sign-extended to 64 bits.
template <int N>
__device__ __forceinline__ void raw_values(const RawRows<N> &v, int dt, int64_t (&x)[N]) {
    if (dt == TQP_INT64) {
#pragma unroll
        for (int r = 0; r < N; r++) x[r] = raw_i64(v, r);
    } else if (dt == TQP_INT32) {
#pragma unroll
        for (int r = 0; r < N; r++) x[r] = raw_i32(v, TQP_INT32, r);
    } else {
#pragma unroll
        for (int r = 0; r < N; r++) x[r] = raw_i32(v, TQP_INT8, r);
    }
}

// Bit r: row r passes tests [t0, t1) of column dtype dt.
template <int N>
__device__ __forceinline__ uint32_t test_rows(const RowTests &t, int t0, int t1, int dt,
                                              const RawRows<N> &v) {
    static_assert(N <= 32, "one bit per row in a word");
    uint32_t mask = N == 32 ? ~0u : (1u << N) - 1u;
    for (int k = t0; k < t1; k++) {
        uint32_t m = 0;
        if (dt == TQP_INT64) {
            const uint64_t lo = uint64_t(t.lo[k]), span = t.span[k];
#pragma unroll
            for (int r = 0; r < N; r++) m |= (uint64_t(raw_i64(v, r)) - lo <= span ? 1u : 0u) << r;
        } else {
            const uint32_t lo = uint32_t(t.lo[k]), span = uint32_t(t.span[k]);
            if (dt == TQP_INT32) {
#pragma unroll
                for (int r = 0; r < N; r++)
                    m |= (uint32_t(raw_i32(v, TQP_INT32, r)) - lo <= span ? 1u : 0u) << r;
            } else {
#pragma unroll
                for (int r = 0; r < N; r++)
                    m |= (uint32_t(raw_i32(v, TQP_INT8, r)) - lo <= span ? 1u : 0u) << r;
            }
        }
        mask &= t.neg[k] ? ~m : m;
    }
    return mask;
}

}  // namespace tqp
