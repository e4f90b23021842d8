// Library-wide pieces: error text, fills, the key-range reduction.
#include <stdarg.h>
#include <stdio.h>
#include <string.h>

#include "tqp_internal.hpp"

namespace tqp {

static thread_local char g_err[512];

int set_error(int code, const char *fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof g_err, fmt, ap);
    va_end(ap);
    return code;
}

void clear_error() { g_err[0] = 0; }

int check_launch(const char *what) {
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return set_error(TQP_EHIP, "%s: %s", what, hipGetErrorString(e));
    return TQP_OK;
}

int dtype_size(int dtype) {
    switch (dtype) {
    case TQP_INT8: return 1;
    case TQP_INT32: return 4;
    case TQP_INT64: return 8;
    default: return 0;
    }
}

bool dtype_ok(int dtype) { return dtype_size(dtype) != 0; }
bool col_aligned(const void *p, int dtype) {
    const int sz = dtype_size(dtype);
    return sz != 0 && reinterpret_cast<uintptr_t>(p) % uintptr_t(sz) == 0;
}

__global__ void k_fill_u64(uint64_t *p, uint64_t v, int64_t n) {
    for (int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; i < n;
         i += int64_t(gridDim.x) * blockDim.x)
        p[i] = v;
}

__global__ void k_fill_u32(uint32_t *p, uint32_t v, int64_t n) {
    for (int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; i < n;
         i += int64_t(gridDim.x) * blockDim.x)
        p[i] = v;
}

int fill_u64(void *dst, uint64_t value, int64_t count, hipStream_t s) {
    if (count <= 0) return TQP_OK;
    int64_t blocks = ceil_div(count, 256);
    if (blocks > 4096) blocks = 4096;
    TQP_LAUNCH("fill_u64", k_fill_u64, dim3(unsigned(blocks)), dim3(256), 0, s,
                       static_cast<uint64_t *>(dst), value, count);
    return check_launch("fill_u64");
}

int fill_u32(void *dst, uint32_t value, int64_t count, hipStream_t s) {
    if (count <= 0) return TQP_OK;
    int64_t blocks = ceil_div(count, 256);
    if (blocks > 4096) blocks = 4096;
    TQP_LAUNCH("fill_u32", k_fill_u32, dim3(unsigned(blocks)), dim3(256), 0, s,
                       static_cast<uint32_t *>(dst), value, count);
    return check_launch("fill_u32");
}

constexpr int kMmNT = 1024;
constexpr int kMmBlocks = 2 * kComputeUnits;

struct MinmaxArgs {
    const void *key[2];
    int64_t n[2];
    const int64_t *d_n[2];
    int64_t *out;
};

__global__ void k_minmax_init(int64_t *out) {
    if (threadIdx.x < 2) out[threadIdx.x] = threadIdx.x ? INT64_MIN : INT64_MAX;
}

// Min and max of the first count keys of column blockIdx.y (INT64_MAX and
// INT64_MIN of none).  PARTS: each workgroup's to its own pair of out; otherwise
// all of them to the pair out[0], out[1], which must hold those of no keys.
//
// What bounds it: one read of the column, so kU loads are in flight per thread; those
// past the end repeat the last key, so none sits behind a branch.  At one pair the
// atomics of all workgroups meet (about 11 ns each), and it has to be cleared
// first: ranges that the host waits for come as parts, which it reduces itself.
// 10M int64 keys (80 MB): 71 us + 9 us of clearing with 2048 workgroups of 256
// threads, one load in flight; 31 us with these. 5M from cache: 36 + 9, now 10 us.
template <class K, bool PARTS>
__global__ __launch_bounds__(kMmNT) void k_minmax(MinmaxArgs a) {
    constexpr int kU = 8;
    const int64_t cnt = count_of(a.d_n[blockIdx.y], a.n[blockIdx.y]);
    const K *key = static_cast<const K *>(a.key[blockIdx.y]);
    int64_t lo = INT64_MAX, hi = INT64_MIN;
    if (cnt > 0) {
        K klo = key[0], khi = klo;
        for (int64_t base = blockIdx.x * int64_t(kMmNT) * kU + threadIdx.x; base - threadIdx.x < cnt;
             base += int64_t(gridDim.x) * kMmNT * kU) {
            K v[kU];
#pragma unroll
            for (int u = 0; u < kU; u++) {
                const int64_t i = base + u * kMmNT;
                v[u] = key[i < cnt ? i : cnt - 1];
            }
#pragma unroll
            for (int u = 0; u < kU; u++) {
                klo = v[u] < klo ? v[u] : klo;
                khi = v[u] > khi ? v[u] : khi;
            }
        }
        lo = klo;
        hi = khi;
    }
#pragma unroll
    for (int m = 1; m < kWave; m <<= 1) {
        int64_t x = shfl_xor(lo, m), y = shfl_xor(hi, m);
        lo = x < lo ? x : lo;
        hi = y > hi ? y : hi;
    }
    __shared__ int64_t slo[kMmNT / kWave], shi[kMmNT / kWave];
    if (lane_id() == 0) { slo[wave_id()] = lo; shi[wave_id()] = hi; }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kMmNT / kWave; w++) {
            lo = slo[w] < lo ? slo[w] : lo;
            hi = shi[w] > hi ? shi[w] : hi;
        }
        if constexpr (PARTS) {
            int64_t *out = a.out + 2 * (int64_t(blockIdx.y) * gridDim.x + blockIdx.x);
            out[0] = lo;
            out[1] = hi;
        } else if (cnt > 0) {
            atomicMin(reinterpret_cast<long long *>(&a.out[0]), (long long)lo);
            atomicMax(reinterpret_cast<long long *>(&a.out[1]), (long long)hi);
        }
    }
}

template <bool PARTS>
static int minmax_pass(const MinmaxArgs &a, int ncol, int dtype, int64_t blocks, hipStream_t s) {
    const dim3 g{unsigned(blocks), unsigned(ncol), 1};
    if (dtype == TQP_INT8)
        TQP_LAUNCH("minmax", (k_minmax<int8_t, PARTS>), g, dim3(kMmNT), 0, s, a);
    else if (dtype == TQP_INT32)
        TQP_LAUNCH("minmax", (k_minmax<int32_t, PARTS>), g, dim3(kMmNT), 0, s, a);
    else
        TQP_LAUNCH("minmax", (k_minmax<int64_t, PARTS>), g, dim3(kMmNT), 0, s, a);
    return check_launch("minmax");
}

int launch_minmax(const void *key, int dtype, int64_t n, const int64_t *d_n,
                  int64_t *out, hipStream_t s) {
    TQP_LAUNCH("minmax_init", k_minmax_init, dim3(1), dim3(kWave), 0, s, out);
    int rc = check_launch("minmax_init");
    if (rc || n <= 0) return rc;
    const int64_t blocks = ceil_div(n, kMmNT * 4);
    return minmax_pass<false>({{key, nullptr}, {n, 0}, {d_n, nullptr}, out}, 1, dtype,
                              blocks < kMmBlocks / 2 ? blocks : kMmBlocks / 2, s);
}

static int derive_ranges(MinmaxArgs a, int ncol, int dtype, void *scratch, size_t scratch_bytes,
                         hipStream_t s, int64_t *key_min, int *key_bits) {
    const int64_t n = ncol > 1 && a.n[1] > a.n[0] ? a.n[1] : a.n[0];
    int64_t blocks = ceil_div(n, kMmNT * 4);
    if (blocks > kMmBlocks) blocks = kMmBlocks;
    const int64_t room = int64_t(scratch_bytes / 16) / ncol;
    if (blocks > room) blocks = room;
    int64_t host[2 * 2 * kMmBlocks];
    if (n > 0) {
        if (!scratch || blocks < 1) return set_error(TQP_ECAPACITY, "key range: no scratch");
        a.out = static_cast<int64_t *>(scratch);
        const int rc = minmax_pass<true>(a, ncol, dtype, blocks, s);
        if (rc) return rc;
        hipError_t e = hipMemcpyAsync(host, a.out, size_t(ncol * blocks) * 16, hipMemcpyDeviceToHost, s);
        if (e == hipSuccess) e = hipStreamSynchronize(s);
        if (e != hipSuccess)
            return set_error(TQP_EHIP, "key range read-back: %s", hipGetErrorString(e));
    }
    for (int c = 0; c < ncol; c++) {
        int64_t lo = INT64_MAX, hi = INT64_MIN;
        for (int64_t b = c * blocks; b < (c + 1) * blocks; b++) {
            lo = host[2 * b] < lo ? host[2 * b] : lo;
            hi = host[2 * b + 1] > hi ? host[2 * b + 1] : hi;
        }
        const bool any = lo <= hi;
        const uint64_t span = any ? uint64_t(hi) - uint64_t(lo) : 0;
        int bits = 0;
        while (bits < 64 && (span >> bits) != 0) bits++;
        key_min[c] = any ? lo : 0;
        key_bits[c] = bits;
    }
    return TQP_OK;
}

int derive_key_range(const void *key, int dtype, int64_t n, const int64_t *d_n, void *scratch,
                     size_t scratch_bytes, hipStream_t s, int64_t *key_min, int *key_bits) {
    return derive_ranges({{key, nullptr}, {n, 0}, {d_n, nullptr}, nullptr}, 1, dtype, scratch,
                         scratch_bytes, s, key_min, key_bits);
}

int derive_key_ranges(const void *const key[2], int dtype, const int64_t n[2],
                      const int64_t *const d_n[2], void *scratch, size_t scratch_bytes,
                      hipStream_t s, int64_t key_min[2], int key_bits[2]) {
    return derive_ranges({{key[0], key[1]}, {n[0], n[1]}, {d_n[0], d_n[1]}, nullptr}, 2, dtype,
                         scratch, scratch_bytes, s, key_min, key_bits);
}

}  // namespace tqp

namespace tqp {

struct KnobDef {
    const char *name;
    int def, lo, hi;
};
static const KnobDef kKnobs[kTuneCount] = {
    {"filter.per_cu", 4, 1, 8},
    {"sort.per_cu", 1, 1, 2},
    {"rle.per_cu", 1, 1, 2},
    {"match.per_cu", 4, 1, 8},
    {"gbscan.per_cu", 2, 1, 4},
    {"part.ovf_cap", 65536, 1, 65536},
    {"sort.mode", 0, 0, 1},
    {"semijoin.per_cu", 4, 1, 8},
    {"semijoin.wg", 4, 1, 4},
};
static int g_knob[kTuneCount] = {4, 1, 1, 4, 2, 65536, 0, 4, 4};

int tune(TuneKnob k) { return g_knob[k]; }

}  // namespace tqp

TQP_API const char *tqp_last_error(void) { return tqp::g_err; }

TQP_API int tqp_tune_set(const char *name, int value) {
    tqp::clear_error();
    for (int k = 0; k < tqp::kTuneCount; k++) {
        if (name && strcmp(name, tqp::kKnobs[k].name) == 0) {
            if (value < tqp::kKnobs[k].lo || value > tqp::kKnobs[k].hi)
                return tqp::set_error(TQP_EINVAL, "tqp_tune_set: %s must be in [%d, %d]", name,
                                      tqp::kKnobs[k].lo, tqp::kKnobs[k].hi);
            tqp::g_knob[k] = value;
            return TQP_OK;
        }
    }
    return tqp::set_error(TQP_EINVAL, "tqp_tune_set: unknown knob %s", name ? name : "(null)");
}

TQP_API int tqp_tune_get(const char *name, int *value, int *lo, int *hi) {
    for (int k = 0; k < tqp::kTuneCount; k++) {
        if (name && strcmp(name, tqp::kKnobs[k].name) == 0) {
            if (value) *value = tqp::g_knob[k];
            if (lo) *lo = tqp::kKnobs[k].lo;
            if (hi) *hi = tqp::kKnobs[k].hi;
            return TQP_OK;
        }
    }
    return tqp::set_error(TQP_EINVAL, "tqp_tune_get: unknown knob %s", name ? name : "(null)");
}

TQP_API const char *tqp_tune_name(int index) {
    return index >= 0 && index < tqp::kTuneCount ? tqp::kKnobs[index].name : nullptr;
}

TQP_API int tqp_minmax(const tqp_col *key, const int64_t *d_n, int64_t *d_out, void *stream) {
    tqp::clear_error();
    if (!key || !tqp::dtype_ok(key->dtype) || key->len < 0 || (key->len > 0 && !key->data) ||
        !tqp::col_aligned(key->data, key->dtype))
        return tqp::set_error(TQP_EINVAL, "tqp_minmax: bad key column");
    if (!d_out) return tqp::set_error(TQP_EINVAL, "tqp_minmax: d_out is required");
    return tqp::launch_minmax(key->data, key->dtype, key->len, d_n, d_out,
                              tqp::as_stream(stream));
}

TQP_API const char *tqp_version(void) { return "tqp-mi355x 0.1 (gfx950)"; }
