// PREDICT inside a query: an fp32 MLP with one ReLU hidden layer scores each
// row.  Every multiply-add is one fused fma, k and j ascending, relu(v) is
// (v > 0 ? v : 0) and ties go to the first class, so the class equals that
// of any implementation taking the same steps.  Each hidden unit feeds the
// logits as soon as it is computed; every logit's chain is still in
// ascending j.
//
// Two kernels.  Two classes over int32 features (a predicate or a CASE over the
// class) have k_mlp_predict2, one instance per feature count; everything else
// takes k_mlp_predict, padded to a bound.
#include "tqp_internal.hpp"

namespace tqp {

constexpr int kPredNT = 256;
constexpr int kMaxFeat = 16;
constexpr int kMaxHidden = 64;
constexpr int kMaxClasses = 8;

struct PredArgs {
    const void *feat[kMaxFeat];
    int64_t flen[kMaxFeat];
    int32_t fdt[kMaxFeat];
    int32_t nfeat, hidden, classes;
    const int32_t *rows;
    const float *model;
    int64_t n;
    const int64_t *d_n;
    int8_t *out;
};

// Two classes, F int32 features.  The weights are the same for every row, so
// they are read as scalars and enter the fma's as scalar operands; a thread
// scores kPredR rows, so that each weight read serves as many, and loads all
// their features before the first fma.  No padding and no branch on a type.
//
// What bounds it: at 8 features the columns (32 bytes per scored row; where most
// rows of a table are scored, every line of it), from 16 hidden units and 12
// features on, also the fma's.  16 hidden units, 10M rows, us with k_mlp_predict /
// with this:
//   features                1     3     5     8     9    12    16
//   57% of rows, by id   58/19 60/26 65/36 87/59 142/68 161/90 186/117
//   all rows             86/28 90/38 100/51 123/76 213/86 242/113 282/149
// The same kernel with the counts, types and classes as run-time bounds spends
// more on choosing operands than it saves: 157 us at 8 features and 4 classes,
// where k_mlp_predict takes 86; so it is not used for those.
constexpr int kPredR = 2;

template <int F>
__global__ __launch_bounds__(kPredNT) void k_mlp_predict2(PredArgs a, const float *__restrict__ model,
                                                          int8_t *__restrict__ out) {
    constexpr int R = kPredR;
    const int64_t cnt = count_of(a.d_n, a.n);
    const int H = a.hidden;
    const float *w1 = model, *b1 = w1 + H * F, *w2 = b1 + H, *b2 = w2 + 2 * H;
    const int64_t stride = int64_t(gridDim.x) * kPredNT * R;
    for (int64_t base = blockIdx.x * int64_t(kPredNT) * R; base < cnt; base += stride) {
        int64_t i[R];
        int32_t row[R];
#pragma unroll
        for (int r = 0; r < R; r++) {
            i[r] = base + r * kPredNT + threadIdx.x;
            const int64_t at = i[r] < cnt ? i[r] : cnt - 1;
            row[r] = a.rows ? a.rows[at] : int32_t(at);
        }
        // A row outside a column reads its element 0 and counts as 0.  Columns
        // mostly have one length: the index is made again only where it changes.
        int32_t raw[F][R];
        uint32_t at[R];
        uint32_t out_of = 0;                     // bit k * R + r: row r is outside column k
#pragma unroll
        for (int k = 0; k < F; k++) {
            if (k == 0 || uint32_t(a.flen[k]) != uint32_t(a.flen[k > 0 ? k - 1 : 0])) {
#pragma unroll
                for (int r = 0; r < R; r++) at[r] = uint32_t(row[r]) < uint32_t(a.flen[k]) ? uint32_t(row[r]) : 0u;
            }
#pragma unroll
            for (int r = 0; r < R; r++) {
                out_of |= uint32_t(uint32_t(row[r]) >= uint32_t(a.flen[k])) << (k * R + r);
                raw[k][r] = static_cast<const int32_t *>(a.feat[k])[at[r]];
            }
        }
        float x[F][R];
#pragma unroll
        for (int k = 0; k < F; k++)
#pragma unroll
            for (int r = 0; r < R; r++) x[k][r] = float(raw[k][r]);
        if (__any(out_of != 0)) {
#pragma unroll
            for (int k = 0; k < F; k++)
#pragma unroll
                for (int r = 0; r < R; r++)
                    if ((out_of >> (k * R + r)) & 1) x[k][r] = 0.0f;
        }
        float z[2][R];
#pragma unroll
        for (int c = 0; c < 2; c++)
#pragma unroll
            for (int r = 0; r < R; r++) z[c][r] = b2[c];
#pragma unroll 4
        for (int j = 0; j < H; j++) {
            float h[R];
#pragma unroll
            for (int r = 0; r < R; r++) h[r] = b1[j];
#pragma unroll
            for (int k = 0; k < F; k++) {
                const float w = w1[j * F + k];
#pragma unroll
                for (int r = 0; r < R; r++) h[r] = __builtin_fmaf(w, x[k][r], h[r]);
            }
#pragma unroll
            for (int r = 0; r < R; r++) h[r] = h[r] > 0.0f ? h[r] : 0.0f;
#pragma unroll
            for (int c = 0; c < 2; c++) {
                const float w = w2[c * H + j];
#pragma unroll
                for (int r = 0; r < R; r++) z[c][r] = __builtin_fmaf(w, h[r], z[c][r]);
            }
        }
#pragma unroll
        for (int r = 0; r < R; r++)
            if (i[r] < cnt) out[i[r]] = int8_t(z[1][r] > z[0][r] ? 1 : 0);
    }
}

// The model is copied into LDS once per workgroup, W1 rows padded and W2 stored
// by hidden unit, so a hidden unit's weights come in a few 16-byte broadcast
// reads; the features of a row are loaded together, one aligned word per column.
// FM >= nfeat and CM >= classes are multiples of 4: the weights are padded
// with zeros to those bounds and every multiply-add runs to the bound, with
// no branch.  The padding changes nothing: x[k] = 0 and W1[j][k] = 0 for
// k >= nfeat, so those steps add +0, which leaves a nonzero sum unchanged
// and can only turn a -0 into +0, and relu maps both zeros to 0; logits past
// `classes` are never compared.
template <int FM, int CM>
__global__ __launch_bounds__(kPredNT) void k_mlp_predict(PredArgs a) {
    __shared__ float4 s_w1[kMaxHidden][FM / 4];      // W1[j][k], zero padded
    __shared__ float4 s_w2[kMaxHidden][CM / 4];      // W2[c][j] stored as [j][c]
    __shared__ float s_b1[kMaxHidden];
    __shared__ float s_b2[CM];
    const int64_t cnt = count_of(a.d_n, a.n);
    const int F = a.nfeat, H = a.hidden, C = a.classes;
    {
        const float *m = a.model;
        float *w1 = reinterpret_cast<float *>(s_w1), *w2 = reinterpret_cast<float *>(s_w2);
        for (int i = threadIdx.x; i < kMaxHidden * FM; i += kPredNT) {
            const int j = i / FM, k = i % FM;
            w1[i] = j < H && k < F ? m[j * F + k] : 0.0f;
        }
        for (int i = threadIdx.x; i < kMaxHidden * CM; i += kPredNT) {
            const int j = i / CM, c = i % CM;
            w2[i] = j < H && c < C ? m[H * F + H + c * H + j] : 0.0f;
        }
        for (int i = threadIdx.x; i < kMaxHidden; i += kPredNT) s_b1[i] = i < H ? m[H * F + i] : 0.0f;
        for (int i = threadIdx.x; i < CM; i += kPredNT) s_b2[i] = i < C ? m[H * F + H + C * H + i] : 0.0f;
    }
    __syncthreads();
    const int64_t stride = int64_t(gridDim.x) * kPredNT;
    for (int64_t i = blockIdx.x * int64_t(kPredNT) + threadIdx.x; i < cnt; i += stride) {
        const int64_t r = a.rows ? a.rows[i] : i;
        uint64_t w[FM];
#pragma unroll
        for (int k = 0; k < FM; k++) {
            const bool in = k < F && r >= 0 && r < a.flen[k];
            w[k] = word_of(k < F ? a.feat[k] : a.feat[0], k < F ? dtype_lg(a.fdt[k]) : 0,
                           in ? r : 0);
        }
        float x[FM];
#pragma unroll
        for (int k = 0; k < FM; k++) {
            const bool in = k < F && r >= 0 && r < a.flen[k];
            x[k] = in ? float(sext_of(from_word(w[k], a.feat[k], dtype_lg(a.fdt[k]), r), a.fdt[k]))
                      : 0.0f;
        }
        float z[CM];
#pragma unroll
        for (int c = 0; c < CM; c++) z[c] = s_b2[c];
        for (int j = 0; j < H; j++) {
            float wr[FM], wc[CM];
#pragma unroll
            for (int q = 0; q < FM / 4; q++) {
                const float4 v = s_w1[j][q];
                wr[4 * q] = v.x; wr[4 * q + 1] = v.y; wr[4 * q + 2] = v.z; wr[4 * q + 3] = v.w;
            }
#pragma unroll
            for (int q = 0; q < CM / 4; q++) {
                const float4 v = s_w2[j][q];
                wc[4 * q] = v.x; wc[4 * q + 1] = v.y; wc[4 * q + 2] = v.z; wc[4 * q + 3] = v.w;
            }
            float acc = s_b1[j];
#pragma unroll
            for (int k = 0; k < FM; k++) acc = __builtin_fmaf(wr[k], x[k], acc);
            const float h = acc > 0.0f ? acc : 0.0f;
#pragma unroll
            for (int c = 0; c < CM; c++) z[c] = __builtin_fmaf(wc[c], h, z[c]);
        }
        int arg = 0;
        float best = z[0];
#pragma unroll
        for (int c = 1; c < CM; c++)
            if (c < C && z[c] > best) {
                best = z[c];
                arg = c;
            }
        a.out[i] = int8_t(arg);
    }
}

}  // namespace tqp

using namespace tqp;

TQP_API int tqp_mlp_predict(const tqp_col *feats, int nfeat, const int32_t *rows, int64_t n,
                            const int64_t *d_n, const float *model, int hidden, int classes,
                            int8_t *out, void *stream) {
    clear_error();
    if (!feats || nfeat < 1 || nfeat > kMaxFeat)
        return set_error(TQP_EINVAL, "tqp_mlp_predict: nfeat must be in [1, %d]", kMaxFeat);
    if (hidden < 1 || hidden > kMaxHidden || classes < 1 || classes > kMaxClasses)
        return set_error(TQP_EINVAL, "tqp_mlp_predict: hidden must be in [1, %d], classes in [1, %d]",
                         kMaxHidden, kMaxClasses);
    if (n < 0 || (n > 0 && (!model || !out)))
        return set_error(TQP_EINVAL, "tqp_mlp_predict: need n >= 0, a model and an output");
    if (rows && !col_aligned(rows, TQP_INT32))
        return set_error(TQP_EINVAL, "tqp_mlp_predict: rows must be 4-byte aligned");
    if (!col_aligned(model, TQP_INT32))
        return set_error(TQP_EINVAL, "tqp_mlp_predict: model must be 4-byte aligned");
    PredArgs a = {};
    for (int k = 0; k < nfeat; k++) {
        if (!dtype_ok(feats[k].dtype) || feats[k].len < 0 || (feats[k].len > 0 && !feats[k].data) ||
            !col_aligned(feats[k].data, feats[k].dtype))
            return set_error(TQP_EINVAL, "tqp_mlp_predict: feature %d is invalid or unaligned", k);
        if (!rows && feats[k].len < n)
            return set_error(TQP_EINVAL, "tqp_mlp_predict: feature %d is shorter than n", k);
        // (a stand-in for an empty column: k_mlp_predict2 reads its first element and takes 0 instead)
        a.feat[k] = feats[k].len > 0 ? feats[k].data : model;
        a.flen[k] = feats[k].len;
        a.fdt[k] = feats[k].dtype;
    }
    if (n == 0) return TQP_OK;
    a.nfeat = nfeat;
    a.hidden = hidden;
    a.classes = classes;
    a.rows = rows;
    a.model = model;
    a.n = n;
    a.d_n = d_n;
    a.out = out;
    hipStream_t s = as_stream(stream);
    // row ids and lengths of k_mlp_predict2 are 32-bit
    bool two = classes == 2 && (rows || n <= INT32_MAX);
    for (int k = 0; k < nfeat; k++) two = two && a.fdt[k] == TQP_INT32 && a.flen[k] <= INT64_C(1) << 31;
    if (two) {
        const unsigned g = block_grid(ceil_div(n, int64_t(kPredNT) * kPredR), d_n);
#define TQP_MLP2(F)                                                                                 \
    case F:                                                                                         \
        TQP_LAUNCH("mlp_predict", k_mlp_predict2<F>, dim3(g), dim3(kPredNT), 0, s, a, model, out); \
        break;
        switch (nfeat) {
            TQP_MLP2(1) TQP_MLP2(2) TQP_MLP2(3) TQP_MLP2(4) TQP_MLP2(5) TQP_MLP2(6) TQP_MLP2(7) TQP_MLP2(8)
            TQP_MLP2(9) TQP_MLP2(10) TQP_MLP2(11) TQP_MLP2(12) TQP_MLP2(13) TQP_MLP2(14) TQP_MLP2(15)
            TQP_MLP2(16)
        }
#undef TQP_MLP2
        return check_launch("tqp_mlp_predict");
    }
    int64_t g = ceil_div(n, int64_t(kPredNT) * 4);
    if (g > 8192) g = 8192;
    if (nfeat <= 8 && classes <= 4)
        TQP_LAUNCH("mlp_predict", (k_mlp_predict<8, 4>), dim3(unsigned(g)), dim3(kPredNT), 0, s, a);
    else if (nfeat <= 8)
        TQP_LAUNCH("mlp_predict", (k_mlp_predict<8, 8>), dim3(unsigned(g)), dim3(kPredNT), 0, s, a);
    else if (classes <= 4)
        TQP_LAUNCH("mlp_predict", (k_mlp_predict<16, 4>), dim3(unsigned(g)), dim3(kPredNT), 0, s, a);
    else
        TQP_LAUNCH("mlp_predict", (k_mlp_predict<16, 8>), dim3(unsigned(g)), dim3(kPredNT), 0, s, a);
    return check_launch("tqp_mlp_predict");
}
