// The GraphSAGE layer with the transform before the aggregation (F_out much smaller than F_in): its products (see
// gemm.hip) and the second stage of its weight gradient.
#include "gemm_core.hpp"
#include "reduce_splits.hpp"

namespace tma {

// Split reduction for the transform-first form: partial is [splits][F][2*Fp]; column c of the left half
// goes to dW_self[:, c], of the right half to dW_neigh[:, c]; the column sums of the left half are dbias.
// Columns in groups of four, which never straddle the halves (Fp is a multiple of four); one column per lane asked for a
// quarter of the bytes at a time (256 splits of 256 x 96: 12.0 -> 8.3 us).
__global__ __launch_bounds__(256) void reduce_splits_halves_kernel(const float *__restrict__ partial,
                                                                   const float *__restrict__ colsum_partial,
                                                                   int n_splits, int F, int Fo, int Fp,
                                                                   float *__restrict__ dW_self,
                                                                   float *__restrict__ dW_neigh,
                                                                   float *__restrict__ dbias)
{
    __shared__ float4 part[kRedSlices][kRedCols];
    const int N = 2 * Fp;
    const int64_t total = int64_t(F) * N;
    const int64_t total_all = total + N;
    const int col = threadIdx.x % kRedCols, q = threadIdx.x / kRedCols;
    const int64_t e = (int64_t(blockIdx.x) * kRedCols + col) * 4;
    const int per = (n_splits + kRedSlices - 1) / kRedSlices;
    const int s_begin = q * per, s_end = (s_begin + per < n_splits) ? s_begin + per : n_splits;
    float4 s = zero4();
    if (e < total_all) {
        const float *from = e < total ? partial + e : colsum_partial + (e - total);
        const int64_t step = e < total ? total : N;
#pragma unroll 8
        for (int sp = s_begin; sp < s_end; ++sp) {
            const float4 v = *reinterpret_cast<const float4 *>(from + int64_t(sp) * step);
            s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
        }
    }
    part[q][col] = s;
    __syncthreads();
    if (q == 0 && e < total_all) {
        float r[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int w = 0; w < kRedSlices; ++w) {
            const float4 v = part[w][col];
            r[0] += v.x; r[1] += v.y; r[2] += v.z; r[3] += v.w;
        }
        const bool weight = e < total;
        const int64_t m = weight ? e / N : 0;
        const int c = int(weight ? e - m * N : e - total);
        const bool second = c >= Fp;
        const int cc = c - (second ? Fp : 0);
        float *out = weight ? (second ? dW_neigh : dW_self) + m * Fo : (second ? nullptr : dbias);
        if (out) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (cc + i < Fo) out[cc + i] = r[i];
        }
    }
}

// ---- transform-before-aggregate form -----------------------------------------
static int pad_cols(int32_t F_out, int32_t dtype) { return int(round_up(size_t(F_out), dtype == TMA_BF16 ? 8 : 4)); }


static int tf_fwd_f32(int64_t n, const float *H, int64_t ldh, int32_t F_in, const float *W_self, const float *W_neigh,
                      int32_t F_out, int Fp, float *Ys, float *Yn, int64_t ldy, hipStream_t s)
{
    TMA_REQUIRE(int64_t(F_in) * F_out >= 4, TMA_ERR_INVALID_ARG, "sage gemm tf fwd: weight matrix below four elements");
    launch_fwd_f32("gemm_tf_fwd", AsyncRows(H, ldh, H, ldh, F_in, F_in, n), AsyncWeights<true>{W_self, W_neigh, F_in, F_out, F_in, Fp},
                   HalvesEpilogue<float>{Ys, Yn, ldy, Fp, F_out}, n, 2 * Fp, s);
    return check_launch("sage gemm tf fwd");
}

static int tf_fwd_bf16(int64_t n, const uint16_t *H, int64_t ldh, int32_t F_in, const float *W_self, const float *W_neigh,
                       int32_t F_out, int Fp, uint16_t *Ys, uint16_t *Yn, int64_t ldy, hipStream_t s, void *spare, size_t spare_bytes)
{
    HalvesEpilogue<uint16_t> e{Ys, Yn, ldy, Fp, F_out};
    if (stream_sage_tf_fwd(n, H, ldh, F_in, W_self, W_neigh, F_out, Fp, Ys, Yn, ldy, spare, spare_bytes, s)) return check_launch("sage gemm tf fwd");
    const int64_t K = F_in, kps = int64_t(round_up(size_t(K), 32));
    // The rows are the k side here: a group that reaches into their padding has to mask it (a NaN there would get through
    // the zero weights it meets), which the plain groups do not.
    const bool va = groups_ok(H, ldh, F_in);
    const bool padded = !va && vec4_ok(H, ldh);
    const bool vb = F_out % 4 == 0 && aligned(W_self, 16) && aligned(W_neigh, 16);
    TMA_REQUIRE(vb || int64_t(F_in) * F_out >= 4, TMA_ERR_INVALID_ARG, "sage gemm tf fwd: weight matrix below four elements");
    const char *name = va || padded ? "gemm_tf_fwd_bf16" : "gemm_tf_fwd_bf16_generic";
    // weights whose rows are not multiples of four: 16-byte loads from 4-byte-aligned addresses
    // (the form is only chosen for F_in >= 8, so the matrices hold at least four elements)
    const auto with_rows = [&](const auto &a, auto grouped_tag) {
        const auto with_weights = [&](const auto &b) {
            launch_by_width<uint16_t, 32, false, decltype(grouped_tag)::value>(name, a, b, e, n, 2 * Fp, K, kps, 1, nullptr, s);
        };
        if (vb) with_weights(SideWeights<kAligned4>{W_self, W_neigh, F_in, F_out, Fp});
        else with_weights(SideWeights<kUnaligned4>{W_self, W_neigh, F_in, F_out, Fp});
    };
    if (va) with_rows(CatRows<uint16_t, true>{H, ldh, H, ldh, F_in, n, F_in}, std::true_type{});
    else if (padded) with_rows(PaddedRows{H, ldh, F_in, n}, std::true_type{});
    else with_rows(CatRows<uint16_t, false>{H, ldh, H, ldh, F_in, n, F_in}, std::false_type{});
    return check_launch("sage gemm tf fwd");
}

int launch_sage_tf_gemm_fwd(int64_t n, const void *H, int64_t ldh, int32_t F_in, const float *W_self,
                            const float *W_neigh, int32_t F_out, int32_t dtype, void *Ys, void *Yn, int64_t ldy,
                            hipStream_t stream, void *spare, size_t spare_bytes)
{
    if (n == 0) return TMA_OK;
    const int Fp = pad_cols(F_out, dtype);
    if (dtype == TMA_F32)
        return tf_fwd_f32(n, static_cast<const float *>(H), ldh, F_in, W_self, W_neigh, F_out, Fp,
                                   static_cast<float *>(Ys), static_cast<float *>(Yn), ldy, stream);
    if (dtype == TMA_BF16)
        return tf_fwd_bf16(n, static_cast<const uint16_t *>(H), ldh, F_in, W_self, W_neigh, F_out, Fp,
                                      static_cast<uint16_t *>(Ys), static_cast<uint16_t *>(Yn), ldy, stream, spare, spare_bytes);
    return fail(TMA_ERR_UNSUPPORTED_DTYPE, "sage gemm tf fwd: dtype %d", dtype);
}

static WeightSplit plan_tf_weight_split(int64_t n, int32_t F_in, int Fp)
{
    const int N = 2 * Fp;
    const int bn = N <= 64 ? 64 : (N <= 96 ? 96 : 128);
    const int64_t tiles = ceil_div(int64_t(F_in), 128) * ceil_div(N, bn);
    int64_t want = ceil_div(512, tiles > 0 ? tiles : 1);
    const int64_t max_useful = ceil_div(n > 0 ? n : 1, 128);
    if (want > max_useful) want = max_useful;
    if (want < 1) want = 1;
    WeightSplit w;
    w.k_per_split = int64_t(round_up(size_t(ceil_div(n > 0 ? n : 1, want)), 32));
    w.n_splits = int(ceil_div(n > 0 ? n : 1, w.k_per_split));
    w.partial_bytes = round_up(size_t(w.n_splits) * size_t(F_in) * size_t(N) * 4, 256);
    w.colsum_bytes = round_up(size_t(w.n_splits) * size_t(N) * 4, 256);
    return w;
}

size_t sage_tf_gemm_bwd_weight_workspace_bytes(int64_t n, int32_t F_in, int32_t F_out, int32_t dtype)
{
    const WeightSplit w = plan_tf_weight_split(n, F_in, pad_cols(F_out, dtype));
    return w.partial_bytes + w.colsum_bytes;
}

template <typename T>
static int tf_bwd_weight_typed(int64_t n, const T *H, int64_t ldh, const T *g, const T *h, int64_t ld_next,
                               const T *dYn, int64_t ldy, int32_t F_in, int32_t F_out, int Fp, bool relu,
                               const WeightSplit &w, float *partial, float *colsum, hipStream_t s)
{
    SplitEpilogue e{partial, int64_t(F_in), 2 * Fp};
    const bool va = padded_groups_ok(H, ldh, F_in);
    const bool vb = padded_groups_ok(g, ld_next, F_out) && (!relu || padded_groups_ok(h, ld_next, F_out)) && vec4_ok(dYn, ldy);
    const char *name = kname<T>("gemm_tf_bwd_weight", "gemm_tf_bwd_weight_generic", "gemm_tf_bwd_weight_bf16",
                                "gemm_tf_bwd_weight_bf16_generic", va && vb);
#define TMA_TF_BW(VA_, VB_, R_)                                                                                       \
    do {                                                                                                              \
        CatRowsT<T, VA_> a{H, ldh, H, ldh, F_in, n, F_in};                                                                       \
        SideGrad<false, T, VB_, R_> b{g, h, dYn, F_out, Fp, ld_next, ldy, n};                                         \
        launch_by_width<T, 32, true, VA_ && VB_>(name, a, b, e, int64_t(F_in), 2 * Fp, n, w.k_per_split, w.n_splits, colsum, s);     \
    } while (0)
#define TMA_TF_BW2(VA_, VB_)         \
    do {                             \
        if (relu) TMA_TF_BW(VA_, VB_, true); \
        else TMA_TF_BW(VA_, VB_, false);     \
    } while (0)
    if (va && vb) TMA_TF_BW2(true, true);
    else if constexpr (sizeof(T) == 4) {
        if (vb && rows_u_ok(n, ldh, F_in)) {
            CatRowsTU a{H, ldh, H, ldh, F_in, pad4(F_in), n};
            auto launch = [&](const auto &b) {
                launch_by_width<T, 32, true, true>(name, a, b, e, int64_t(F_in), 2 * Fp, n, w.k_per_split, w.n_splits, colsum, s);
            };
            if (relu) launch(SideGrad<false, T, true, true>{g, h, dYn, F_out, Fp, ld_next, ldy, n});
            else launch(SideGrad<false, T, true, false>{g, h, dYn, F_out, Fp, ld_next, ldy, n});
        } else TMA_TF_BW2(false, false);
    } else if (va) TMA_TF_BW2(true, false);
    else if (vb) TMA_TF_BW2(false, true);
    else TMA_TF_BW2(false, false);
#undef TMA_TF_BW2
#undef TMA_TF_BW
    return check_launch("sage gemm tf bwd weight");
}

int launch_sage_tf_gemm_bwd_weight(int64_t n, const void *H, int64_t ldh, const void *dHnext, const void *Hnext,
                                   int64_t ld_next, const void *dYn, int64_t ldy, int32_t F_in, int32_t F_out,
                                   int32_t act, int32_t dtype, float *dW_self, float *dW_neigh, float *dbias, void *ws,
                                   size_t ws_bytes, hipStream_t stream)
{
    if (dtype != TMA_F32 && dtype != TMA_BF16) return fail(TMA_ERR_UNSUPPORTED_DTYPE, "sage gemm tf bwd: dtype %d", dtype);
    const int Fp = pad_cols(F_out, dtype);
    WeightSplit w = plan_tf_weight_split(n, F_in, Fp);
    if (ws_bytes < w.partial_bytes + w.colsum_bytes)
        return fail(TMA_ERR_WORKSPACE_TOO_SMALL, "sage gemm tf bwd weight: workspace %zu < %zu", ws_bytes,
                    w.partial_bytes + w.colsum_bytes);
    float *partial = static_cast<float *>(ws);
    float *colsum = reinterpret_cast<float *>(static_cast<char *>(ws) + w.partial_bytes);
    const bool relu = act == TMA_ACT_RELU;
    int rc = TMA_OK;
    if (n == 0) {
        // no rows: nothing to multiply (operands may be NULL); the second stage writes the zero gradients
    } else if (dtype == TMA_BF16 && !relu &&
               stream_sage_tf_bwd_weight(n, static_cast<const uint16_t *>(H), ldh, static_cast<const uint16_t *>(dHnext), ld_next,
                                         static_cast<const uint16_t *>(dYn), ldy, F_in, F_out, Fp, w, partial, colsum, stream)) {
        rc = check_launch("sage gemm tf bwd weight");
    } else if (dtype == TMA_F32)
        rc = tf_bwd_weight_typed<float>(n, static_cast<const float *>(H), ldh, static_cast<const float *>(dHnext),
                                        static_cast<const float *>(Hnext), ld_next, static_cast<const float *>(dYn),
                                        ldy, F_in, F_out, Fp, relu, w, partial, colsum, stream);
    else
        rc = tf_bwd_weight_typed<uint16_t>(n, static_cast<const uint16_t *>(H), ldh,
                                           static_cast<const uint16_t *>(dHnext),
                                           static_cast<const uint16_t *>(Hnext), ld_next,
                                           static_cast<const uint16_t *>(dYn), ldy, F_in, F_out, Fp, relu, w, partial,
                                           colsum, stream);
    if (rc) return rc;
    const int64_t total_all = int64_t(F_in) * 2 * Fp + 2 * Fp;
    TMA_TIMED("reduce_splits_halves", stream);
    hipLaunchKernelGGL(reduce_splits_halves_kernel, dim3(unsigned(ceil_div(total_all, 4 * kRedCols))), dim3(256), 0, stream,
                       partial, colsum, n > 0 ? w.n_splits : 0, F_in, F_out, Fp, dW_self, dW_neigh, dbias);
    return check_launch("sage gemm tf bwd weight reduce");
}

template <typename T>
static int tf_bwd_data_typed(int64_t n, const T *g, const T *h, int64_t ld_next, const T *dYn, int64_t ldy,
                             const float *W_self, const float *W_neigh, int32_t F_in, int32_t F_out, int Fp, bool relu,
                             T *dH, int64_t ldh, hipStream_t s)
{
    RowsEpilogue<T> e{dH, ldh};
    const int64_t K = 2 * int64_t(Fp), kps = int64_t(round_up(size_t(K), 32));
    const bool va = padded_groups_ok(g, ld_next, F_out) && (!relu || padded_groups_ok(h, ld_next, F_out)) && vec4_ok(dYn, ldy);
    const bool vb = F_out % 4 == 0 && aligned(W_self, 16) && aligned(W_neigh, 16);
    TMA_REQUIRE(vb || int64_t(F_in) * F_out >= 4, TMA_ERR_INVALID_ARG, "sage gemm tf bwd data: weight matrix below four elements");
    const char *name = kname<T>("gemm_tf_bwd_data", "gemm_tf_bwd_data_generic", "gemm_tf_bwd_data_bf16",
                                "gemm_tf_bwd_data_bf16_generic", va);
#define TMA_TF_BD(VA_, VB_, R_)                                                                        \
    do {                                                                                               \
        SideGrad<true, T, VA_, R_> a{g, h, dYn, F_out, Fp, ld_next, ldy, n};                           \
        SideWeightsT<VB_> b{W_self, W_neigh, F_in, F_out, Fp};                                         \
        if constexpr (sizeof(T) == 4) launch_split<false, VA_>(name, a, b, e, n, F_in, K, kps, 1, nullptr, s); \
        else launch_gemm<128, 128, 32, 2, 2, false, T>(name, a, b, e, n, F_in, K, kps, 1, nullptr, s); \
    } while (0)
#define TMA_TF_BD2(VA_, VB_)                 \
    do {                                     \
        if (relu) TMA_TF_BD(VA_, VB_, true); \
        else TMA_TF_BD(VA_, VB_, false);     \
    } while (0)
    if (va && vb) TMA_TF_BD2(true, kAligned4);
    else if (va) TMA_TF_BD2(true, kUnaligned4);
    else if (vb) TMA_TF_BD2(false, kAligned4);
    else TMA_TF_BD2(false, kUnaligned4);
#undef TMA_TF_BD2
#undef TMA_TF_BD
    return check_launch("sage gemm tf bwd data");
}

int launch_sage_tf_gemm_bwd_data(int64_t n, const void *dHnext, const void *Hnext, int64_t ld_next, const void *dYn,
                                 int64_t ldy, const float *W_self, const float *W_neigh, int32_t F_in, int32_t F_out,
                                 int32_t act, int32_t dtype, void *dH, int64_t ldh, hipStream_t stream, void *spare, size_t spare_bytes)
{
    if (n == 0) return TMA_OK;
    const int Fp = pad_cols(F_out, dtype);
    const bool relu = act == TMA_ACT_RELU;
    if (dtype == TMA_BF16 && !relu && stream_sage_tf_bwd_data(n, static_cast<const uint16_t *>(dHnext), ld_next, static_cast<const uint16_t *>(dYn), ldy,
                                                              W_self, W_neigh, F_in, F_out, Fp, static_cast<uint16_t *>(dH), ldh, spare, spare_bytes,
                                                              stream))
        return check_launch("sage gemm tf bwd data");
    if (dtype == TMA_F32)
        return tf_bwd_data_typed<float>(n, static_cast<const float *>(dHnext), static_cast<const float *>(Hnext),
                                        ld_next, static_cast<const float *>(dYn), ldy, W_self, W_neigh, F_in, F_out, Fp,
                                        relu, static_cast<float *>(dH), ldh, stream);
    if (dtype == TMA_BF16)
        return tf_bwd_data_typed<uint16_t>(n, static_cast<const uint16_t *>(dHnext),
                                           static_cast<const uint16_t *>(Hnext), ld_next,
                                           static_cast<const uint16_t *>(dYn), ldy, W_self, W_neigh, F_in, F_out, Fp,
                                           relu, static_cast<uint16_t *>(dH), ldh, stream);
    return fail(TMA_ERR_UNSUPPORTED_DTYPE, "sage gemm tf bwd data: dtype %d", dtype);
}

}  // namespace tma
