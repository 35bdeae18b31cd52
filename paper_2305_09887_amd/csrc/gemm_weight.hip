// Weight gradients of the GraphSAGE layer, [dW_self ; dW_neigh] = [H | M]^T dZ and db = 1^T dZ: split planning, the
// products (see gemm.hip) and their fixed-order second stage, which the other layers' weight gradients share.
#include "gemm_core.hpp"
#include "reduce_splits.hpp"

namespace tma {

__global__ __launch_bounds__(256) void reduce_splits_kernel(const float *__restrict__ partial,
                                                            const float *__restrict__ colsum_partial, int n_splits,
                                                            int F, int N, int halves, float *__restrict__ dW_self,
                                                            float *__restrict__ dW_neigh, float *__restrict__ dbias)
{
    __shared__ float4 part[kRedSlices][kRedCols];
    const int64_t total = int64_t(halves) * F * N;      // weight-gradient entries; then N bias entries
    const int64_t total_all = total + N;
    const int col = threadIdx.x % kRedCols, q = threadIdx.x / kRedCols;
    const int64_t e0 = (int64_t(blockIdx.x) * kRedCols + col) * 4;
    const int per = (n_splits + kRedSlices - 1) / kRedSlices;
    const int s_begin = q * per, s_end = (s_begin + per < n_splits) ? s_begin + per : n_splits;
    float4 s = zero4();
    if (e0 < total_all) {
        const bool vec = (e0 + 3 < total) && (total % 4 == 0);
        if (vec) {
#pragma unroll 8
            for (int sp = s_begin; sp < s_end; ++sp) {
                const float4 v = *reinterpret_cast<const float4 *>(partial + int64_t(sp) * total + e0);
                s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
            }
        } else {
            float t[4] = {0.0f, 0.0f, 0.0f, 0.0f};
            for (int sp = s_begin; sp < s_end; ++sp)
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const int64_t e = e0 + c;
                    if (e < total) t[c] += partial[int64_t(sp) * total + e];
                    else if (e < total_all) t[c] += colsum_partial[int64_t(sp) * N + (e - total)];
                }
            s = make_float4(t[0], t[1], t[2], t[3]);
        }
    }
    part[q][col] = s;
    __syncthreads();
    if (q == 0 && e0 < total_all) {
        float r[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int w = 0; w < kRedSlices; ++w) {
            const float4 v = part[w][col];
            r[0] += v.x; r[1] += v.y; r[2] += v.z; r[3] += v.w;
        }
        const int64_t half = int64_t(F) * N;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int64_t e = e0 + c;
            if (e < half) dW_self[e] = r[c];
            else if (e < total) dW_neigh[e - half] = r[c];
            else if (e < total_all && dbias) dbias[e - total] = r[c];
        }
    }
}

int launch_reduce_splits(const float *partial, const float *colsum_partial, int n_splits, int32_t F, int32_t N,
                         int halves, float *dW_first, float *dW_second, float *dbias, hipStream_t stream)
{
    const int64_t total_all = int64_t(halves) * F * N + N;
    TMA_TIMED("reduce_splits", stream);
    hipLaunchKernelGGL(reduce_splits_kernel, dim3(unsigned(ceil_div(total_all, 4 * kRedCols))), dim3(256), 0, stream,
                       partial, colsum_partial, n_splits, F, N, halves, dW_first, dW_second, dbias);
    return check_launch("split reduce");
}

// ---- backward: weights ------------------------------------------------------

static int64_t wanted_ranges(int64_t n, int32_t F_in, int32_t F_out)
{
    const int64_t tiles = ceil_div(2 * int64_t(F_in), 128) * ceil_div(F_out, F_out <= 64 ? 64 : 128);
    int64_t want = ceil_div(512, tiles > 0 ? tiles : 1);
    const int64_t max_useful = ceil_div(n > 0 ? n : 1, 128);
    if (want > max_useful) want = max_useful;
    return want < 1 ? 1 : want;
}

static WeightSplit plan_weight_split(int64_t n, int32_t F_in, int32_t F_out)
{
    const int64_t want = wanted_ranges(n, F_in, F_out);
    WeightSplit w;
    w.k_per_split = int64_t(round_up(size_t(ceil_div(n > 0 ? n : 1, want)), 32));
    w.n_splits = int(ceil_div(n > 0 ? n : 1, w.k_per_split));
    w.partial_bytes = round_up(size_t(w.n_splits) * 2 * size_t(F_in) * size_t(F_out) * 4, 256);
    w.colsum_bytes = round_up(size_t(w.n_splits) * size_t(F_out) * 4, 256);
    return w;
}

// least: what a call needs; else what is asked for: room for the ranges before they are rounded to 32 rows, which never shrinks with more rows (what a
// trainer on blocks reserves for its most rows holds for every batch), and for what the streamed product makes use of
size_t sage_gemm_bwd_weight_workspace_bytes(int64_t n, int32_t F_in, int32_t F_out, int32_t dtype, bool least)
{
    if (least) {
        const WeightSplit w = plan_weight_split(n, F_in, F_out);
        return w.partial_bytes + w.colsum_bytes;
    }
    const size_t want = size_t(wanted_ranges(n, F_in, F_out));
    size_t bytes = round_up(want * 2 * size_t(F_in) * size_t(F_out) * 4, 256) + round_up(want * size_t(F_out) * 4, 256);
    WeightSplit u;
    if (dtype == TMA_BF16 && plan_stream_weight(n, F_in, F_out, SIZE_MAX, u) && u.partial_bytes + u.colsum_bytes > bytes) bytes = u.partial_bytes + u.colsum_bytes;
    return bytes;
}

template <typename T, bool V, class AView, class BView, class Epi>
static void bwd_weight_launch(const AView &a, const BView &b, const Epi &e, int64_t Mtot, int F_in, int F_out, int64_t n,
                              const WeightSplit &w, float *colsum, hipStream_t s)
{
    if constexpr (sizeof(T) == 4)
        launch_split<true, V>(F_out <= 64 ? (V ? "gemm_bwd_weight_128x64" : "gemm_bwd_weight_128x64_generic")
                                          : (V ? "gemm_bwd_weight_128x128" : "gemm_bwd_weight_128x128_generic"),
                              a, b, e, Mtot, F_out, n, w.k_per_split, w.n_splits, colsum, s);
    else if (F_out <= 64)
        launch_gemm<128, 64, 32, 4, 1, true, T>(V ? "gemm_bwd_weight_128x64_bf16" : "gemm_bwd_weight_128x64_bf16_generic", a, b, e,
                                                Mtot, F_out, n, w.k_per_split, w.n_splits, colsum, s);
    else
        launch_gemm<128, 128, 32, 2, 2, true, T>(V ? "gemm_bwd_weight_128x128_bf16" : "gemm_bwd_weight_128x128_bf16_generic", a, b, e,
                                                 Mtot, F_out, n, w.k_per_split, w.n_splits, colsum, s);
}

template <typename T, bool VA, bool VB, bool kRelu>
static void bwd_weight_dispatch(int64_t n, const T *H, int64_t ldh, const T *M, int64_t ldm, const T *g, const T *h,
                                int64_t ld_next, int F_in, int F_out, const WeightSplit &w, const SplitEpilogue &e,
                                float *colsum, hipStream_t s)
{
    MaskedGrad<false, T, VB, kRelu> b{g, h, F_out, ld_next, n};
    if constexpr (sizeof(T) == 4 && VB && !VA) {   // F_in is no multiple of four
        CatRowsTU a{H, ldh, M, ldm, F_in, pad4(F_in), n};
        bwd_weight_launch<T, true>(a, b, SplitEpiloguePad{e.partial, F_in, pad4(F_in), F_out}, 2 * int64_t(pad4(F_in)), F_in,
                                   F_out, n, w, colsum, s);
    } else {
        CatRowsT<T, VA> a{H, ldh, M, ldm, F_in, n, 2 * F_in};
        bwd_weight_launch<T, VA && VB>(a, b, e, 2 * int64_t(F_in), F_in, F_out, n, w, colsum, s);
    }
}

template <typename T>
static int bwd_weight_typed(int64_t n, const T *H, int64_t ldh, const T *M, int64_t ldm, const T *g, const T *h, int64_t ld_next,
                            int32_t F_in, int32_t F_out, int32_t act, const WeightSplit &w, const SplitEpilogue &e,
                            float *colsum, hipStream_t stream)
{
    const bool relu = act == TMA_ACT_RELU;
    const bool va = groups_ok(H, ldh, F_in) && groups_ok(M, ldm, F_in);
    const bool vb = padded_groups_ok(g, ld_next, F_out) && (!relu || padded_groups_ok(h, ld_next, F_out));
    const bool small = sizeof(T) == 4 && !va && (!rows_u_ok(n, ldh, F_in) || !rows_u_ok(n, ldm, F_in));
#define TMA_BWD_WEIGHT(VA_, VB_)                                                                                           \
    (relu ? bwd_weight_dispatch<T, VA_, VB_, true>(n, H, ldh, M, ldm, g, h, ld_next, F_in, F_out, w, e, colsum, stream)         \
          : bwd_weight_dispatch<T, VA_, VB_, false>(n, H, ldh, M, ldm, g, h, ld_next, F_in, F_out, w, e, colsum, stream))
    if (va && vb) {
        TMA_BWD_WEIGHT(true, true);
        return check_launch("sage gemm bwd weight");
    }
    if constexpr (sizeof(T) == 2)
        if (va) {
            TMA_BWD_WEIGHT(true, false);
            return check_launch("sage gemm bwd weight");
        }
    if (vb && !small) TMA_BWD_WEIGHT(false, true);
    else TMA_BWD_WEIGHT(false, false);
#undef TMA_BWD_WEIGHT
    return check_launch("sage gemm bwd weight");
}

int launch_sage_gemm_bwd_weight(int64_t n, const void *H, int64_t ldh, const void *M, int64_t ldm, const void *dHnext,
                                const void *Hnext, int64_t ld_next, int32_t F_in, int32_t F_out, int32_t act,
                                int32_t dtype, float *dW_self, float *dW_neigh, float *dbias, void *ws, size_t ws_bytes,
                                hipStream_t stream)
{
    if (dtype != TMA_F32 && dtype != TMA_BF16) return fail(TMA_ERR_UNSUPPORTED_DTYPE, "sage gemm bwd: dtype %d", dtype);
    if (F_out == 0) return TMA_OK;
    const bool relu_ = act == TMA_ACT_RELU;
    const WeightSplit w = plan_weight_split(n, F_in, F_out);
    if (ws_bytes < w.partial_bytes + w.colsum_bytes)
        return fail(TMA_ERR_WORKSPACE_TOO_SMALL, "sage gemm bwd weight: workspace %zu < %zu", ws_bytes,
                    w.partial_bytes + w.colsum_bytes);
    float *partial = static_cast<float *>(ws);
    float *colsum = reinterpret_cast<float *>(static_cast<char *>(ws) + w.partial_bytes);
    const int64_t Mtot = 2 * int64_t(F_in);
    SplitEpilogue e{partial, Mtot, F_out};
    // An empty node set leaves nothing to multiply: the operands may then be NULL, and the kernel's clamped
    // loads would have no valid row to fall back to.  The second stage alone writes the zero gradients.
    const bool have_rows = F_in > 0 && n > 0;
    WeightSplit u;
    if (dtype == TMA_BF16 && have_rows && plan_stream_weight(n, F_in, F_out, ws_bytes, u)) {
        colsum = reinterpret_cast<float *>(static_cast<char *>(ws) + u.partial_bytes);
        if (stream_sage_bwd_weight(n, static_cast<const uint16_t *>(H), ldh, static_cast<const uint16_t *>(M), ldm, static_cast<const uint16_t *>(dHnext),
                                   static_cast<const uint16_t *>(Hnext), ld_next, F_in, F_out, relu_, u, partial, colsum, stream)) {
            if (int rc = check_launch("sage gemm bwd weight")) return rc;
            return launch_reduce_splits(partial, colsum, u.n_splits, F_in, F_out, 2, dW_self, dW_neigh, dbias, stream);
        }
        colsum = reinterpret_cast<float *>(static_cast<char *>(ws) + w.partial_bytes);
    }
    if (have_rows) {
        int rc;
        if (dtype == TMA_F32)
            rc = bwd_weight_typed<float>(n, static_cast<const float *>(H), ldh, static_cast<const float *>(M), ldm,
                                         static_cast<const float *>(dHnext), static_cast<const float *>(Hnext), ld_next,
                                         F_in, F_out, act, w, e, colsum, stream);
        else
            rc = bwd_weight_typed<uint16_t>(n, static_cast<const uint16_t *>(H), ldh, static_cast<const uint16_t *>(M), ldm,
                                            static_cast<const uint16_t *>(dHnext),
                                            static_cast<const uint16_t *>(Hnext), ld_next, F_in, F_out, act, w, e,
                                            colsum, stream);
        if (rc) return rc;
    }
    return launch_reduce_splits(partial, colsum, have_rows ? w.n_splits : 0, F_in, F_out, 2, dW_self, dW_neigh, dbias,
                                stream);
}

}  // namespace tma
