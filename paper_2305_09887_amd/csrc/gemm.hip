// Dense per-layer transform of the mean-aggregation GraphSAGE layer and its
// gradients, on the matrix cores (the only MFMA-bound part of the path):
//   forward   Z = [H | M] [W_self ; W_neigh] + b,  H' = act(Z)
//   backward  [dH_self | D^-1 dM] = dZ [W_self^T | W_neigh^T]
//             [dW_self ; dW_neigh] = [H | M]^T dZ,   db = 1^T dZ     (gemm_weight.hip)
// with dZ = dH' (.) act'(Z) formed while loading (chain rule as in the proof of
// the paper's Thm. 1).  The transform-first form of the layer is in gemm_tf.hip.
//
// The products run in the tile kernels of gemm_core.hpp (fp32 storage: forward on the fp32 matrix instruction, backward
// as fp32-accurate products from bf16 parts; bf16 storage: bf16 MFMA with fp32 accumulation); these files hold the
// operand / epilogue combinations of the GraphSAGE layer.
#include "gemm_core.hpp"

namespace tma {

// ---- forward (fp32: launch_fwd_f32; these: bf16 storage) ----------------------
template <bool VA, class AL, class BL>
static void fwd_launch(const AL &a, const BL &b, const FwdEpilogue<uint16_t> &e, int64_t n, int F_out, int64_t K, int64_t kps,
                       hipStream_t s)
{
    const bool narrow = F_out <= 64 || few_tiles(n, F_out);
    if (few_rows_narrow(n, n, F_out, 1, 128, narrow ? 64 : VA && F_out > 128 && F_out <= 256 ? 256 : 128, 120))
        launch_gemm<64, 64, 32, 2, 2, false, uint16_t, 3>(VA ? "gemm_fwd_64x64_bf16" : "gemm_fwd_64x64_bf16_generic", a, b, e, n, F_out, K, kps, 1, nullptr, s);
    else if (narrow)
        launch_gemm<128, 64, 32, 4, 1, false, uint16_t>(VA ? "gemm_fwd_128x64_bf16" : "gemm_fwd_128x64_bf16_generic", a, b, e, n, F_out, K,
                                                 kps, 1, nullptr, s);
    else if constexpr (VA) {
        // the product is bound by streaming [H | M]; a tile as wide as the output reads it once
        if (F_out > 128 && F_out <= 256)
            launch_gemm<128, 256, 32, 2, 4, false, uint16_t>("gemm_fwd_128x256_bf16", a, b, e, n, F_out, K, kps, 1, nullptr, s);
        else if (std::is_same<BL, CatWeights<true>>::value && K % 32 != 0) {
            if constexpr (std::is_same<BL, CatWeights<true>>::value)
                launch_gemm<128, 128, 32, 2, 2, false, uint16_t>("gemm_fwd_128x128_bf16", a, CatWeightsRest{b}, e, n, F_out, K, kps, 1, nullptr, s);
        } else
            launch_gemm<128, 128, 32, 2, 2, false, uint16_t>("gemm_fwd_128x128_bf16", a, b, e, n, F_out, K, kps, 1, nullptr, s);
    } else
        launch_gemm<128, 128, 32, 2, 2, false, uint16_t>("gemm_fwd_128x128_bf16_generic", a, b, e, n, F_out, K, kps, 1, nullptr, s);
}

template <bool VA, bool VB>
static void fwd_dispatch(int64_t n, const uint16_t *H, int64_t ldh, const uint16_t *M, int64_t ldm, int F_in, const float *W_self,
                         const float *W_neigh, const FwdEpilogue<uint16_t> &e, int F_out, hipStream_t s)
{
    CatRows<uint16_t, VA> a{H, ldh, M, ldm, F_in, n, 2 * F_in};
    const int64_t K = 2 * int64_t(F_in);
    const int64_t kps = int64_t(round_up(size_t(K), 32));
    CatWeights<VB> b{W_self, W_neigh, F_in, F_out};
    fwd_launch<VA>(a, b, e, n, F_out, K, kps, s);
}

// bf16 storage with the weights prepared as Wt[o][k] (bf16): both operands are rows of packed bf16, contiguous
// along k, and go into LDS as loaded -- no conversion, no 2-byte fragment reads of a [k][n] weight tile.
static void fwd_prepared(int64_t n, const uint16_t *H, int64_t ldh, const uint16_t *M, int64_t ldm, int F_in,
                         const uint16_t *Wt, const FwdEpilogue<uint16_t> &e, int F_out, hipStream_t s)
{
    CatRows<uint16_t, true> a{H, ldh, M, ldm, F_in, n, 2 * F_in};
    CatRows<uint16_t, true> b{Wt, 2 * int64_t(F_in), Wt, 2 * int64_t(F_in), 2 * F_in, F_out, 2 * F_in};
    const int64_t K = 2 * int64_t(F_in);
    fwd_launch<true>(a, b, e, n, F_out, K, int64_t(round_up(size_t(K), 32)), s);
}

__global__ __launch_bounds__(256) void narrow_transpose_weights_kernel(const float *__restrict__ Ws,
                                                                       const float *__restrict__ Wn, int F, int N,
                                                                       uint16_t *__restrict__ Wt)
{
    const int64_t idx = int64_t(blockIdx.x) * 256 + threadIdx.x;   // over [2F][N]: coalesced reads
    if (idx >= 2 * int64_t(F) * N) return;
    const int k = int(idx / N), o = int(idx - int64_t(k) * N);
    const float v = k < F ? Ws[int64_t(k) * N + o] : Wn[int64_t(k - F) * N + o];
    Wt[int64_t(o) * 2 * F + k] = f32_to_bf16(v);
}

size_t sage_weights_bf16_bytes(int32_t F_in, int32_t F_out)
{
    return round_up(2 * size_t(F_in) * size_t(F_out) * sizeof(uint16_t), 256);
}

int launch_sage_prepare_weights_bf16(const float *W_self, const float *W_neigh, int32_t F_in, int32_t F_out, void *Wt_out,
                                     hipStream_t stream)
{
    const int64_t total = 2 * int64_t(F_in) * F_out;
    TMA_TIMED("prepare_weights_bf16", stream);
    hipLaunchKernelGGL(narrow_transpose_weights_kernel, dim3(unsigned(ceil_div(total, 256))), dim3(256), 0, stream, W_self,
                       W_neigh, F_in, F_out, static_cast<uint16_t *>(Wt_out));
    return check_launch("prepare weights");
}

static int fwd_f32(int64_t n, const float *H, int64_t ldh, const float *M, int64_t ldm, int32_t F_in, const float *W_self,
                   const float *W_neigh, const float *bias, int32_t F_out, int32_t act, float *Hnext, int64_t ld_next,
                   hipStream_t stream)
{
    launch_fwd_f32(F_out <= 64 || few_tiles(n, F_out) ? "gemm_fwd_128x64" : "gemm_fwd_128x128",   // (the name of its size class)
                   AsyncRows(H, ldh, M, ldm, F_in, 2 * F_in, n), AsyncWeights<false>{W_self, W_neigh, F_in, F_out, 2 * F_in, 0},
                   FwdEpilogue<float>{Hnext, ld_next, bias, act == TMA_ACT_RELU}, n, F_out, stream);
    return check_launch("sage gemm fwd");
}

static int fwd_bf16(int64_t n, const uint16_t *H, int64_t ldh, const uint16_t *M, int64_t ldm, int32_t F_in, const float *W_self,
                    const float *W_neigh, const float *bias, int32_t F_out, int32_t act, uint16_t *Hnext, int64_t ld_next,
                    hipStream_t stream)
{
    FwdEpilogue<uint16_t> e{Hnext, ld_next, bias, act == TMA_ACT_RELU};
    const bool va = vec4_ok(H, ldh) && vec4_ok(M, ldm) && F_in % 4 == 0;
    const bool vb = vec4_ok(W_self, F_out) && vec4_ok(W_neigh, F_out);
    if (va && vb) fwd_dispatch<true, true>(n, H, ldh, M, ldm, F_in, W_self, W_neigh, e, F_out, stream);
    else if (va) fwd_dispatch<true, false>(n, H, ldh, M, ldm, F_in, W_self, W_neigh, e, F_out, stream);
    else if (vb) fwd_dispatch<false, true>(n, H, ldh, M, ldm, F_in, W_self, W_neigh, e, F_out, stream);
    else fwd_dispatch<false, false>(n, H, ldh, M, ldm, F_in, W_self, W_neigh, e, F_out, stream);
    return check_launch("sage gemm fwd");
}

int launch_sage_gemm_fwd(int64_t n, const void *H, int64_t ldh, const void *M, int64_t ldm, int32_t F_in, const float *W_self,
                         const float *W_neigh, const float *bias, int32_t F_out, int32_t act, int32_t dtype,
                         void *Hnext, int64_t ld_next, hipStream_t stream, const void *Wt_bf16)
{
    if (n == 0 || F_out == 0) return TMA_OK;
    if (Wt_bf16 && dtype == TMA_BF16) {
        const uint16_t *h = static_cast<const uint16_t *>(H), *m = static_cast<const uint16_t *>(M);
        if (stream_sage_fwd(n, h, ldh, m, ldm, F_in, static_cast<const uint16_t *>(Wt_bf16), bias, F_out, act == TMA_ACT_RELU,
                            static_cast<uint16_t *>(Hnext), ld_next, stream))
            return check_launch("sage gemm fwd");
        // the packed path needs groups of four bf16 at 8-byte aligned addresses in both operands
        if (vec4_ok(h, ldh) && vec4_ok(m, ldm) && F_in % 4 == 0 && aligned(Wt_bf16, 8)) {
            FwdEpilogue<uint16_t> e{static_cast<uint16_t *>(Hnext), ld_next, bias, act == TMA_ACT_RELU};
            fwd_prepared(n, h, ldh, m, ldm, F_in, static_cast<const uint16_t *>(Wt_bf16), e, F_out, stream);
            return check_launch("sage gemm fwd");
        }
    }
    if (dtype == TMA_F32)
        return fwd_f32(n, static_cast<const float *>(H), ldh, static_cast<const float *>(M), ldm, F_in, W_self,
                                W_neigh, bias, F_out, act, static_cast<float *>(Hnext), ld_next, stream);
    if (dtype == TMA_BF16)
        return fwd_bf16(n, static_cast<const uint16_t *>(H), ldh, static_cast<const uint16_t *>(M), ldm, F_in,
                                   W_self, W_neigh, bias, F_out, act, static_cast<uint16_t *>(Hnext), ld_next, stream);
    return fail(TMA_ERR_UNSUPPORTED_DTYPE, "sage gemm fwd: dtype %d", dtype);
}

// ---- backward: data ---------------------------------------------------------
// BView: CatWeightsT<true / false>, or CatWeightsTU (fp32, F_out no multiple of four)
template <typename T, bool VA, class BView, bool kRelu>
static void bwd_data_dispatch(int64_t n, const T *g, const T *h, int64_t ld_next, const float *W_self,
                              const float *W_neigh, int F_in, int F_out, const BwdDataEpilogue<T> &e, hipStream_t s)
{
    MaskedGrad<true, T, VA, kRelu> a{g, h, F_out, ld_next, n};
    BView b{W_self, W_neigh, F_in, F_out};
    const int N = 2 * F_in;
    const int64_t K = F_out;
    const char *name = kname<T>("gemm_bwd_data_128x128", "gemm_bwd_data_128x128_generic", "gemm_bwd_data_128x128_bf16",
                                "gemm_bwd_data_128x128_bf16_generic", VA);
    const char *narrow = kname<T>("gemm_bwd_data_128x64", "gemm_bwd_data_128x64_generic", "gemm_bwd_data_128x64_bf16",
                                  "gemm_bwd_data_128x64_bf16_generic", VA);
    if constexpr (sizeof(T) == 4) {
        launch_split<false, VA>(few_tiles(n, N) ? narrow : name, a, b, e, n, N, K, K, 1, nullptr, s);
    } else if (few_tiles(n, N)) {
        launch_gemm<128, 64, 32, 4, 1, false, T>(narrow, a, b, e, n, N, K, int64_t(round_up(size_t(K), 32)), 1, nullptr, s);
    } else if (VA && N >= 256 && K > 48) {
        if constexpr (VA)   // half as many passes over the gradient rows
            launch_gemm<128, 256, 32, 2, 4, false, T>("gemm_bwd_data_128x256_bf16", a, b, e, n, N, K,
                                                      int64_t(round_up(size_t(K), 32)), 1, nullptr, s);
    } else if (K <= 48) {  // short reduction: 16-wide slabs waste less of the last one
        const int64_t kps = int64_t(round_up(size_t(K), 16));
        launch_gemm<128, 128, 16, 2, 2, false, T>(name, a, b, e, n, N, K, kps, 1, nullptr, s);
    } else {
        const int64_t kps = int64_t(round_up(size_t(K), 32));
        launch_gemm<128, 128, 32, 2, 2, false, T>(name, a, b, e, n, N, K, kps, 1, nullptr, s);
    }
}

template <typename T>
static int bwd_data_typed(int64_t n, const T *g, const T *h, int64_t ld_next, const float *inv_deg,
                          const float *W_self, const float *W_neigh, int32_t F_in, int32_t F_out, int32_t act,
                          T *dH_self_out, int64_t ldh, T *dM_scaled_out, hipStream_t stream)
{
    const bool relu = act == TMA_ACT_RELU;
    BwdDataEpilogue<T> e{dH_self_out, ldh, dM_scaled_out, inv_deg, F_in};
    const bool va = padded_groups_ok(g, ld_next, F_out) && (!relu || padded_groups_ok(h, ld_next, F_out));
#define TMA_BWD_DATA(VA_, BView_)                                                                                 \
    (relu ? bwd_data_dispatch<T, VA_, BView_, true>(n, g, h, ld_next, W_self, W_neigh, F_in, F_out, e, stream)    \
          : bwd_data_dispatch<T, VA_, BView_, false>(n, g, h, ld_next, W_self, W_neigh, F_in, F_out, e, stream))
    if constexpr (sizeof(T) == 4) {
        if (va && F_out % 4 == 0) TMA_BWD_DATA(true, CatWeightsT<true>);
        else if (va && weights_u_ok(F_in, F_out)) TMA_BWD_DATA(true, CatWeightsTU);
        else TMA_BWD_DATA(false, CatWeightsT<false>);
    } else {
        const bool vb = vec4_ok(W_self, F_out) && vec4_ok(W_neigh, F_out);
        if (va && vb) TMA_BWD_DATA(true, CatWeightsT<true>);
        else if (va) TMA_BWD_DATA(true, CatWeightsT<false>);
        else if (vb) TMA_BWD_DATA(false, CatWeightsT<true>);
        else TMA_BWD_DATA(false, CatWeightsT<false>);
    }
#undef TMA_BWD_DATA
    return check_launch("sage gemm bwd data");
}

int launch_sage_gemm_bwd_data(int64_t n, const void *dHnext, const void *Hnext, int64_t ld_next,
                              const float *inv_deg, const float *W_self, const float *W_neigh, int32_t F_in,
                              int32_t F_out, int32_t act, int32_t dtype, void *dH_self_out, int64_t ldh,
                              void *dM_scaled_out, hipStream_t stream, void *spare, size_t spare_bytes)
{
    if (n == 0 || F_in == 0) return TMA_OK;
    if (dtype == TMA_BF16 && stream_sage_bwd_data(n, static_cast<const uint16_t *>(dHnext), static_cast<const uint16_t *>(Hnext), ld_next, inv_deg,
                                                  W_self, W_neigh, F_in, F_out, act == TMA_ACT_RELU, static_cast<uint16_t *>(dH_self_out), ldh,
                                                  static_cast<uint16_t *>(dM_scaled_out), spare, spare_bytes, stream))
        return check_launch("sage gemm bwd data");
    if (dtype == TMA_F32)
        return bwd_data_typed<float>(n, static_cast<const float *>(dHnext), static_cast<const float *>(Hnext), ld_next,
                                     inv_deg, W_self, W_neigh, F_in, F_out, act, static_cast<float *>(dH_self_out),
                                     ldh, static_cast<float *>(dM_scaled_out), stream);
    if (dtype == TMA_BF16)
        return bwd_data_typed<uint16_t>(n, static_cast<const uint16_t *>(dHnext), static_cast<const uint16_t *>(Hnext),
                                        ld_next, inv_deg, W_self, W_neigh, F_in, F_out, act,
                                        static_cast<uint16_t *>(dH_self_out), ldh,
                                        static_cast<uint16_t *>(dM_scaled_out), stream);
    return fail(TMA_ERR_UNSUPPORTED_DTYPE, "sage gemm bwd: dtype %d", dtype);
}

}  // namespace tma
