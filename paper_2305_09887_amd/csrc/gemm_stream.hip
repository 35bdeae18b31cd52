// The products of bf16 storage over many nodes: operands, narrowed weights and tiles of gemm_bf16_async.hpp.
#include "gemm_core.hpp"
#include "dense_epilogue.hpp"
#include "gemm_bf16_async.hpp"

namespace tma {

// Which products come here.  From a tile of 256 rows per compute unit on, and from twice that for a product of few operations a row;
// where a tile is padded, or slabs are fetched pair by pair, only where bytes alone count.  us, gemm_bf16_kernel -> here:
//   forward, 65,536 / 125,237 rows: 128 -> 256 38 -> 32 / 66 -> 59, 256 -> 256 57 -> 49 / 97 -> 85; both at 12,500,000: 11,200 -> 6,890 (4.7 TB/s)
//   64 -> 128 21 -> 21, 45 -> 39 at 181,000; 100 -> 120 72 -> 78 at 181,000, 555 -> 552 at 1,500,000; 96 -> 64 46 -> 48, 344 -> 347
//   input gradient with ReLU (with the gather after it): 256 -> 256 85 -> 70 / 163 -> 134, alone at 12,500,000 11,520 -> 7,040; 128 -> 128
//   without ReLU 37 -> 33 at 65,536; 96 -> 64 88 -> 83 at 181,000, 178 -> 184 at 400,000, 642 -> 580 at 1,500,000; 64 -> 128 (half the tile) 60 -> 89
//   dense input gradient, 98,304 / 181,000 / 1,500,000 rows: 256 <- 256 46 -> 36 / 86 -> 56 / 680 -> 395, with ReLU 70 -> 47 / 127 -> 69 / 958 -> 511;
//   256 <- 64 39 -> 27 / 72 -> 43 / 565 -> 326; 256 <- 47 (slabs pair by pair) 26 -> 25 / 45 -> 45 / 373 -> 414
//   transformed first, forward 256 -> 47: 28 -> 27 / 48 -> 42 / 2,460 -> 1,730 (5.1 TB/s); 128 -> 47 23 -> 23 at 65,536, 49 -> 43 at 181,000
//   transformed first, input gradient: 128 -> 47 14 -> 17 at 65,536, 30 -> 26 at 181,000; 256 -> 20 (slabs pair by pair) 85 -> 90 at
//   400,000, 353 -> 303 at 1,500,000; 256 -> 47 3,850 -> 1,690 (5.2 TB/s) at 12,500,000
constexpr int64_t kManyRows = 65536, kTransformRows = 98304, kStreamRows = int64_t(1) << 20;
// tiles of 256 rows leave a fifth of the units, or more, without one in the last round
static bool unfilled(int64_t n)
{
    const int64_t tiles = ceil_div(n, 256);
    return tiles * 5 < ceil_div(tiles, 256) * 256 * 4;
}
// rows that gemm_bf16_kernel reads in groups of four; others element by element (2 x 102 -> 300 at
// 65,600 rows 117 us, 62 here), and lines below that were drawn against groups do not hold
static bool quads(const uint16_t *p, int64_t ld) { return aligned(p, 8) && ld % 4 == 0; }
// kNarrow: results of 96 columns and fewer come here; paired: columns 2c and 2c + 1 are one word (as Epi::pairs_ok says on the device)
template <bool kMask, bool kNarrow = true, class Epi>
static void launch_rows16(const char *what, const AsyncRows16 &a, const uint16_t *mask, const AsyncRows16 &b, const Epi &e, int64_t M, int N, bool paired, hipStream_t s)
{
    if constexpr (kMask) {
        launch_async16<256, 256, 4, 2, 3, true>(what, a, mask, b, e, M, N, paired, s);
    } else {
        if constexpr (kNarrow)
            if (N <= 96) return launch_async16<256, 96, 4, 1, 3, false>(what, a, mask, b, e, M, N, paired, s);
        // (and where tiles of 256 would reach past more columns.  us, with them / so / gemm_bf16_kernel, 181,000 rows: forward 256 -> 300
        // 168 / 150 / 195, 64 -> 384 80 / 64 / 80; input gradient of 300 from 256 96 / 78 / 118.  The mask is better applied once to 256, and
        // columns that go out one by one are bound by that: 110 -> 273, 528,911 rows 349 / 383)
        if (N <= 128 || (paired && ceil_div(N, 128) % 2 == 1)) launch_async16<256, 128, 4, 1, 3, false>(what, a, mask, b, e, M, N, paired, s);
        else launch_async16<256, 256, 4, 2, 4, false>(what, a, mask, b, e, M, N, paired, s);
    }
}
// rows of narrowed weights beside what a product reads them for: out[r][c], c < pitch (names of launches: one for each kernel)
struct NarrowStack {   // [W0 ; W1] of R rows each, N columns, zeros up to the pitch
    static constexpr const char *kName = "narrow_stack_bf16";
    const float *W0, *W1;
    int R, N;
    __device__ __forceinline__ float at(int r, int c) const { return c < N ? (r < R ? W0 + int64_t(r) * N : W1 + int64_t(r - R) * N)[c] : 0.0f; }
};
struct NarrowSides {   // [W0 | W1], N columns each padded with zeros to Np
    static constexpr const char *kName = "narrow_sides_bf16";
    const float *W0, *W1;
    int N, Np;
    __device__ __forceinline__ float at(int r, int c) const
    {
        const int cc = c < Np ? c : c - Np;
        return cc < N ? (c < Np ? W0 : W1)[int64_t(r) * N + cc] : 0.0f;
    }
};
struct NarrowSidesT {  // the transpose of [W0 | W1]: row r is column r, R long, zeros up to the pitch
    static constexpr const char *kName = "narrow_sides_t_bf16";
    const float *W0, *W1;
    int N, Np, R;
    __device__ __forceinline__ float at(int r, int c) const
    {
        const int col = r < Np ? r : r - Np;
        return col < N && c < R ? (r < Np ? W0 : W1)[int64_t(c) * N + col] : 0.0f;
    }
};
template <class From>
static __global__ __launch_bounds__(256) void narrow_rows_kernel(From from, int rows, int pitch, uint16_t *__restrict__ out)
{
    const int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (i < int64_t(rows) * pitch) out[i] = f32_to_bf16(from.at(int(i / pitch), int(i % pitch)));
}
template <class From>
static AsyncRows16 narrow_rows(const From &from, int rows, int K, int pitch, void *out, hipStream_t s)
{
    TMA_TIMED(From::kName, s);
    uint16_t *w = static_cast<uint16_t *>(out);
    hipLaunchKernelGGL(narrow_rows_kernel<From>, dim3(unsigned(ceil_div(int64_t(rows) * pitch, 256))), dim3(256), 0, s, from, rows, pitch, w);
    return AsyncRows16{w, pitch, w, pitch, K, K, K, rows};
}

bool stream_sage_fwd(int64_t n, const uint16_t *H, int64_t ldh, const uint16_t *M, int64_t ldm, int F_in, const uint16_t *Wt, const float *bias,
                     int F_out, bool relu, uint16_t *Hnext, int64_t ld_next, hipStream_t s)
{
    const int K = 2 * F_in;
    const AsyncRows16 a{H, ldh, M, ldm, F_in, F_in, K, n};
    if (n < kManyRows || !a.ok() || F_out <= 64) return false;
    if (F_in % kAsyncK16 != 0 && F_out <= 128 && n < kStreamRows) return false;
    if (F_in % kAsyncK16 != 0 && F_in % 4 == 0 && F_in < 128 && quads(H, ldh) && quads(M, ldm)) {   // halves that end inside a slab: one or two slabs pair by pair
        const bool two = F_in % 16 != 0, half = ceil_div(F_out, 128) % 2 == 1;
        if (F_out > 256) {
            // 131,072 / 200,000 / 400,000 / 1,048,576 rows: 28 -> 300 (tiles of 128) 51 -> 55 / 72 -> 84 / 140 -> 152 / 396 -> 410, -> 400 60 -> 62 / 85 -> 100 /
            // 166 -> 186 / 480 -> 472; 44 -> 300 59 -> 62 / 83 -> 94 / 166 -> 175 / 474 -> 466; 56 -> 300 65 -> 65 / 94 -> 100 / 188 -> 186; 100 -> 300 89 -> 84 / 126 -> 126
            const int64_t rows = !two || F_in >= 96 ? 2 * kManyRows : F_in >= 48 ? 4 * kManyRows : F_in >= 32 ? 8 * kManyRows : half ? INT64_MAX : kStreamRows;
            if (n < rows) return false;
        } else if (two) {
            // -> 256, a whole tile of the other kernel: 66,000 / 86,000 / 140,000 /
            // 200,000 rows 20 28 -> 33 / 29 -> 34 / 41 -> 45 / 53 -> 57, 100 47 -> 51 / 50 -> 51 / 68 -> 67 / 101 -> 100; -> 200, a cut one, 20 86,000 1.04 times, 140,000 0.95
            if (unfilled(n) && (F_out == 256 || (F_in < 32 && n <= 2 * kManyRows))) return false;
        }
    }
    launch_rows16<false>("gemm_fwd", a, nullptr,
                         AsyncRows16{Wt, K, Wt, K, K, K, K, F_out}, FwdEpilogue<uint16_t>{Hnext, ld_next, bias, relu}, n, F_out, F_out % 2 == 0 && ld_next % 2 == 0, s);
    return true;
}

bool stream_sage_bwd_data(int64_t n, const uint16_t *dHnext, const uint16_t *Hnext, int64_t ld_next, const float *inv_deg, const float *W_self,
                          const float *W_neigh, int F_in, int F_out, bool relu, uint16_t *dH_self_out, int64_t ldh, uint16_t *dM_scaled_out,
                          void *spare, size_t spare_bytes, hipStream_t s)
{
    const int N = 2 * F_in, pitch = int(round_up(size_t(F_out), 8));
    const AsyncRows16 a{dHnext, ld_next, dHnext, ld_next, F_out, F_out, F_out, n};
    if (n < kManyRows || (N < 256 && n < kStreamRows) || N <= (relu ? 128 : 64)) return false;
    // (a last slab pair by pair, one of four or fewer, where gemm_bf16_kernel reads groups of four: 128 -> 100 32 -> 38 at 98,304 rows, 41 -> 40 at 131,072, 130 ->
    // 110 at 400,000; with ReLU 69 -> 76 at 181,000 and 155 -> 148.  With the weight gradient and the gather, 122,000 rows: 256 -> 76 0.74 -> 0.67 of the time before
    // both, 128 -> 232 0.78, with ReLU 256 -> 232 0.79 -> 0.70)
    if (F_out % kAsyncK16 != 0 && F_out % 4 == 0 && F_out < 128 && (relu || N <= 256) && quads(dHnext, ld_next) && (!relu || quads(Hnext, ld_next)) && n < (relu ? 4 : 2) * kManyRows) return false;
    if (!a.ok() || (relu && !aligned(Hnext, 4)) || !spare || size_t(N) * pitch * 2 > spare_bytes) return false;
    const AsyncRows16 b = narrow_rows(NarrowStack{W_self, W_neigh, F_in, F_out}, N, F_out, pitch, spare, s);
    const BwdDataEpilogue<uint16_t> e{dH_self_out, ldh, dM_scaled_out, inv_deg, F_in};
    const bool paired = F_in % 2 == 0 && ldh % 2 == 0;
    if (relu) launch_rows16<true>("gemm_bwd_data", a, Hnext, b, e, n, N, paired, s);
    else launch_rows16<false>("gemm_bwd_data", a, nullptr, b, e, n, N, paired, s);
    return true;
}

bool stream_dense_bwd_data(int64_t n, const uint16_t *dY, const uint16_t *Y, int64_t ld, const float *W, int F_in, int F_out, bool relu,
                           const float *row_scale, uint16_t *dX, int64_t ldx, void *spare, size_t spare_bytes, hipStream_t s)
{
    const int pitch = int(round_up(size_t(F_out), 8));
    const AsyncRows16 a{dY, ld, dY, ld, F_out, F_out, F_out, n};
    if (n < kTransformRows || (F_in < 256 && n < kStreamRows) || F_in <= 128 || F_out < 64) return false;
    // (a last slab pair by pair: 256 <- 66 and 100 32 -> 36, 33 -> 39 at 98,304 rows, 41 -> 37, 42 -> 40 at 131,072; with the weight gradient 100 with ReLU 98 -> 90 at
    // 122,000; with ReLU in tiles of 256 that the last
    // column cuts 384 <- 66 86 -> 104 at 181,000, 192 -> 212 at 400,000, 508 -> 500 at 1,048,576.  Five slabs and more: with the weight gradient 256 <- 250 0.76 -> 0.56
    // of the time before both at 122,000)
    if (F_out % kAsyncK16 != 0 && F_out < 128 && quads(dY, ld) && (!relu || quads(Y, ld)) && (relu && F_in > 256 ? n < kStreamRows / 2 : unfilled(n) && n < 2 * kManyRows)) return false;
    if (!a.ok() || (relu && !aligned(Y, 4)) || !spare || !aligned(spare, 16) || size_t(F_in) * pitch * 2 > spare_bytes) return false;
    const AsyncRows16 b = narrow_rows(NarrowStack{W, W, F_in, F_out}, F_in, F_out, pitch, spare, s);
    const auto launch = [&](const auto &e) {
        if (relu) launch_rows16<true>("gemm_dense_bwd_data", a, Y, b, e, n, F_in, F_in % 2 == 0 && ldx % 2 == 0, s);
        else launch_rows16<false, false>("gemm_dense_bwd_data", a, nullptr, b, e, n, F_in, F_in % 2 == 0 && ldx % 2 == 0, s);
    };
    if (row_scale) launch(DenseEpilogue<uint16_t, true>{dX, ldx, nullptr, row_scale, false, F_in});
    else launch(DenseEpilogue<uint16_t, false>{dX, ldx, nullptr, nullptr, false, F_in});
    return true;
}

bool stream_sage_tf_fwd(int64_t n, const uint16_t *H, int64_t ldh, int F_in, const float *W_self, const float *W_neigh, int F_out, int Fp,
                        uint16_t *Ys, uint16_t *Yn, int64_t ldy, void *spare, size_t spare_bytes, hipStream_t s)
{
    const AsyncRows16 a{H, ldh, H, ldh, F_in, F_in, F_in, n};
    const int pitch = int(round_up(size_t(F_in), 8));
    if (n < (quads(H, ldh) && (F_in < 256 || Fp <= 24) ? 2 * kManyRows : kTransformRows) || (F_in % kAsyncK16 != 0 && n < kStreamRows)) return false;
    // (two halves of 32 are a whole tile of 64 there and two thirds of one here: 128 -> 32 22 -> 28 at 181,000 rows, 40 -> 43 at 400,000, 106 -> 100 at
    // 1,048,576; 100 -> 32 114 -> 132)
    if (Fp == 32 && quads(H, ldh) && (n < kStreamRows / 2 || F_in % kAsyncK16 != 0)) return false;
    if (!a.ok() || !spare || size_t(2) * Fp * pitch * 2 > spare_bytes) return false;
    const AsyncRows16 b = narrow_rows(NarrowSidesT{W_self, W_neigh, F_out, Fp, F_in}, 2 * Fp, F_in, pitch, spare, s);
    launch_rows16<false>("gemm_tf_fwd", a, nullptr, b, HalvesEpilogue<uint16_t>{Ys, Yn, ldy, Fp, F_out}, n, 2 * Fp, true, s);
    return true;
}

bool stream_sage_tf_bwd_data(int64_t n, const uint16_t *dHnext, int64_t ld_next, const uint16_t *dYn, int64_t ldy, const float *W_self,
                             const float *W_neigh, int F_in, int F_out, int Fp, uint16_t *dH, int64_t ldh, void *spare, size_t spare_bytes,
                             hipStream_t s)
{
    const AsyncRows16 a{dHnext, ld_next, dYn, ldy, Fp, F_out, 2 * Fp, n};
    // (slabs pair by pair where a half ends in one, two of them where its width is 8 mod 16, and tiles that are half empty.  Both launches, 131,072 /
    // 262,144 / 400,000 rows: 128 <- 40 21 -> 28 / 35 -> 41 / 52 -> 60, 153 -> 136 at 1,048,576; 128 <- 32 19 -> 21 / 30 -> 29 / 43 -> 41; 256 <- 40 36 -> 36 / 70
    // -> 61, 43 -> 46 at 160,000; 160 <- 56 45 -> 39 / 84 -> 65; with the weight gradient 256 <- 76 118 -> 107 at 122,000)
    const bool half = F_in > 96 && F_in <= 128, two = Fp % 16 != 0 && Fp < 96;
    if (n < (!quads(dHnext, ld_next) || (Fp >= 64 && !two) ? (Fp < 32 ? kStreamRows : kTransformRows)
                                     : Fp < 32 || (half && two) ? kStreamRows : half || two ? 4 * kManyRows : 2 * kManyRows)) return false;
    if (!a.ok() || !spare || size_t(F_in) * 2 * Fp * 2 > spare_bytes) return false;
    const AsyncRows16 b = narrow_rows(NarrowSides{W_self, W_neigh, F_out, Fp}, F_in, 2 * Fp, 2 * Fp, spare, s);
    launch_rows16<false>("gemm_tf_bwd_data", a, nullptr, b, RowsEpilogue<uint16_t>{dH, ldh}, n, F_in, F_in % 2 == 0 && ldh % 2 == 0, s);
    return true;
}

// ---- weight gradients
// A tile of 256 rows per compute unit and twice that from kStreamRows on, where the partial results are a small part of the bytes; not
// where most of a tile is padding.  us, gemm_bf16_kernel -> here, both with the second stage:
//   with ReLU, 65,536 / 181,000 / 1,500,000 nodes: 128 -> 256 64 -> 52 / 125 -> 77 / 569 -> 480, 256 -> 256 92 -> 56 / 211 -> 110 / 941 -> 751,
//   100 -> 128 50 -> 39 / 79 -> 55 / 421 -> 295, 120 -> 64 31 -> 37 / 55 -> 51 / 326 -> 266, 64 -> 64 35 -> 36 / 46 -> 54 / 181 -> 306;
//   150 -> 150, element by element before, 195 -> 50 / 503 -> 88 / 4,850 -> 647; 256 -> 256 without ReLU 84 -> 46 / 191 -> 78 / 846 -> 472 (4.9 TB/s)
//   transformed first: 256 -> 47 49 -> 43 / 87 -> 65 / 434 -> 301, 128 -> 47 38 -> 47 / 69 -> 69 / 271 -> 251, 128 -> 20 83 -> 89 at 400,000
bool plan_stream_weight(int64_t n, int32_t F_in, int32_t F_out, size_t ws_bytes, WeightSplit &w)
{
    if (F_in < 8 || F_out < 8 || (F_in <= 64 && F_out <= 64) || n < (F_out <= 64 ? 2 * kManyRows : kManyRows)) return false;
    const int64_t tiles = ceil_div(2 * round_up(size_t(F_in), 8), 256) * ceil_div(F_out, F_out > 128 ? 256 : 128);
    const size_t per_split = size_t(2) * F_in * F_out * 4 + size_t(F_out) * 4, operands = size_t(n) * (2 * size_t(F_in) + size_t(F_out)) * 2;
    // (one item fewer for every eighth unit where the partial results would be more than half of the operands: 65,536 nodes, 128 / 224 / 256 items: 128 -> 256
    // 39 / 39 / 42, 66 -> 130 36 / 36 / 38, 256 -> 256 49 / 44 / 47; with less: 181,000 nodes, 128 / 256 items: 128 -> 256 60 / 58, with ReLU 92 / 76, 256 -> 256 95 /
    // 79 and 163 / 112)
    int64_t want = (n >= kStreamRows ? 512 : size_t(256 / tiles) * per_split > operands / 2 ? 224 : 256) / tiles;
    if (want < 1) want = 1;
    if (ws_bytes < 512 + per_split) return false;
    if (size_t(want) > (ws_bytes - 512) / per_split) want = int64_t((ws_bytes - 512) / per_split);
    w.k_per_split = int64_t(round_up(size_t(ceil_div(n, want)), kAsyncK16));
    w.n_splits = int(ceil_div(n, w.k_per_split));
    w.partial_bytes = round_up(size_t(w.n_splits) * 2 * size_t(F_in) * size_t(F_out) * 4, 256);
    w.colsum_bytes = round_up(size_t(w.n_splits) * size_t(F_out) * 4, 256);
    return true;
}

bool stream_sage_bwd_weight(int64_t n, const uint16_t *H, int64_t ldh, const uint16_t *M, int64_t ldm, const uint16_t *dHnext, const uint16_t *Hnext,
                            int64_t ld_next, int F_in, int F_out, bool relu, const WeightSplit &w, float *partial, float *colsum, hipStream_t s)
{
    const int Fq = int(round_up(size_t(F_in), 8)), No = int(round_up(size_t(F_out), 8));
    const AsyncCols16 a{H, ldh, M, ldm, F_in, Fq, 2 * Fq, n}, b{dHnext, ld_next, dHnext, ld_next, F_out, No, No, n};
    // (half of the tile empty and a mask for all of it: 64 -> 96 99 -> 80 at 400,000 nodes, 144 -> 123 at 700,000, but 250 -> 255 at 1,500,000 and 812 -> 879 at
    // 6,000,000, where the partial results no longer tell; 48 -> 96 243 -> 259 and 806 -> 905)
    if (relu && F_in <= 64 && F_in % 4 == 0 && F_out <= 128 && n >= kStreamRows && quads(H, ldh) && quads(M, ldm) && quads(dHnext, ld_next) && quads(Hnext, ld_next))
        return false;
    if (!a.ok() || !b.ok() || (relu && !aligned(Hnext, 4))) return false;
    if (F_out > 128) {
        if (relu) launch_weight16<256, 2, 3, true>("gemm_bwd_weight", a, b, Hnext, F_out, w.k_per_split, w.n_splits, partial, colsum, s);
        else launch_weight16<256, 2, 4, false>("gemm_bwd_weight", a, b, nullptr, F_out, w.k_per_split, w.n_splits, partial, colsum, s);
    } else {
        if (relu) launch_weight16<128, 1, 4, true>("gemm_bwd_weight", a, b, Hnext, F_out, w.k_per_split, w.n_splits, partial, colsum, s);
        else launch_weight16<128, 1, 6, false>("gemm_bwd_weight", a, b, nullptr, F_out, w.k_per_split, w.n_splits, partial, colsum, s);
    }
    return true;
}

// A plan made for tiles of 128 may leave a last round of items that few of the compute units have one of (three of those tiles: 171 ranges, 342
// items of two of these): fewer ranges of nodes then, so that every unit has as many.  us at 181,000 nodes, gemm_bf16_kernel / as planned / so:
//   dense with ReLU 264 -> 66 94 / 106 / 73, 384 -> 47 75 / 104 / 71, 100 -> 300 109 / 124 / 88; transformed first 264 -> 20 86 / 90 / 69
static void whole_rounds(int64_t n, int64_t tiles, WeightSplit &w)
{
    const int64_t items = tiles * w.n_splits, ranges = items / 256 * 256 / tiles;
    if (items <= 256 || ranges < 1) return;
    w.k_per_split = int64_t(round_up(size_t(ceil_div(n, ranges)), kAsyncK16));
    w.n_splits = int(ceil_div(n, w.k_per_split));
}

// The dense layer's, in the ranges of nodes that it plans: where they make an item for half of the compute units or more, and not where
// much of a narrow tile is padding.  us, gemm_bf16_kernel -> here, both with the second stage, 98,304 / 181,000 / 1,500,000 nodes:
//   256 -> 256 72 -> 46 / 109 -> 62 / 712 -> 339 (128 items), with ReLU 83 -> 62 / 125 -> 94 / 790 -> 595; 128 -> 256 62 -> 48 / 86 -> 62 /
//   432 -> 359; 256 -> 47 37 -> 36 / 54 -> 41 / 308 -> 172; 150 -> 150, element by element before, 148 -> 44 / 279 -> 58 / 2,352 -> 324;
//   300 -> 47 58 -> 56 / 71 -> 78 / 605 -> 433
bool stream_dense_bwd_weight(int64_t n, const uint16_t *X, int64_t ldx, const uint16_t *dY, const uint16_t *Y, int64_t ld, int F_in, int F_out,
                             bool relu, WeightSplit &w, float *partial, float *colsum, hipStream_t s)
{
    const int Fq = int(round_up(size_t(F_in), 8)), No = int(round_up(size_t(F_out), 8));
    const AsyncCols16 a{X, ldx, X, ldx, F_in, Fq, Fq, n}, b{dY, ld, dY, ld, F_out, No, No, n};
    const int64_t tiles = ceil_div(Fq, 256) * ceil_div(F_out, F_out > 128 ? 256 : 128);
    // (half of a narrow tile empty, or three quarters: 256 -> 64 34 -> 36 at 80,000 nodes, 39 -> 38 at 98,304; with ReLU 40 -> 43 and 59 -> 53 at 181,000.  With the
    // input gradient, 1,048,576 / 4,000,000 nodes: 64 -> 16 with ReLU 190 -> 235 / 679 -> 818, 64 -> 96 302 -> 327 / 1,040 -> 1,107, 64 -> 128 at 2,000,000 0.99 times;
    // without 128 -> 64 268 -> 279, 0.96 at 1,500,000)
    if (quads(X, ldx) && quads(dY, ld) && (!relu || quads(Y, ld))) {
        if (F_out <= 64 && Fq <= 256 && n < (relu ? 2 * kManyRows : kTransformRows)) return false;
        if (F_in <= 128 && (relu ? F_out <= 96 : F_out <= 64 && n < kStreamRows * 5 / 4)) return false;
    }
    if (n < kManyRows || tiles * w.n_splits < 112 || (F_in <= 128 && F_out <= 128 && n < kStreamRows) ||
        (F_out <= 64 && ceil_div(Fq, 256) * 256 * 2 > 3 * Fq && n < kStreamRows) || !a.ok() || !b.ok() || (relu && !aligned(Y, 4))) return false;
    whole_rounds(n, tiles, w);
    if (F_out > 128) {
        if (relu) launch_weight16<256, 2, 3, true>("gemm_dense_bwd_weight", a, b, Y, F_out, w.k_per_split, w.n_splits, partial, colsum, s);
        else launch_weight16<256, 2, 4, false>("gemm_dense_bwd_weight", a, b, nullptr, F_out, w.k_per_split, w.n_splits, partial, colsum, s);
    } else {
        if (relu) launch_weight16<128, 1, 4, true>("gemm_dense_bwd_weight", a, b, Y, F_out, w.k_per_split, w.n_splits, partial, colsum, s);
        else launch_weight16<128, 1, 6, false>("gemm_dense_bwd_weight", a, b, nullptr, F_out, w.k_per_split, w.n_splits, partial, colsum, s);
    }
    return true;
}

bool stream_sage_tf_bwd_weight(int64_t n, const uint16_t *H, int64_t ldh, const uint16_t *dHnext, int64_t ld_next, const uint16_t *dYn, int64_t ldy,
                               int F_in, int F_out, int Fp, WeightSplit &w, float *partial, float *colsum, hipStream_t s)
{
    const int Fq = int(round_up(size_t(F_in), 8));
    const AsyncCols16 a{H, ldh, H, ldh, F_in, Fq, Fq, n}, b{dHnext, ld_next, dYn, ldy, F_out, Fp, 2 * Fp, n};
    // (a quarter of the tile: 128 -> 32 117 -> 130, 100 -> 20 117 -> 124 at 1,048,576 nodes, 128 -> 20 358 -> 341 at 2,000,000)
    if (n < (F_in > 128 ? kManyRows : Fp <= 32 && quads(H, ldh) && quads(dHnext, ld_next) ? 2 * kStreamRows : kStreamRows) || !a.ok() || !b.ok()) return false;
    whole_rounds(n, ceil_div(Fq, 256) * ceil_div(2 * Fp, 2 * Fp > 128 ? 256 : 128), w);
    if (2 * Fp > 128) launch_weight16<256, 2, 4, false>("gemm_tf_bwd_weight", a, b, nullptr, 2 * Fp, w.k_per_split, w.n_splits, partial, colsum, s);
    else launch_weight16<128, 1, 6, false>("gemm_tf_bwd_weight", a, b, nullptr, 2 * Fp, w.k_per_split, w.n_splits, partial, colsum, s);
    return true;
}

}  // namespace tma
