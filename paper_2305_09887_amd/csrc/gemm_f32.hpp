// The tile product of fp32 storage on v_mfma_f32_32x32x2_f32, fp32 in, fp32 accumulate: backward products of few rows.  (The
// forward products sum in the same order, in a kernel of their own: gemm_f32_async.hpp.)
//
// Why not the product of bf16 parts (gemm_split.hpp), which the other backward products take and which is faster: what a layer
// puts out is compared with zero (ReLU, PReLU, in this layer or one that follows), and an input of such a comparison that
// lies within a rounding of zero falls on the other side when its sum is taken in another order.  In a mini-batch of some
// thousand rows ONE such unit is worth 1e-4 to 5e-4 of the weights' gradient, a thousand times what the rounding itself
// is.  The order is therefore part of a forward result, whatever the size and the tile:
//     c <- fma(a[k], b[k], c)    for k = 0, 4, 1, 5, 2, 6, 3, 7 of every eight k-values, from one accumulator.
// (An instruction takes two k-values, the first half of the wavefront's before the second's.)  A gradient decides nothing in
// its own step, but the next one from its weights: see few_rows.
//
// Tiling: BM x BN block tile, each wavefront owning a (BM/WM) x (BN/WN) patch of 32x32 MFMA tiles, k in slabs of BK through
// two LDS buffers (one barrier per slab) while the next slab's global loads are in flight in registers.  Every operand keeps
// the orientation it has in memory:
//   k-contiguous operand : LDS [mn][BK+4]; a lane fetches four k-values of its row with one 16-byte read, for four MFMAs;
//   mn-contiguous operand: LDS [BK][MN+4]; a lane reads one element per k-value.
#pragma once

namespace tma {

// C[M,N] = A[M,K] B[K,N], k split into ranges of k_per_split; work items and their order over the dies as in gemm_bf16_kernel.
template <int BM, int BN, int BK, int WM, int WN, bool kColSum, class AL, class BL, class Epi>
__global__ __launch_bounds__(WM *WN * 64, 2) void gemm_f32_kernel(
    AL a, BL b, Epi epi, int64_t M, int N, int64_t K, int64_t k_per_split, int n_tiles, int64_t tiles_per_split, int64_t total_work,
    float *__restrict__ colsum_partial)
{
    constexpr int NT = WM * WN * 64;
    constexpr int TM = BM / WM / 32;
    constexpr int TN = BN / WN / 32;
    constexpr int A_Q = BM * BK / 4, B_Q = BN * BK / 4;   // 16-byte pieces of a slab
    constexpr int A_V = (A_Q + NT - 1) / NT;              // load slots per thread; when the pieces do not divide
    constexpr int B_V = (B_Q + NT - 1) / NT;              // evenly the last slots repeat the last piece (same value)
    constexpr int GK = 8;                                 // k-values of a fragment: four MFMAs
    constexpr int KG = BK / GK;
    constexpr int A_LD = AL::kContigK ? BK + kPad : BM + kPad;
    constexpr int B_LD = BL::kContigK ? BK + kPad : BN + kPad;
    constexpr int A_WORDS = AL::kContigK ? BM * A_LD : BK * A_LD;
    constexpr int B_WORDS = BL::kContigK ? BN * B_LD : BK * B_LD;
    static_assert(BM % (WM * 32) == 0 && BN % (WN * 32) == 0 && BK % GK == 0, "tile shape");
    static_assert(!kColSum || !BL::kContigK, "column sums are taken from a [k][n] tile");
    static_assert(A_WORDS >= BN && B_WORDS >= BM, "epilogue staging fits");

    __shared__ __attribute__((aligned(16))) float As[2][A_WORDS];
    __shared__ __attribute__((aligned(16))) float Bs[2][B_WORDS];
    float *const a_aux = &As[0][0];   // per-column / per-row epilogue inputs
    float *const b_aux = &Bs[0][0];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int l31 = lane & 31;
    const int hi = lane >> 5;
    const int wave = tid >> 6;
    const int wm0 = (wave / WN) * (BM / WM);
    const int wn0 = (wave % WN) * (BN / WN);

    // loop-invariant positions of this thread's load slots inside a tile, and their LDS word offsets
    int a_mn[A_V], a_k[A_V], a_lds[A_V], b_mn[B_V], b_k[B_V], b_lds[B_V];
#pragma unroll
    for (int i = 0; i < A_V; ++i) {
        const int idx = (tid + i * NT) < A_Q ? (tid + i * NT) : A_Q - 1;
        a_mn[i] = AL::kContigK ? idx / (BK / 4) : (idx % (BM / 4)) * 4;
        a_k[i] = AL::kContigK ? (idx % (BK / 4)) * 4 : idx / (BM / 4);
        a_lds[i] = AL::kContigK ? a_mn[i] * A_LD + a_k[i] : a_k[i] * A_LD + a_mn[i];
    }
#pragma unroll
    for (int i = 0; i < B_V; ++i) {
        const int idx = (tid + i * NT) < B_Q ? (tid + i * NT) : B_Q - 1;
        b_mn[i] = BL::kContigK ? idx / (BK / 4) : (idx % (BN / 4)) * 4;
        b_k[i] = BL::kContigK ? (idx % (BK / 4)) * 4 : idx / (BN / 4);
        b_lds[i] = BL::kContigK ? b_mn[i] * B_LD + b_k[i] : b_k[i] * B_LD + b_mn[i];
    }

    const int64_t blocks_per_die = gridDim.x / kXcds;
    const int64_t per_die = (total_work + kXcds - 1) / kXcds;
    const int64_t die = blockIdx.x % kXcds;
    int64_t die_end = (die + 1) * per_die;
    if (die_end > total_work) die_end = total_work;

    typename AL::Lane alane[A_V];
    typename BL::Lane blane[B_V];
    // first slab of the tile that comes next; the slabs inside a tile's main loop have registers of their own
    typename AL::Raw afirst[A_V];
    typename BL::Raw bfirst[B_V];
    struct Tile {
        int64_t m0;
        int n0, split;
        int64_t k_begin, k_end;
    };
    Tile t{};
    auto prepare = [&](int64_t work) {
        t.split = int(work / tiles_per_split);
        const int64_t tile = work % tiles_per_split;
        t.m0 = (tile / n_tiles) * BM;
        t.n0 = int(tile % n_tiles) * BN;
        t.k_begin = int64_t(t.split) * k_per_split;
        t.k_end = t.k_begin + k_per_split < K ? t.k_begin + k_per_split : K;
#pragma unroll
        for (int i = 0; i < A_V; ++i) alane[i] = a.prepare(t.m0 + a_mn[i]);
#pragma unroll
        for (int i = 0; i < B_V; ++i) blane[i] = b.prepare(t.n0 + b_mn[i]);
    };
    auto fetch = [&](int64_t kt, typename AL::Raw(&ar)[A_V], typename BL::Raw(&br)[B_V]) {   // any slab
#pragma unroll
        for (int i = 0; i < A_V; ++i) ar[i] = a.load(alane[i], kt + a_k[i]);
#pragma unroll
        for (int i = 0; i < B_V; ++i) br[i] = b.load(blane[i], kt + b_k[i]);
    };
    auto fetch_whole = [&](int64_t kt, typename AL::Raw(&ar)[A_V], typename BL::Raw(&br)[B_V]) {   // inside the k range
#pragma unroll
        for (int i = 0; i < A_V; ++i) ar[i] = a.load_plain(alane[i], kt, a_k[i]);
#pragma unroll
        for (int i = 0; i < B_V; ++i) br[i] = b.load_plain(blane[i], kt, b_k[i]);
    };
    auto stage = [&](int buf, const typename AL::Raw(&ar)[A_V], const typename BL::Raw(&br)[B_V]) {
#pragma unroll
        for (int i = 0; i < A_V; ++i) *reinterpret_cast<float4 *>(&As[buf][a_lds[i]]) = AL::resolve(ar[i]);
#pragma unroll
        for (int i = 0; i < B_V; ++i) *reinterpret_cast<float4 *>(&Bs[buf][b_lds[i]]) = BL::resolve(br[i]);
    };
    // This lane's k-values of group g (the upper half of the wavefront holds the upper half of the group) of its
    // row/column.
    auto frag_a = [&](int buf, int g, int i) -> float4 {
        const int mn = wm0 + i * 32 + l31;
        const int k = g * GK + (GK / 2) * hi;
        if constexpr (AL::kContigK) return *reinterpret_cast<const float4 *>(&As[buf][mn * A_LD + k]);
        const float *p = &As[buf][k * A_LD + mn];
        return make_float4(p[0], p[A_LD], p[2 * A_LD], p[3 * A_LD]);
    };
    auto frag_b = [&](int buf, int g, int j) -> float4 {
        const int mn = wn0 + j * 32 + l31;
        const int k = g * GK + (GK / 2) * hi;
        if constexpr (BL::kContigK) return *reinterpret_cast<const float4 *>(&Bs[buf][mn * B_LD + k]);
        const float *p = &Bs[buf][k * B_LD + mn];
        return make_float4(p[0], p[B_LD], p[2 * B_LD], p[3 * B_LD]);
    };

    int64_t work = die * per_die + blockIdx.x / kXcds;
    if (work >= die_end) return;
    prepare(work);
    fetch(t.k_begin, afirst, bfirst);
    while (true) {
        floatx16 acc[TM][TN];
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
        float colsum = 0.0f;

        __syncthreads();  // the previous tile's epilogue has finished reading LDS
        stage(0, afirst, bfirst);
        __syncthreads();

        // one slab from LDS buffer `buf`: fragment reads one group ahead of the MFMAs that use them
        auto multiply = [&](int buf) {
            float4 fa[2][TM], fb[2][TN];
#pragma unroll
            for (int i = 0; i < TM; ++i) fa[0][i] = frag_a(buf, 0, i);
#pragma unroll
            for (int j = 0; j < TN; ++j) fb[0][j] = frag_b(buf, 0, j);
#pragma unroll
            for (int g = 0; g < KG; ++g) {
                const int cur = g & 1, nxt = cur ^ 1;
                if (g + 1 < KG) {  // next group's fragments are in flight while this group's MFMAs run
#pragma unroll
                    for (int i = 0; i < TM; ++i) fa[nxt][i] = frag_a(buf, g + 1, i);
#pragma unroll
                    for (int j = 0; j < TN; ++j) fb[nxt][j] = frag_b(buf, g + 1, j);
                }
#pragma unroll
                for (int q = 0; q < 4; ++q)   // the four k-pairs in turn, round-robin over the output tiles
#pragma unroll
                    for (int i = 0; i < TM; ++i)
#pragma unroll
                        for (int j = 0; j < TN; ++j) {
                            const float av = q == 0 ? fa[cur][i].x : q == 1 ? fa[cur][i].y : q == 2 ? fa[cur][i].z : fa[cur][i].w;
                            const float bv = q == 0 ? fb[cur][j].x : q == 1 ? fb[cur][j].y : q == 2 ? fb[cur][j].z : fb[cur][j].w;
                            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(av, bv, acc[i][j], 0, 0, 0);
                        }
            }
            if (kColSum && t.m0 == 0 && tid < BN) {
#pragma unroll
                for (int k = 0; k < BK; ++k) colsum += Bs[buf][k * B_LD + tid];
            }
        };
        auto main_loop = [&](auto whole_tag) {
            typename AL::Raw areg[A_V];
            typename BL::Raw breg[B_V];
            int buf = 0;
            for (int64_t kt = t.k_begin; kt < t.k_end; kt += BK) {
                const bool more = kt + BK < t.k_end;
                if (more) {  // in flight while this slab is multiplied
                    if constexpr (decltype(whole_tag)::value) fetch_whole(kt + BK, areg, breg);
                    else fetch(kt + BK, areg, breg);
                }
                multiply(buf);
                if (more) stage(buf ^ 1, areg, breg);  // the other buffer was last read before the previous barrier
                __syncthreads();
                buf ^= 1;
            }
        };
        if ((t.k_end - t.k_begin) % BK == 0) main_loop(std::true_type{});
        else main_loop(std::false_type{});

        // Per-column / per-row epilogue inputs (bias, 1/deg) go through LDS (see gemm_bf16_kernel).
        if (Epi::kColAux && tid < BN) a_aux[tid] = epi.col_aux(t.n0 + tid < N ? t.n0 + tid : N - 1);
        if (Epi::kRowAux && tid < BM) b_aux[tid] = epi.row_aux(t.m0 + tid < M ? t.m0 + tid : M - 1);
        if (Epi::kColAux || Epi::kRowAux) __syncthreads();

        const Tile done = t;
        const float done_colsum = colsum;
        const int64_t next = work + blocks_per_die;
        const bool has_next = next < die_end;
        if (has_next) {   // its latency passes behind the write-out below
            prepare(next);
            fetch(t.k_begin, afirst, bfirst);
        }

        // MFMA 32x32 result layout: register r of lane l holds row 8*(r/4) + 4*(l/32) + r%4, column l%32.
        float caux[TN];
#pragma unroll
        for (int j = 0; j < TN; ++j) caux[j] = Epi::kColAux ? a_aux[wn0 + j * 32 + l31] : 0.0f;
        auto write_out = [&](auto inside_tag) {
            constexpr bool kInside = decltype(inside_tag)::value;   // the whole tile lies inside the result
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                float raux[16];
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    raux[r] = Epi::kRowAux ? b_aux[wm0 + i * 32 + 8 * (r / 4) + 4 * hi + (r % 4)] : 0.0f;
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    const int col = done.n0 + wn0 + j * 32 + l31;
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int64_t row = done.m0 + wm0 + i * 32 + 8 * (r / 4) + 4 * hi + (r % 4);
                        const float val = epi.value(acc[i][j][r], caux[j], raux[r], col);
                        if (kInside || (row < M && col < N)) epi.store(row, col, val, done.split);
                    }
                }
            }
        };
        if (done.m0 + BM <= M && done.n0 + BN <= N) write_out(std::true_type{});
        else write_out(std::false_type{});
        if (kColSum && done.m0 == 0 && tid < BN && done.n0 + tid < N)
            colsum_partial[int64_t(done.split) * N + done.n0 + tid] = done_colsum;
        if (!has_next) break;
        work = next;
    }
}

}  // namespace tma
