// Products of bf16 storage whose rows are nodes, on v_mfma_f32_32x32x16_bf16, both operands fetched straight into LDS as in
// gemm_f32_async.hpp: rows of bf16 along k, the nodes' from one or two arrays, the weights' from a narrowed copy.
//
// These products are bound by streaming the nodes' rows in and the results out (2 x 256 -> 256: 1.5 KB and 262 kFLOP a row, a
// third of the matrix rate at 5 TB/s).  What they need is bytes in flight at all times, so: tiles as wide as the result (every
// row is read once), a ring of slabs of 32 k-values fetched kStages - 1 ahead through tile boundaries (the next rows arrive
// while results are written), and no registers, conversions or LDS writes between memory and the matrix units.  A ReLU mask is
// applied to the fragments, from a third stream into LDS.
//
// 12,500,000 rows, gemm_bf16_kernel -> here: forward products of 128 -> 256 and 256 -> 256 11.2 -> 6.9 ms (4.7 TB/s), input gradient of 2 x 256
// from 256 with ReLU 11.5 -> 7.0 (3.6 TB/s), transformed first 2.5 -> 1.7 (5.1) and 3.9 -> 1.7 (5.2); a large copy reaches 5.0 TB/s.
//
// Sums: groups of 16 k-values in order, one accumulator, as in gemm_bf16_kernel: the same bits.
#pragma once

#include <cstdio>

namespace tma {

constexpr int kAsyncK16 = 32;          // k-values of a slab: 64 bytes of a row

// X[m][k] = k < F ? P0[m][k] : P1[m][k-F]  for k < K.  Of the first part only Fv columns are its own; [Fv, F) reads as zero (but
// for column Fv where Fv is odd: the kernel clears it).  Pieces of eight elements at 4-byte-aligned addresses where a slab lies
// inside one part, else pairs of elements lane by lane: F and the pitches are even, the bases 4-byte aligned.
struct AsyncRows16 {
    const uint16_t *P0;
    int64_t ld0;
    const uint16_t *P1;
    int64_t ld1;
    int F, Fv, K;
    int64_t rows;
    __host__ __device__ __forceinline__ int run(int kt) const { return kt < F ? (kt < Fv ? (Fv - kt) / kAsyncK16 : 0) : (K - kt) / kAsyncK16; }
    // the pair of elements k, k + 1 (k even)
    __host__ __device__ __forceinline__ const uint16_t *at(int64_t m, int k, const void *zeros) const
    {
        const int64_t row = m < rows ? m : rows - 1;
        return k < Fv ? P0 + row * ld0 + k : k >= F && k < K ? P1 + row * ld1 + (k - F) : static_cast<const uint16_t *>(zeros);
    }
    // what the kernel needs of them; a pitch keeps offsets inside a tile in 32 bits
    __host__ bool ok() const
    {
        const auto even = [](const uint16_t *p, int64_t ld) { return (reinterpret_cast<uintptr_t>(p) & 3) == 0 && ld % 2 == 0 && ld <= (1 << 21); };
        return F % 2 == 0 && K % 2 == 0 && even(P0, ld0) && (K == F || even(P1, ld1));
    }
};

// One operand's slabs of ROWS rows on their way into LDS, [ROWS][32], the 16-byte pieces of a row exchanged by a quarter of its row number:
// wavefront loads of 16 rows, kLoads of them by each wavefront.  LDS has 64 banks, 256 bytes, which four rows take, and 16 lanes of a
// fragment read are served at once: of their 16 rows those that share banks are four apart.  (Exchanged by half of the row number two of them met:
// such reads alone 235 and 120 bytes a clock and unit; 2 x 256 -> 256 at 2,000,000 rows 789 and 751 us, the other products up to 2 % apart.)
template <int ROWS, int kWaves, bool kPaired = false>
struct Fetch16 {
    static constexpr int kI = ROWS / 16, kLoads = (kI + kWaves - 1) / kWaves;   // (where they do not divide the last is fetched twice)
    const uint16_t *at;     // of the next slab of the run, of row 0 of the tile
    uint32_t off[kLoads];
    static __device__ __forceinline__ int load_of(int v, int wave) { return v * kWaves + wave < kI ? v * kWaves + wave : kI - 1; }
    static __device__ __forceinline__ int piece(int row, int slot) { return slot ^ ((row >> 2) & 3); }
    // the operand's row that lies in row r: kPaired, of every whole 64 the even ones and then the odd ones (see the write-out)
    static __device__ __forceinline__ int source(int r) { return kPaired && r < ROWS / 64 * 64 ? (r & ~63) | (r & 31) << 1 | (r >> 5 & 1) : r; }
    __device__ __forceinline__ void enter_run(const AsyncRows16 &x, int64_t m0, int kt, int wave, int lane)
    {
        const bool first = kt < x.F;
        at = first ? x.P0 + m0 * x.ld0 + kt : x.P1 + m0 * x.ld1 + (kt - x.F);
        const int64_t left = x.rows - 1 - m0;
#pragma unroll
        for (int v = 0; v < kLoads; ++v) {
            const int r = load_of(v, wave) * 16 + lane / 4, from = source(r), row = from < left ? from : int(left);
            off[v] = (uint32_t(row) * uint32_t(first ? x.ld0 : x.ld1) + uint32_t(piece(r, lane & 3) * 8)) * 2u;
        }
    }
    __device__ __forceinline__ void whole(uint32_t to, const uint16_t *base, int wave) const
    {
#pragma unroll
        for (int v = 0; v < kLoads; ++v) lds_fetch<4>(to + uint32_t(load_of(v, wave)) * 1024u, reinterpret_cast<const float *>(base), off[v]);
    }
    // any position, pair by pair
    __device__ __forceinline__ static void slowly(const AsyncRows16 &x, int64_t m0, int kt, uint32_t to, int wave, int lane)
    {
#pragma unroll 1
        for (int v = 0; v < 4 * kLoads; ++v) {
            const int q = v * kWaves + wave < 4 * kI ? v * kWaves + wave : 4 * kI - 1;      // 4 rows each
            const int r = q * 4 + lane / 16, slot = (lane >> 2) & 3;
            lds_fetch<1>(to + uint32_t(q) * 256u, reinterpret_cast<const float *>(x.at(m0 + source(r), kt + piece(r, slot) * 8 + (lane & 3) * 2, kZeros)));
        }
    }
};

// The values of g where h > 0 (h NaN: not), zeros elsewhere; two bf16 in a word.  With a comparison the compiler makes selects of it,
// half by half, eight instructions with waits between them; so it makes four packed ones.  Not in assembler: between a vector instruction
// and the matrix instruction that reads its result two others have to pass, and the compiler only counts those that it knows.
typedef unsigned short ushortx2 __attribute__((ext_vector_type(2)));
typedef short shortx2 __attribute__((ext_vector_type(2)));
__host__ __device__ __forceinline__ uint32_t where_positive(uint32_t g, uint32_t h)
{
    const ushortx2 below = __builtin_bit_cast(ushortx2, h) - ushortx2{1, 1};                     // 0 .. 0x7F7F: positive, up to infinity
    const ushortx2 top = __builtin_elementwise_add_sat(below, ushortx2{0x80, 0x80});             // its top bit: clear for those
    return g & ~__builtin_bit_cast(uint32_t, __builtin_bit_cast(shortx2, top) >> shortx2{15, 15});
}

// C[M,N] = A[M,K] B[N,K]^T.  kMask: A's elements count where `mask`, an array like A's only part, is positive.  kCut: the last column
// cuts a tile, whose results are then stored in pairs too (element by element a cut tile of 256 was dearer than the whole ones of 128
// that it replaced: input gradient of 384 columns from 64 with ReLU, 181,000 rows, 102 -> 74 us against 92); in a kernel of its own, for
// the comparisons slow the others (128 -> 256 with ReLU at 400,000 rows 156 -> 163).  Persistent blocks over tiles numbered as in
// gemm_bf16_kernel, m then n.
template <int BM, int BN, int WM, int WN, int kStages, bool kMask, bool kCut, class Epi>
__global__ __launch_bounds__(WM *WN * 64, 2) void gemm_bf16_async_kernel(AsyncRows16 a, const uint16_t *mask, AsyncRows16 b, Epi epi, int64_t M, int N,
                                                                         int n_tiles, int64_t total_work)
{
    constexpr int kWaves = WM * WN;
    constexpr int TM = BM / WM / 32, TN = BN / WN / 32;
    typedef Fetch16<BM, kWaves> FA;
    typedef Fetch16<BN, kWaves, true> FB;
    constexpr int kA = BM * kAsyncK16, kB = BN * kAsyncK16;    // elements of a slab
    constexpr int kLoads = (kMask ? 2 : 1) * FA::kLoads + FB::kLoads;
    constexpr int kAhead = kStages - 1;
    constexpr int kStores = TM * TN * 8;                       // of a whole tile, at least
    constexpr int kYoung = (kAhead - 1) * kLoads;              // fetches that may be in flight behind a slab's own
    constexpr int kYoungStores = kYoung + kStores < 63 ? kYoung + kStores : 63;
    constexpr int kColChunks = Epi::kColAux ? (BN + 63) / 64 : 0, kRowChunks = Epi::kRowAux ? (BM + 63) / 64 : 0;
    constexpr int kAuxSlots = kStages;      // the cursor is kAhead slabs, so at most as many tiles, ahead
    static_assert(BM % (WM * 32) == 0 && BN % (WN * 32) == 0 && (WN == 1 || BN % (WN * 64) == 0) && kYoung <= 63 && kColChunks <= kWaves && kRowChunks <= kWaves, "tile shape");

    __shared__ __attribute__((aligned(1024))) uint16_t As[kStages][kA];
    __shared__ __attribute__((aligned(1024))) uint16_t Ms[kMask ? kStages : 1][kMask ? kA : 8];
    __shared__ __attribute__((aligned(1024))) uint16_t Bs[kStages][kB];
    __shared__ float col_aux[kAuxSlots][kColChunks * 64 + 1];
    __shared__ float row_aux[kAuxSlots][kRowChunks * 64 + 1];

    const int tid = threadIdx.x, lane = tid & 63, l31 = lane & 31, hi = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm0 = (wave / WN) * (BM / WM), wn0 = (wave % WN) * (BN / WN);

    const int64_t blocks_per_die = gridDim.x / kXcds;
    const int64_t per_die = (total_work + kXcds - 1) / kXcds;
    const int64_t die = blockIdx.x % kXcds;
    int64_t die_end = (die + 1) * per_die;
    if (die_end > total_work) die_end = total_work;
    int64_t work = die * per_die + blockIdx.x / kXcds;
    if (work >= die_end) return;

    // The last tile begins early enough to be whole: some rows are computed and stored twice, the same bits.  (Stored element by element under
    // comparisons a cut one was 5 us behind the others, 131,071 rows of 2 x 128 -> 256 59 us against 53 of 131,072.)
    const int64_t last_row = M > BM ? M - BM : 0;
    auto first_row = [&](int64_t item) { return item / n_tiles * BM < last_row ? item / n_tiles * BM : last_row; };

    // ---- the cursor: the slab that is fetched next
    const uint32_t as0 = lds_address(&As[0][0]), ms0 = lds_address(&Ms[0][0]), bs0 = lds_address(&Bs[0][0]);
    const int n_slabs = (a.K + kAsyncK16 - 1) / kAsyncK16;
    const int64_t to_mask = kMask ? reinterpret_cast<intptr_t>(mask) - reinterpret_cast<intptr_t>(a.P0) : 0;
    int64_t c_work = work, c_m0 = 0;
    int c_slab = 0, a_run = 0, b_run = 0, c_aux = 0, c_n0 = 0;
    uint32_t c_stage = 0;
    bool c_open = true;
    FA fa;
    FB fb;
    auto fetch_next = [&]() {
        if (!c_open) return;
        const uint32_t a_to = as0 + c_stage * uint32_t(kA * 2), m_to = ms0 + c_stage * uint32_t(kA * 2), b_to = bs0 + c_stage * uint32_t(kB * 2);
        if (c_slab == 0) {
            c_m0 = first_row(c_work);
            c_n0 = int(c_work % n_tiles) * BN;
            a_run = b_run = 0;
            // (chunks past the last are fetched again: the same values to the same place)
            if constexpr (kColChunks > 0) {
                const int c = wave % kColChunks * 64;
                lds_fetch<1>(lds_address(&col_aux[c_aux][0]) + c * 4, epi.col_at(c_n0 + c + lane < N ? c_n0 + c + lane : N - 1));
            }
            if constexpr (kRowChunks > 0) {
                const int r = wave % kRowChunks * 64;
                lds_fetch<1>(lds_address(&row_aux[c_aux][0]) + r * 4, epi.row_at(c_m0 + r + lane < M ? c_m0 + r + lane : M - 1));
            }
        }
        const int kt = c_slab * kAsyncK16;
        if (a_run == 0) {
            a_run = a.run(kt);
            if (a_run > 0) fa.enter_run(a, c_m0, kt, wave, lane);
        }
        if (b_run == 0) {
            b_run = b.run(kt);
            if (b_run > 0) fb.enter_run(b, c_n0, kt, wave, lane);
        }
        if (a_run > 0) {
            --a_run;
            fa.whole(a_to, fa.at, wave);
            if constexpr (kMask) fa.whole(m_to, reinterpret_cast<const uint16_t *>(reinterpret_cast<const char *>(fa.at) + to_mask), wave);
            fa.at += kAsyncK16;
        } else {
            FA::slowly(a, c_m0, kt, a_to, wave, lane);
            if constexpr (kMask) {
                AsyncRows16 m = a;
                m.P0 = mask;
                FA::slowly(m, c_m0, kt, m_to, wave, lane);
            }
        }
        if (b_run > 0) {
            --b_run;
            fb.whole(b_to, fb.at, wave);
            fb.at += kAsyncK16;
        } else {
            FB::slowly(b, c_n0, kt, b_to, wave, lane);
        }
        c_stage = c_stage == kStages - 1 ? 0 : c_stage + 1;
        if (++c_slab == n_slabs) {
            c_slab = 0;
            c_aux = c_aux == kAuxSlots - 1 ? 0 : c_aux + 1;
            c_work += blocks_per_die;
            c_open = c_work < die_end;
        }
    };
#pragma unroll
    for (int s = 0; s < kAhead; ++s) fetch_next();

    const int odd_at = a.Fv % 2 ? a.Fv : -1;     // the column of padding that came with a pair
    int stage = 0, aux = 0;
    int storing = 0;     // slabs that are waited for while the stores of a whole tile may be in flight behind their fetches
    const int swap = (l31 >> 2) & 3;
    const int piece[2] = {(hi ^ swap) * 8, ((2 + hi) ^ swap) * 8};
    const int a_frag = (wm0 + l31) * kAsyncK16, b_frag = (wn0 + l31) * kAsyncK16;
    for (;; work += blocks_per_die) {
        const int64_t m0 = first_row(work);
        const int n0 = int(work % n_tiles) * BN;
        floatx16 acc[TM][TN];
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

        for (int s = 0; s < n_slabs; ++s) {
            if (!c_open) wait_and_meet<0>();
            else if (storing > 0) wait_and_meet<kYoungStores>();
            else wait_and_meet<kYoung>();
            --storing;
            fetch_next();       // into the buffer that every wavefront has read before this meeting
            const uint16_t *A0 = &As[0][0] + stage * kA + a_frag, *M0 = &Ms[0][0] + (kMask ? stage * kA + a_frag : 0), *B0 = &Bs[0][0] + stage * kB + b_frag;
            uint4 xa[2][TM], xb[2][TN];
#pragma unroll
            for (int g = 0; g < 2; ++g) {
#pragma unroll
                for (int i = 0; i < TM; ++i) {
                    xa[g][i] = *reinterpret_cast<const uint4 *>(A0 + i * 32 * kAsyncK16 + piece[g]);
                    if constexpr (kMask) {
                        const uint4 h = *reinterpret_cast<const uint4 *>(M0 + i * 32 * kAsyncK16 + piece[g]);
                        xa[g][i] = make_uint4(where_positive(xa[g][i].x, h.x), where_positive(xa[g][i].y, h.y),
                                              where_positive(xa[g][i].z, h.z), where_positive(xa[g][i].w, h.w));
                    }
                }
#pragma unroll
                for (int j = 0; j < TN; ++j) xb[g][j] = *reinterpret_cast<const uint4 *>(B0 + j * 32 * kAsyncK16 + piece[g]);
            }
            if (odd_at >= s * kAsyncK16 && odd_at < (s + 1) * kAsyncK16) {
#pragma unroll
                for (int g = 0; g < 2; ++g) {
                    const int at = odd_at - s * kAsyncK16 - g * 16 - hi * 8;     // its place among this lane's eight
#pragma unroll
                    for (int i = 0; i < TM; ++i) {
                        xa[g][i].x &= at == 1 ? 0xFFFFu : ~0u;
                        xa[g][i].y &= at == 3 ? 0xFFFFu : ~0u;
                        xa[g][i].z &= at == 5 ? 0xFFFFu : ~0u;
                        xa[g][i].w &= at == 7 ? 0xFFFFu : ~0u;
                    }
                }
            }
#pragma unroll
            for (int g = 0; g < 2; ++g)
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, xa[g][i]), __builtin_bit_cast(bf16x8, xb[g][j]),
                                                                            acc[i][j], 0, 0, 0);
            stage = stage == kStages - 1 ? 0 : stage + 1;
        }

        // MFMA 32x32 result layout: register r of lane l holds row 8*(r/4) + 4*(l/32) + r%4, column l%32 of the fragments.  Of two fragments side by side
        // the first holds the even columns and the second the odd ones: a lane has both values of a pair, and a wavefront's store goes to two
        // whole lines of 128 bytes.  (With 32 neighbouring columns in a fragment pairs were traded between lanes through LDS, and a store went to
        // 64 bytes of four rows each: at 12,500,000 rows, so -> now, forward 128 -> 256 and 256 -> 256 3.02 -> 2.63 and 4.63 -> 4.26 ms, 256 -> 2 x 48
        // 1.82 -> 1.73, input gradient of 2 x 256 with ReLU 7.56 -> 7.04, of 256 from 2 x 48 2.08 -> 1.69.)
        auto column = [&](int j) { return wn0 + (j + 1 < TN || j % 2 == 1 ? j / 2 * 64 + 2 * l31 + j % 2 : j * 32 + l31); };
        float caux[TN];
#pragma unroll
        for (int j = 0; j < TN; ++j) caux[j] = Epi::kColAux ? col_aux[aux][column(j)] : 0.0f;
        const bool whole = m0 + BM <= M && n0 + BN <= N;
        const bool pairs = (kCut ? m0 + BM <= M && N % 2 == 0 : whole) && pairs_ok_of(epi);
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            float raux[16];
#pragma unroll
            for (int r = 0; r < 16; ++r) raux[r] = Epi::kRowAux ? row_aux[aux][wm0 + i * 32 + 8 * (r / 4) + 4 * hi + (r % 4)] : 0.0f;
            const int64_t row0 = m0 + wm0 + i * 32 + 4 * hi;
            auto value = [&](int j, int r) {
                const int col = n0 + column(j);
                return epi.value(epi.padding(col) ? 0.0f : acc[i][j][r], caux[j], raux[r], col);
            };
            if (pairs) {
#pragma unroll
                for (int j = 0; j < TN; j += 2) {
                    const int col = n0 + column(j);
                    if (kCut && col >= N) continue;
                    if (j + 1 < TN) {
#pragma unroll
                        for (int r = 0; r < 16; ++r) store_pair(epi, row0 + 8 * (r / 4) + r % 4, col, pack_bf16(value(j, r), value(j + 1 < TN ? j + 1 : j, r)));
                    } else {        // neighbouring lanes trade every other value (see gemm_bf16_kernel)
                        const int odd = l31 & 1;
                        const uint32_t select = traded_bytes(l31);
#pragma unroll
                        for (int r = 0; r < 16; r += 2)
                            store_pair(epi, row0 + 8 * (r / 4) + r % 4 + odd, col - odd, traded_pair(value(j, r), value(j, r + 1), select));
                    }
                }
            } else {
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    const int col = n0 + column(j);
                    if (col < N) {
#pragma unroll
                        for (int r = 0; r < 16; ++r) {
                            const int64_t row = row0 + 8 * (r / 4) + r % 4;
                            if (row < M) epi.store(row, col, value(j, r), 0);
                        }
                    }
                }
            }
        }
        storing = whole ? kAhead : 0;     // (fewer stores may not be counted on)
        aux = aux == kAuxSlots - 1 ? 0 : aux + 1;
        if (work + blocks_per_die >= die_end) break;
    }
}

template <int BM, int BN, int WM, int WN, int kStages, bool kMask, class Epi>
static void launch_async16(const char *what, const AsyncRows16 &a, const uint16_t *mask, const AsyncRows16 &b, const Epi &e, int64_t M, int N, bool paired, hipStream_t s)
{
    constexpr int kPerCu = 8 / (WM * WN);
    static_assert(kPerCu * kStages * ((kMask ? 2 : 1) * BM + BN) * 64 <= 152 * 1024, "LDS of the blocks of a unit");
    const int n_tiles = int(ceil_div(N, BN));
    const int64_t total = ceil_div(M, BM) * n_tiles;
    int64_t blocks_per_die = ceil_div(total, kXcds);
    if (blocks_per_die > 32 * kPerCu) blocks_per_die = 32 * kPerCu;
    char name[48];
    snprintf(name, sizeof(name), "%s_%dx%d_bf16", what, BM, BN);
    TMA_TIMED(name, s);
    const dim3 grid(unsigned(blocks_per_die * kXcds)), block(WM * WN * 64);
    if (N % BN == 0 || !paired)      // (where pairs are no words the other only costs: 273 from 128, 123,903 rows, with the weight gradient 162 / 179)
        hipLaunchKernelGGL((gemm_bf16_async_kernel<BM, BN, WM, WN, kStages, kMask, false, Epi>), grid, block, 0, s, a, mask, b, e, M, N, n_tiles, total);
    else
        hipLaunchKernelGGL((gemm_bf16_async_kernel<BM, BN, WM, WN, kStages, kMask, true, Epi>), grid, block, 0, s, a, mask, b, e, M, N, n_tiles, total);
}

// ---------------------------------------------------------------------------
// Weight gradients of bf16 storage: C[M,N] = A^T B summed over nodes, the k side, both operands rows of nodes.  They come into LDS as
// they lie, [32 nodes][columns], and ds_read_b64_tr_b16 turns them: of four nodes' 16 columns, which the lanes of a quarter
// wavefront address in pieces of four, each lane receives one column.  (gemm_bf16_kernel gathers the same fragments in eight
// 2-byte reads.)  The rest as in gemm_bf16_async_kernel: tiles of 256 rows of the result, so that the nodes' rows are read once or
// twice, and a ring of slabs that is bound by the memory alone.  12,500,000 nodes: 2 x 128 -> 256 and 2 x 256 -> 256 with ReLU 12.2 -> 9.5 ms
// (4.7 TB/s), 256 -> 2 x 48 2.9 -> 1.5; 1,500,000: 2 x 256 -> 256 without ReLU 846 -> 472 us (4.9 TB/s).
// ---------------------------------------------------------------------------

// X[k][c], columns of one or two parts of F each, padded to Fq (a multiple of eight): c < Fq ? P0[k][c] : P1[k][c-Fq].  What is read in the
// place of padding is anything: it reaches only results of its own column, which are not stored.
struct AsyncCols16 {
    const uint16_t *P0;
    int64_t ld0;
    const uint16_t *P1;
    int64_t ld1;
    int F, Fq, width;      // width: Fq or 2 Fq
    int64_t rows;
    __host__ __device__ __forceinline__ bool second(int c) const { return c >= Fq && c < width; }
    __host__ __device__ __forceinline__ int column(int c) const
    {
        const int cc = c - (second(c) ? Fq : 0);
        return cc < F ? cc : 0;
    }
    __host__ __device__ __forceinline__ int64_t ld(int c) const { return second(c) ? ld1 : ld0; }
    // column c of node k; eight from there on may be read if another row follows
    __host__ __device__ __forceinline__ const uint16_t *piece(int64_t k, int c) const { return (second(c) ? P1 : P0) + k * ld(c) + column(c); }
    // the pair of columns c, c + 1 (c even)
    __host__ __device__ __forceinline__ const uint16_t *at(int64_t k, int c, const void *zeros) const
    {
        return k < rows ? piece(k, c) : static_cast<const uint16_t *>(zeros);
    }
    __host__ bool ok() const
    {
        const auto even = [&](const uint16_t *p, int64_t l) { return (reinterpret_cast<uintptr_t>(p) & 3) == 0 && l % 2 == 0 && l >= F + F % 2 && l <= (1 << 21); };
        return F >= 8 && even(P0, ld0) && (width == Fq || even(P1, ld1));
    }
};

// A slab of 32 nodes and COLS columns on its way into LDS, [32][COLS], the groups of four pieces of a node's row exchanged by its number.
template <int COLS, int kWaves>
struct FetchCols16 {
    static constexpr int kPieces = COLS / 8, kI = kPieces / 2, kLoads = kI / kWaves;
    static_assert(kI % kWaves == 0 && kPieces >= 16 && (kPieces & (kPieces - 1)) == 0, "columns of a slab");
    const char *from[kLoads];
    uint32_t step[kLoads];
    // (16-byte place in the slab: its node, its first column)
    static __device__ __forceinline__ int node(int place) { return place / kPieces; }
    static __device__ __forceinline__ int column(int place) { return ((place % kPieces) ^ (4 * (node(place) & 3))) * 8; }
    __device__ __forceinline__ void enter(const AsyncCols16 &x, int64_t k, int c0, int wave, int lane)
    {
#pragma unroll
        for (int v = 0; v < kLoads; ++v) {
            const int place = (v * kWaves + wave) * 64 + lane, c = c0 + column(place);
            from[v] = reinterpret_cast<const char *>(x.piece(k + node(place), c));
            step[v] = uint32_t(x.ld(c)) * 2u * uint32_t(kAsyncK16);
        }
    }
    __device__ __forceinline__ void whole(uint32_t to, int64_t shift, int wave) const
    {
#pragma unroll
        for (int v = 0; v < kLoads; ++v) lds_fetch<4>(to + uint32_t(v * kWaves + wave) * 1024u, reinterpret_cast<const float *>(from[v] + shift));
    }
    __device__ __forceinline__ void advance()
    {
#pragma unroll
        for (int v = 0; v < kLoads; ++v) from[v] += step[v];
    }
    // any nodes, pair by pair
    __device__ __forceinline__ static void slowly(const AsyncCols16 &x, int64_t k, int c0, uint32_t to, int wave, int lane)
    {
#pragma unroll 1
        for (int v = 0; v < 4 * kLoads; ++v) {
            const int q = v * kWaves + wave, place = q * 16 + lane / 4;
            lds_fetch<1>(to + uint32_t(q) * 256u, reinterpret_cast<const float *>(x.at(k + node(place), c0 + column(place) + (lane & 3) * 2, kZeros)));
        }
    }
};

typedef short shortx4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) shortx4 lds_shortx4;
// eight k-values of a lane's column: of nodes 0..3 and 4..7 from `at` on, `row` elements apart
__device__ __forceinline__ uint4 turned(const uint16_t *at, int row)
{
    const uint2 lo = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_shortx4 *)(at)));
    const uint2 hi = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_shortx4 *)(at + 4 * row)));
    return make_uint4(lo.x, lo.y, hi.x, hi.y);
}
__device__ __forceinline__ float sum_of(const uint4 &v)
{
    const auto two = [](uint32_t w) { return __uint_as_float(w << 16) + __uint_as_float(w & 0xFFFF0000u); };
    return (two(v.x) + two(v.y)) + (two(v.z) + two(v.w));
}

// partial[split][m][n] and colsum_partial[split][n] (the sums over nodes of B); work items (split, m-tile, n-tile) numbered as in gemm_bf16_kernel
template <int BN, int WN, int kStages, bool kMask>
__global__ __launch_bounds__(256 * WN, WN == 2 ? 2 : 1) void gemm_bf16_weight_kernel(AsyncCols16 a, AsyncCols16 b, const uint16_t *mask,
                                                                                    int64_t k_per_split, int N, int n_tiles, int tiles,
                                                                                    int64_t total_work, float *__restrict__ partial,
                                                                                    float *__restrict__ colsum_partial)
{
    constexpr int BM = 256, kWaves = 4 * WN, TM = 2, TN = BN / WN / 32;
    typedef FetchCols16<BM, kWaves> FA;
    typedef FetchCols16<BN, kWaves> FB;
    constexpr int kA = BM * kAsyncK16, kB = BN * kAsyncK16;
    constexpr int kLoads = FA::kLoads + (kMask ? 2 : 1) * FB::kLoads, kAhead = kStages - 1, kYoung = (kAhead - 1) * kLoads;
    static_assert(TN == 4 && kYoung <= 63, "wavefront (m, n) sums column block m of its four");

    __shared__ __attribute__((aligned(1024))) uint16_t As[kStages][kA];
    __shared__ __attribute__((aligned(1024))) uint16_t Bs[kStages][kB];
    __shared__ __attribute__((aligned(1024))) uint16_t Ms[kMask ? kStages : 1][kMask ? kB : 8];

    const int tid = threadIdx.x, lane = tid & 63, l31 = lane & 31, hi = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave / WN, wn = wave % WN;

    const int64_t blocks_per_die = gridDim.x / kXcds;
    const int64_t per_die = (total_work + kXcds - 1) / kXcds;
    const int64_t die = blockIdx.x % kXcds;
    int64_t die_end = (die + 1) * per_die;
    if (die_end > total_work) die_end = total_work;
    int64_t work = die * per_die + blockIdx.x / kXcds;
    if (work >= die_end) return;

    const uint32_t as0 = lds_address(&As[0][0]), bs0 = lds_address(&Bs[0][0]), ms0 = lds_address(&Ms[0][0]);
    const int64_t nodes = a.rows, to_mask = kMask ? reinterpret_cast<intptr_t>(mask) - reinterpret_cast<intptr_t>(b.P0) : 0;
    auto end_of = [&](int64_t split) { return (split + 1) * k_per_split < nodes ? (split + 1) * k_per_split : nodes; };
    // ---- the cursor: the slab that is fetched next
    int64_t c_work = work, c_k = 0, c_end = 0;
    int c_m0 = 0, c_n0 = 0;
    uint32_t c_stage = 0;
    bool c_open = true, c_fresh = true;
    FA fa;
    FB fb;
    auto fetch_next = [&]() {
        if (!c_open) return;
        const uint32_t a_to = as0 + c_stage * uint32_t(kA * 2), b_to = bs0 + c_stage * uint32_t(kB * 2), m_to = ms0 + c_stage * uint32_t(kB * 2);
        if (c_fresh) {
            const int64_t split = c_work / tiles;
            const int tile = int(c_work % tiles);
            c_m0 = tile / n_tiles * BM;
            c_n0 = tile % n_tiles * BN;
            c_k = split * k_per_split;
            c_end = end_of(split);
            fa.enter(a, c_k, c_m0, wave, lane);
            fb.enter(b, c_k, c_n0, wave, lane);
            c_fresh = false;
        }
        if (c_k + kAsyncK16 < nodes) {     // (a piece may run past the end of its row: not in the last one)
            fa.whole(a_to, 0, wave);
            fb.whole(b_to, 0, wave);
            if constexpr (kMask) fb.whole(m_to, to_mask, wave);
            fa.advance();
            fb.advance();
        } else {
            FA::slowly(a, c_k, c_m0, a_to, wave, lane);
            FB::slowly(b, c_k, c_n0, b_to, wave, lane);
            if constexpr (kMask) {
                AsyncCols16 m = b;
                m.P0 = mask;
                FB::slowly(m, c_k, c_n0, m_to, wave, lane);
            }
        }
        c_stage = c_stage == kStages - 1 ? 0 : c_stage + 1;
        c_k += kAsyncK16;
        if (c_k >= c_end) {
            c_work += blocks_per_die;
            c_open = c_work < die_end;
            c_fresh = true;
        }
    };
#pragma unroll
    for (int s = 0; s < kAhead; ++s) fetch_next();

    // this lane's place in its quarter wavefront's 4 x 16 block, of nodes and columns as the fragment of a group wants them
    const int quarter = lane >> 4, i = lane & 15, swap = i >> 2;
    const int node0 = 8 * (quarter >> 1) + (i >> 2), col0 = 16 * (quarter & 1) + 4 * (i & 3);
    auto offset = [&](int block, int row) { return node0 * row + (((block & ~3) | ((block & 3) ^ swap)) * 32) + col0; };   // block: 32 columns
    int a_at[TM], b_at[TN];
#pragma unroll
    for (int t = 0; t < TM; ++t) a_at[t] = offset(wm * TM + t, BM);
#pragma unroll
    for (int t = 0; t < TN; ++t) b_at[t] = offset(wn * TN + t, BN);
    int stage = 0;
    for (;; work += blocks_per_die) {
        const int64_t split = work / tiles;
        const int tile = int(work % tiles), m0 = tile / n_tiles * BM, n0 = tile % n_tiles * BN;
        const int n_slabs = int((end_of(split) - split * k_per_split + kAsyncK16 - 1) / kAsyncK16);
        const bool sums = m0 == 0;
        float colsum = 0.0f;
        floatx16 acc[TM][TN];
#pragma unroll
        for (int t = 0; t < TM; ++t)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[t][j][r] = 0.0f;

        for (int s = 0; s < n_slabs; ++s) {
            if (!c_open) wait_and_meet<0>();
            else wait_and_meet<kYoung>();
            fetch_next();       // into the buffer that every wavefront has read before this meeting
            const uint16_t *A0 = &As[0][0] + stage * kA, *B0 = &Bs[0][0] + stage * kB, *M0 = &Ms[0][0] + (kMask ? stage * kB : 0);
#pragma unroll
            for (int g = 0; g < 2; ++g) {
                uint4 xa[TM], xb[TN];
#pragma unroll
                for (int t = 0; t < TM; ++t) xa[t] = turned(A0 + a_at[t] + g * 16 * BM, BM);
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    xb[j] = turned(B0 + b_at[j] + g * 16 * BN, BN);
                    if constexpr (kMask) {
                        const uint4 h = turned(M0 + b_at[j] + g * 16 * BN, BN);
                        xb[j] = make_uint4(where_positive(xb[j].x, h.x), where_positive(xb[j].y, h.y), where_positive(xb[j].z, h.z),
                                           where_positive(xb[j].w, h.w));
                    }
                }
#pragma unroll
                for (int t = 0; t < TM; ++t)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        acc[t][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, xa[t]), __builtin_bit_cast(bf16x8, xb[j]),
                                                                            acc[t][j], 0, 0, 0);
                if (sums) {
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        if (wm == j) colsum += sum_of(xb[j]);
                }
            }
            stage = stage == kStages - 1 ? 0 : stage + 1;
        }

        // MFMA 32x32 result layout: register r of lane l holds row 8*(r/4) + 4*(l/32) + r%4, column l%32.
        float *out = partial + split * int64_t(a.width == a.Fq ? a.F : 2 * a.F) * N;
#pragma unroll
        for (int t = 0; t < TM; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int m = m0 + (wm * TM + t) * 32 + 8 * (r / 4) + 4 * hi + r % 4;
                const int c = m - (a.second(m) ? a.Fq : 0);
                if (c < a.F && m < a.width) {
                    float *row = out + (c + (a.second(m) ? a.F : 0)) * int64_t(N);
#pragma unroll
                    for (int j = 0; j < TN; ++j) {
                        const int n = n0 + (wn * TN + j) * 32 + l31;
                        if (n < N) row[n] = acc[t][j][r];
                    }
                }
            }
        if (sums) {
            colsum += __shfl_xor(colsum, 32, kWave);
            const int n = n0 + (wn * TN + wm) * 32 + l31;
            if (hi == 0 && n < N) colsum_partial[split * N + n] = colsum;
        }
        if (work + blocks_per_die >= die_end) break;
    }
}

template <int BN, int WN, int kStages, bool kMask>
static void launch_weight16(const char *what, const AsyncCols16 &a, const AsyncCols16 &b, const uint16_t *mask, int N, int64_t k_per_split,
                            int n_splits, float *partial, float *colsum, hipStream_t s)
{
    static_assert(kStages * (256 + (kMask ? 2 : 1) * BN) * 64 <= 152 * 1024, "LDS of a unit");
    const int n_tiles = int(ceil_div(N, BN)), tiles = int(ceil_div(a.width, 256)) * n_tiles;
    const int64_t total = int64_t(tiles) * n_splits;
    int64_t blocks_per_die = ceil_div(total, kXcds);
    if (blocks_per_die > 32) blocks_per_die = 32;
    char name[48];
    snprintf(name, sizeof(name), "%s_256x%d_bf16", what, BN);
    TMA_TIMED(name, s);
    hipLaunchKernelGGL((gemm_bf16_weight_kernel<BN, WN, kStages, kMask>), dim3(unsigned(blocks_per_die * kXcds)), dim3(256 * WN), 0, s, a, b, mask,
                       k_per_split, N, n_tiles, tiles, total, partial, colsum);
}

}  // namespace tma
