// Products of bf16 storage whose rows are nodes, on v_mfma_f32_32x32x16_bf16, both operands fetched straight into LDS as in
// gemm_f32_async.hpp: rows of bf16 along k, the nodes' from one or two arrays, the weights' from a narrowed copy.
//
// These products are bound by streaming the nodes' rows in and the results out (2 x 256 -> 256: 1.5 KB and 262 kFLOP a row, a
// third of the matrix rate at 5 TB/s).  What they need is bytes in flight at all times, so: tiles as wide as the result (every
// row is read once), a ring of slabs of 32 k-values fetched kStages - 1 ahead through tile boundaries (the next rows arrive
// while results are written), and no registers, conversions or LDS writes between memory and the matrix units.  A ReLU mask is
// applied to the fragments, from a third stream into LDS.
//
// Sums: groups of 16 k-values in order, one accumulator, as in gemm_bf16_kernel: the same bits.
#pragma once

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

// One operand's slabs of ROWS rows on their way into LDS, [ROWS][32], the 16-byte pieces of a row exchanged by its row number
// (fragment reads then spread over the banks): wavefront loads of 16 rows, kLoads of them by each wavefront.
template <int ROWS, int kWaves>
struct Fetch16 {
    static constexpr int kI = ROWS / 16, kLoads = (kI + kWaves - 1) / kWaves;   // (where they do not divide the last is fetched twice)
    const uint16_t *at;     // of the next slab of the run, of row 0 of the tile
    uint32_t off[kLoads];
    static __device__ __forceinline__ int load_of(int v, int wave) { return v * kWaves + wave < kI ? v * kWaves + wave : kI - 1; }
    static __device__ __forceinline__ int piece(int row, int slot) { return slot ^ ((row >> 1) & 3); }
    // `other`: an array in the place of the first part (the mask), of its pitch
    __device__ __forceinline__ void enter_run(const AsyncRows16 &x, int64_t m0, int kt, int wave, int lane)
    {
        const bool first = kt < x.F;
        at = first ? x.P0 + m0 * x.ld0 + kt : x.P1 + m0 * x.ld1 + (kt - x.F);
        const int64_t left = x.rows - 1 - m0;
#pragma unroll
        for (int v = 0; v < kLoads; ++v) {
            const int r = load_of(v, wave) * 16 + lane / 4, row = r < left ? r : int(left);
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
            lds_fetch<1>(to + uint32_t(q) * 256u, reinterpret_cast<const float *>(x.at(m0 + r, kt + piece(r, slot) * 8 + (lane & 3) * 2, kZeros)));
        }
    }
};

// the values of g where h > 0 (h NaN: not), zeros elsewhere; two bf16 in a word
__device__ __forceinline__ uint32_t where_positive(uint32_t g, uint32_t h)
{
    typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
    const u16x2 bits = __builtin_bit_cast(u16x2, h) - u16x2{1, 1};              // 0 .. 0x7F7F: positive, up to infinity
    const u16x2 one = __builtin_elementwise_min(__builtin_elementwise_sub_sat(u16x2{0x7F80, 0x7F80}, bits), u16x2{1, 1});
    return __builtin_bit_cast(uint32_t, u16x2(__builtin_bit_cast(u16x2, g) * one));
}

// C[M,N] = A[M,K] B[N,K]^T.  kMask: A's elements count where `mask`, an array like A's only part, is positive.  Persistent blocks
// over tiles numbered as in gemm_bf16_kernel, m then n.
template <int BM, int BN, int WM, int WN, int kStages, bool kMask, class Epi>
__global__ __launch_bounds__(WM *WN * 64, 2) void gemm_bf16_async_kernel(AsyncRows16 a, const uint16_t *mask, AsyncRows16 b, Epi epi, int64_t M, int N,
                                                                         int n_tiles, int64_t total_work)
{
    constexpr int kWaves = WM * WN;
    constexpr int TM = BM / WM / 32, TN = BN / WN / 32;
    typedef Fetch16<BM, kWaves> FA;
    typedef Fetch16<BN, kWaves> FB;
    constexpr int kA = BM * kAsyncK16, kB = BN * kAsyncK16;    // elements of a slab
    constexpr int kLoads = (kMask ? 2 : 1) * FA::kLoads + FB::kLoads;
    constexpr int kAhead = kStages - 1;
    constexpr int kStores = TM * TN * 8;                       // of a whole tile, at least
    constexpr int kYoung = (kAhead - 1) * kLoads;              // fetches that may be in flight behind a slab's own
    constexpr int kYoungStores = kYoung + kStores < 63 ? kYoung + kStores : 63;
    constexpr int kColChunks = Epi::kColAux ? (BN + 63) / 64 : 0, kRowChunks = Epi::kRowAux ? (BM + 63) / 64 : 0;
    constexpr int kAuxSlots = kStages;      // the cursor is kAhead slabs, so at most as many tiles, ahead
    static_assert(BM % (WM * 32) == 0 && BN % (WN * 32) == 0 && kYoung <= 63 && kColChunks <= kWaves && kRowChunks <= kWaves, "tile shape");

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
            c_m0 = (c_work / n_tiles) * BM;
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
    const int swap = (l31 >> 1) & 3;
    const int piece[2] = {(hi ^ swap) * 8, ((2 + hi) ^ swap) * 8};
    const int a_frag = (wm0 + l31) * kAsyncK16, b_frag = (wn0 + l31) * kAsyncK16;
    for (;; work += blocks_per_die) {
        const int64_t m0 = (work / n_tiles) * BM;
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

        // MFMA 32x32 result layout: register r of lane l holds row 8*(r/4) + 4*(l/32) + r%4, column l%32.
        float caux[TN];
#pragma unroll
        for (int j = 0; j < TN; ++j) caux[j] = Epi::kColAux ? col_aux[aux][wn0 + j * 32 + l31] : 0.0f;
        const bool whole = m0 + BM <= M && n0 + BN <= N;
        const bool pairs = whole && pairs_ok_of(epi);
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            float raux[16];
#pragma unroll
            for (int r = 0; r < 16; ++r) raux[r] = Epi::kRowAux ? row_aux[aux][wm0 + i * 32 + 8 * (r / 4) + 4 * hi + (r % 4)] : 0.0f;
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int col = n0 + wn0 + j * 32 + l31;
                const bool padding = epi.padding(col);
                const int64_t row0 = m0 + wm0 + i * 32 + 4 * hi;
                if (pairs) {        // neighbouring lanes trade every other value (see gemm_bf16_kernel)
                    const int odd = l31 & 1;
#pragma unroll
                    for (int r = 0; r < 16; r += 2) {
                        const float v0 = epi.value(padding ? 0.0f : acc[i][j][r], caux[j], raux[r], col);
                        const float v1 = epi.value(padding ? 0.0f : acc[i][j][r + 1], caux[j], raux[r + 1], col);
                        const float got = __shfl_xor(odd ? v0 : v1, 1, kWave);
                        store_pair(epi, row0 + 8 * (r / 4) + r % 4 + odd, col - odd, odd ? pack_bf16(got, v1) : pack_bf16(v0, got));
                    }
                } else if (col < N) {
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int64_t row = row0 + 8 * (r / 4) + r % 4;
                        const float val = epi.value(padding ? 0.0f : acc[i][j][r], caux[j], raux[r], col);
                        if (row < M) epi.store(row, col, val, 0);
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
static void launch_async16(const char *name, const AsyncRows16 &a, const uint16_t *mask, const AsyncRows16 &b, const Epi &e, int64_t M, int N, hipStream_t s)
{
    constexpr int kPerCu = 8 / (WM * WN);
    static_assert(kPerCu * kStages * ((kMask ? 2 : 1) * BM + BN) * 64 <= 152 * 1024, "LDS of the blocks of a unit");
    const int n_tiles = int(ceil_div(N, BN));
    const int64_t total = ceil_div(M, BM) * n_tiles;
    int64_t blocks_per_die = ceil_div(total, kXcds);
    if (blocks_per_die > 32 * kPerCu) blocks_per_die = 32 * kPerCu;
    TMA_TIMED(name, s);
    hipLaunchKernelGGL((gemm_bf16_async_kernel<BM, BN, WM, WN, kStages, kMask, Epi>), dim3(unsigned(blocks_per_die * kXcds)), dim3(WM * WN * 64), 0, s, a,
                       mask, b, e, M, N, n_tiles, total);
}

}  // namespace tma
