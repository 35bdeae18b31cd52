// The forward products of fp32 storage on v_mfma_f32_32x32x2_f32, their operands fetched straight into LDS.
//
// The order of the sums is the one of gemm_f32.hpp (c <- fma(a[k], b[k], c) for k = 0, 4, 1, 5, 2, 6, 3, 7 of every eight
// k-values, from one accumulator), and why the fp32 instruction is taken stands there.  That instruction runs on the vector
// units: every other vector instruction of the loop is taken off its time.  So operands go from memory to LDS without
// passing through registers (global_load_lds_dwordx4: no staging, no selects, no LDS writes), a slab's addresses are a scalar
// base and a lane's offset that stays (no vector arithmetic), and the slabs of all tiles of a block are one sequence
// through a ring of kStages buffers, fetched kStages - 1 ahead with one barrier per slab: the first slabs of a tile arrive
// while the results of the one before are written.
//
// us at 5,000 / 12,000 / 125,237 / 1,000,000 rows, 2 x 128 -> 256, staged through registers -> so, the product alone, called again and again:
//   26 -> 13 / 38 -> 20 / 171 -> 135 / 1,165 -> 1,030      (127 TFLOP/s; what a further slab adds is 150 TFLOP/s, 95 % of
//   the unit; zeros instead of random data 991: the rest is the write-out, 4 vector instructions a value, and power)
// In the headline step, after kernels that leave little of its operands in the caches, 125,237 rows take 174 -> 145 to 154.  Counters of
// that launch: 2.27 of 2.4 GHz, the matrix units busy in 75 % of its cycles; its 1,958 tiles are two rounds and a half of the 768 blocks
// that the chip holds, so that three rounds' time is paid (85 %).
// Small products are bound by what a slab takes one wavefront beside its 8 MFMAs: the scalar work of a fetch is kept to a
// handful of instructions (runs of slabs, a step apart): 16.8 -> 13.2 at 5,000 rows.
//
// Waits.  A wavefront's memory operations complete in order.  The fetches are written in assembler, with no register as
// their result, and the waits for them too: vmcnt counts the younger operations that may stay in flight, the next slabs' fetches
// and, in the first slabs of a tile, the stores of the one before.  (The compiler knows nothing of these fetches, so its own
// waits for loads are stricter than needed, never weaker.)
#pragma once

namespace tma {

typedef __attribute__((address_space(3))) const void lds_void;
__device__ __forceinline__ uint32_t lds_address(const void *p) { return uint32_t(reinterpret_cast<uintptr_t>((lds_void *)(p))); }

#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"   // (m0 is named as reserved: it is set, all the same, and the compiler sets it again for its own use)
// E elements per lane from base + the lane's offset in bytes, to consecutive LDS addresses from `lds` on
template <int E>
__device__ __forceinline__ void lds_fetch(uint32_t lds, const float *base, uint32_t offset)
{
    if constexpr (E == 4)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(offset), "s"(base) : "memory", "m0");
    else
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" ::"s"(lds), "v"(offset), "s"(base) : "memory", "m0");
}
template <int E>
__device__ __forceinline__ void lds_fetch(uint32_t lds, const float *p)
{
    if constexpr (E == 4)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds), "v"(p) : "memory", "m0");
    else
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off" ::"s"(lds), "v"(p) : "memory", "m0");
}
#pragma clang diagnostic pop
// All but this wavefront's kVm youngest memory operations are done, and its LDS reads; then the whole block meets.
template <int kVm>
__device__ __forceinline__ void wait_and_meet()
{
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(kVm) : "memory");
}

constexpr int kAsyncK = 16;            // k-values of a slab
static __device__ const float kZeros[4] = {0.0f, 0.0f, 0.0f, 0.0f};   // what positions outside an operand are fetched from

// Operands.  A slab that lies inside one array is fetched in pieces of four elements at any 4-byte-aligned address; one that
// does not (it straddles two arrays, or ends past the last k) lane by lane, element by element where pieces could straddle.

struct AsyncRows {  // A[m][k] = k < F ? H[m][k] : M[m][k-F]   for k < K  (K = 2F, or K = F and M is not read)
    const float *H;
    int64_t ldh;
    const float *M;
    int64_t ldm;
    int F, K;
    int64_t rows;
    bool near;       // offsets inside a tile of rows fit 32 bits
    AsyncRows(const float *H_, int64_t ldh_, const float *M_, int64_t ldm_, int F_, int K_, int64_t rows_)
        : H(H_), ldh(ldh_), M(M_), ldm(ldm_), F(F_), K(K_), rows(rows_), near(ldh_ <= (1 << 21) && ldm_ <= (1 << 21))
    {
    }
    // whole slabs from kt on that lie inside one array
    __host__ __device__ __forceinline__ int run(int kt) const { return near ? ((kt < F ? F : K) - kt) / kAsyncK : 0; }
    __host__ __device__ __forceinline__ bool pieces() const { return (F | K) % 4 == 0; }
    __host__ __device__ __forceinline__ const float *at(int64_t m, int k, const float *zeros) const
    {
        const int64_t row = m < rows ? m : rows - 1;
        return k < F ? H + row * ldh + k : k < K ? M + row * ldm + (k - F) : zeros;
    }
};

// kSide = false: B[k][n] = k < R ? W0[k][n] : W1[k-R][n]; true: B[k][n] = n < Np ? W0[k][n] : W1[k][n-Np].  Matrices of
// [R, N], k < K.  Columns past N read as anything finite or not: the epilogue clears what it stores of them.
template <bool kSide>
struct AsyncWeights {
    const float *W0, *W1;
    int R, N, K, Np;
    __host__ __device__ __forceinline__ int half(int n) const { return kSide && n >= Np && n < 2 * Np; }
    __host__ __device__ __forceinline__ int column(int n) const
    {
        const int c = n - (half(n) ? Np : 0);
        return c < N ? c : 0;
    }
    // whole slabs from kt on inside one matrix; a piece that runs past the end of a row, by three elements at most, must find other rows there:
    // one, two of two elements, three of one (256 -> 1, the last layer of a link decoder, 12,000 / 125,000 rows: 20.8 / 43.0 us with every slab lane by
    // lane, 10.9 / 25.7 so)
    __host__ __device__ __forceinline__ int run(int kt) const
    {
        const int end = (!kSide && kt >= R ? K : R) - (N % 4 == 0 ? 0 : N >= 3 ? 1 : 4 - N);
        return end > kt ? (end - kt) / kAsyncK : 0;
    }
    __host__ __device__ __forceinline__ bool pieces() const { return N % 4 == 0; }
    __host__ __device__ __forceinline__ const float *first(int kt) const
    {
        return !kSide && kt >= R ? W1 + int64_t(kt - R) * N : W0 + int64_t(kt) * N;
    }
    __host__ __device__ __forceinline__ const float *at(int k, int n, const float *zeros) const
    {
        if (k >= K) return zeros;
        if (kSide) return (half(n) ? W1 : W0) + int64_t(k) * N + column(n);
        return first(k) + column(n);
    }
};

// C[M,N] = A[M,K] B[K,N].  Persistent blocks over tiles numbered as in gemm_bf16_kernel, m then n.
// LDS: A [BM][16], the 16-byte pieces of a row exchanged by its row number so that the fragment reads (one row per lane)
// spread over the banks; B [16][BN].
template <int BM, int BN, int WM, int WN, int kStages, int kPerSimd, class BL, class Epi>
__global__ __launch_bounds__(WM *WN * 64, kPerSimd) void gemm_f32_async_kernel(AsyncRows a, BL b, Epi epi, int64_t M, int N, int n_tiles,
                                                                               int64_t total_work)
{
    constexpr int kWaves = WM * WN;
    constexpr int TM = BM / WM / 32, TN = BN / WN / 32;
    constexpr int kA = BM * kAsyncK, kB = BN * kAsyncK;        // elements of a slab
    constexpr int A_I = kA / 256, B_I = kB / 256;            // wavefront loads of a slab, in pieces of four
    constexpr int A_V = (A_I + kWaves - 1) / kWaves, B_V = (B_I + kWaves - 1) / kWaves;   // of one wavefront; where they do not
    constexpr int kLoads = A_V + B_V;                                                     // divide the last is fetched twice
    constexpr int kAhead = kStages - 1;
    constexpr int kStores = TM * TN * 16;
    constexpr int kYoung = (kAhead - 1) * kLoads;            // fetches that may be in flight behind a slab's own
    constexpr int kYoungStores = kYoung + kStores < 63 ? kYoung + kStores : 63;
    constexpr int kColChunks = Epi::kColAux ? (BN + 63) / 64 : 0, kRowChunks = Epi::kRowAux ? (BM + 63) / 64 : 0;
    constexpr int kAuxSlots = kStages;      // the cursor is kAhead slabs, so at most as many tiles, ahead
    static_assert(BM % (WM * 32) == 0 && BN % (WN * 32) == 0 && A_I * 256 == kA && B_I * 256 == kB && kYoung <= 63, "tile shape");

    __shared__ __attribute__((aligned(1024))) float As[kStages][kA];
    __shared__ __attribute__((aligned(1024))) float Bs[kStages][kB];
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

    // element e of A's slab is row e / 16, and this k
    auto k_of = [](int e) { return ((((e >> 2) & 3) ^ ((e >> 5) & 3)) << 2) | (e & 3); };
    const uint32_t as0 = lds_address(&As[0][0]), bs0 = lds_address(&Bs[0][0]);

    // ---- the cursor: the slab that is fetched next, in runs of slabs whose addresses are a scalar step apart
    const int n_slabs = (a.K + kAsyncK - 1) / kAsyncK;
    int64_t c_work = work, c_m0 = 0;
    int c_slab = 0, c_run = 0, c_aux = 0, c_n0 = 0;
    uint32_t c_stage = 0;
    bool c_open = true;
    const float *c_a = nullptr, *c_b = nullptr;
    uint32_t a_off[A_V], b_off[B_V];
    const float *b_col[B_V];
    auto enter_tile = [&]() {
        c_m0 = (c_work / n_tiles) * BM;
        c_n0 = int(c_work % n_tiles) * BN;
#pragma unroll
        for (int v = 0; v < B_V; ++v) {
            const int q = v * kWaves + wave, e = (q < B_I ? q : B_I - 1) * 256 + lane * 4;
            const int n = c_n0 + e % BN;
            b_off[v] = (uint32_t(e / BN) * uint32_t(b.N) + uint32_t(b.column(n))) * 4u;
            b_col[v] = b.half(n) ? b.W1 : b.W0;
        }
    };
    auto enter_run = [&](int kt) {
        const int ra = a.run(kt), rb = b.run(kt);
        c_run = ra < rb ? ra : rb;
        const bool first = kt < a.F;
        c_a = first ? a.H + c_m0 * a.ldh + kt : a.M + c_m0 * a.ldm + (kt - a.F);
        c_b = b.first(kt);
        const int64_t left = a.rows - 1 - c_m0;
#pragma unroll
        for (int v = 0; v < A_V; ++v) {
            const int q = v * kWaves + wave, e = (q < A_I ? q : A_I - 1) * 256 + lane * 4;
            const int row = e / kAsyncK < left ? e / kAsyncK : int(left);
            a_off[v] = (uint32_t(row) * uint32_t(first ? a.ldh : a.ldm) + uint32_t(k_of(e))) * 4u;
        }
    };
    // a slab lane by lane: any position
    auto fetch_slowly = [&](int kt, uint32_t a_to, uint32_t b_to) {
        if (a.pieces()) {
#pragma unroll
            for (int v = 0; v < A_V; ++v) {
                const int q = v * kWaves + wave < A_I ? v * kWaves + wave : A_I - 1, e = q * 256 + lane * 4;
                lds_fetch<4>(a_to + uint32_t(q) * 1024u, a.at(c_m0 + e / kAsyncK, kt + k_of(e), kZeros));
            }
        } else {
#pragma unroll 1
            for (int v = 0; v < 4 * A_V; ++v) {
                const int q = v * kWaves + wave < 4 * A_I ? v * kWaves + wave : 4 * A_I - 1, e = q * 64 + lane;
                lds_fetch<1>(a_to + uint32_t(q) * 256u, a.at(c_m0 + e / kAsyncK, kt + k_of(e), kZeros));
            }
        }
        if (b.pieces()) {
#pragma unroll
            for (int v = 0; v < B_V; ++v) {
                const int q = v * kWaves + wave < B_I ? v * kWaves + wave : B_I - 1, e = q * 256 + lane * 4;
                lds_fetch<4>(b_to + uint32_t(q) * 1024u, b.at(kt + e / BN, c_n0 + e % BN, kZeros));
            }
        } else {
#pragma unroll 1
            for (int v = 0; v < 4 * B_V; ++v) {
                const int q = v * kWaves + wave < 4 * B_I ? v * kWaves + wave : 4 * B_I - 1, e = q * 64 + lane;
                lds_fetch<1>(b_to + uint32_t(q) * 256u, b.at(kt + e / BN, c_n0 + e % BN, kZeros));
            }
        }
    };
    auto fetch_next = [&]() {
        if (!c_open) return;
        const uint32_t a_to = as0 + c_stage * uint32_t(kA * 4), b_to = bs0 + c_stage * uint32_t(kB * 4);
        if (c_slab == 0) {
            enter_tile();
            c_run = 0;
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
        if (c_run == 0) enter_run(c_slab * kAsyncK);
        if (c_run > 0) {
            --c_run;
#pragma unroll
            for (int v = 0; v < A_V; ++v) {
                const int q = v * kWaves + wave;
                lds_fetch<4>(a_to + uint32_t(q < A_I ? q : A_I - 1) * 1024u, c_a, a_off[v]);
            }
            c_a += kAsyncK;
#pragma unroll
            for (int v = 0; v < B_V; ++v) {
                const int q = v * kWaves + wave;
                const uint32_t to = b_to + uint32_t(q < B_I ? q : B_I - 1) * 1024u;
                if constexpr (std::is_same<BL, AsyncWeights<true>>::value)
                    lds_fetch<4>(to, reinterpret_cast<const float *>(reinterpret_cast<const char *>(b_col[v] + int64_t(c_slab) * kAsyncK * b.N) + b_off[v]));
                else lds_fetch<4>(to, c_b, b_off[v]);
            }
            c_b += int64_t(kAsyncK) * b.N;
        } else {
            fetch_slowly(c_slab * kAsyncK, a_to, b_to);
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

    int stage = 0, aux = 0;
    int storing = 0;     // slabs that are waited for while the stores of a whole tile may be in flight behind their fetches
    const int a_frag = (wm0 + l31) * kAsyncK, swap = (l31 >> 1) & 3;
    const int a_piece[2] = {(hi ^ swap) * 4, ((2 + hi) ^ swap) * 4};
    const int b_frag = 4 * hi * BN + wn0 + l31;
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
            const float *A0 = &As[0][0] + stage * kA + a_frag, *B0 = &Bs[0][0] + stage * kB + b_frag;
            float4 fa[2][TM];
            float fb[2][TN][4];
#pragma unroll
            for (int g = 0; g < 2; ++g) {
#pragma unroll
                for (int i = 0; i < TM; ++i) fa[g][i] = *reinterpret_cast<const float4 *>(A0 + i * 32 * kAsyncK + a_piece[g]);
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int q = 0; q < 4; ++q) fb[g][j][q] = B0[(g * 8 + q) * BN + j * 32];
            }
#pragma unroll
            for (int g = 0; g < 2; ++g)
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int i = 0; i < TM; ++i)
#pragma unroll
                        for (int j = 0; j < TN; ++j) {
                            const float av = q == 0 ? fa[g][i].x : q == 1 ? fa[g][i].y : q == 2 ? fa[g][i].z : fa[g][i].w;
                            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(av, fb[g][j][q], acc[i][j], 0, 0, 0);
                        }
            stage = stage == kStages - 1 ? 0 : stage + 1;
        }

        // MFMA 32x32 result layout: register r of lane l holds row 8*(r/4) + 4*(l/32) + r%4, column l%32.
        float caux[TN];
#pragma unroll
        for (int j = 0; j < TN; ++j) caux[j] = Epi::kColAux ? col_aux[aux][wn0 + j * 32 + l31] : 0.0f;
        const bool whole_rows = m0 + BM <= M;
        auto write_out = [&](auto rows_tag) {
            constexpr bool kWhole = decltype(rows_tag)::value;
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                float raux[16];
#pragma unroll
                for (int r = 0; r < 16; ++r) raux[r] = Epi::kRowAux ? row_aux[aux][wm0 + i * 32 + 8 * (r / 4) + 4 * hi + (r % 4)] : 0.0f;
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    const int col = n0 + wn0 + j * 32 + l31;
                    if (col < N) {
                        const bool padding = epi.padding(col);
#pragma unroll
                        for (int r = 0; r < 16; ++r) {
                            const int64_t row = m0 + wm0 + i * 32 + 8 * (r / 4) + 4 * hi + (r % 4);
                            const float val = epi.value(padding ? 0.0f : acc[i][j][r], caux[j], raux[r], col);
                            if (kWhole || row < M) epi.store(row, col, val, 0);
                        }
                    }
                }
            }
        };
        if (whole_rows) write_out(std::true_type{});
        else write_out(std::false_type{});
        storing = whole_rows && n0 + BN <= N ? kAhead : 0;     // (fewer stores may not be counted on)
        aux = aux == kAuxSlots - 1 ? 0 : aux + 1;
        if (work + blocks_per_die >= die_end) break;
    }
}

template <int BM, int BN, int WM, int WN, int kStages, int kPerSimd, class BL, class Epi>
static void launch_async(const char *name, const AsyncRows &a, const BL &b, const Epi &e, int64_t M, int N, hipStream_t s)
{
    constexpr int kPerCu = kPerSimd * 4 / (WM * WN);
    const int n_tiles = int(ceil_div(N, BN));
    const int64_t total = ceil_div(M, BM) * n_tiles;
    int64_t blocks_per_die = ceil_div(total, kXcds);
    if (blocks_per_die > 32 * kPerCu) blocks_per_die = 32 * kPerCu;
    TMA_TIMED(name, s);
    hipLaunchKernelGGL((gemm_f32_async_kernel<BM, BN, WM, WN, kStages, kPerSimd, BL, Epi>), dim3(unsigned(blocks_per_die * kXcds)),
                       dim3(WM * WN * 64), 0, s, a, b, e, M, N, n_tiles, total);
}

}  // namespace tma
