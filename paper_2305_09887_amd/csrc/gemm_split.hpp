// The backward tile product of fp32 storage: fp32 operands, fp32-accurate results, on the bf16 matrix instruction.
// (Forward products, and backward ones of few rows, keep the fp32 instruction and its order of sums: see gemm_f32.hpp.)
//
// The fp32 matrix instruction multiplies at a sixteenth of the bf16 one's rate and bounded every wide fp32 product.
// Here each operand value is taken apart on its way into LDS into three bf16 values whose sum it is (x = h + m + l,
// each the rounding of what the ones before left over: 3 x 8 significant bits hold the 24), and a product becomes
// the six products of parts that reach fp32 accuracy,
//   a b = ah bh + (ah bm + am bh) + (am bm + ah bl + al bh) + ...,      the dropped rest below 2^-24 |a b|
// (two terms of up to 2^-25 near 1 + 2^-8 and a smaller one).  Splitting a number into parts of fewer bits by exact
// differences of roundings is a known method (Dekker, "A floating-point technique for extending the available precision",
// 1971); three parts are what a 24-bit significand takes.
// ah bh has accumulators of its own: the other five are 2^-8 and less of it, and added up beside it their roundings
// vanish, so that a k-group of 16 rounds the large sum once where the fp32 instruction rounds it eight times.
// Relative error of the sum against 64 bits, one 32x32 tile, fp32 instruction -> this, at K = 256 / 2,048 / 16,384:
// N(0,1) x 0.1 N(0,1) 2.9e-7 / 8.7e-7 / 2.3e-6 -> 0.9e-7 / 2.7e-7 / 0.8e-6; non-negative operands 2.3e-7 / 6.2e-7 /
// 1.7e-6 -> 0.9e-7 / 2.2e-7 / 0.6e-6; all six products in one accumulator would be no better than the fp32
// instruction.
//
// Range.  bf16 ends where fp32 does, so the smaller parts of a value below 2^-110 would end before its 24 bits do.  Values
// are multiplied by 2^24 before they are taken apart and the sum by 2^-48 at the end, both exact: the last bit of the
// smallest fp32 value is then a normal bf16 number.  At the other end a value without such parts (Inf, NaN, magnitudes from
// 2^104 on) or a sum from 2^80 on makes a result non-finite; a tile that would store one is multiplied again with the fp32
// instruction, so that large values, infinities, NaNs and overflows come out as they do there.
//
// Tiling: BM x BN block tile, k in slabs of 16 (one k-group), double-buffered in LDS with one barrier per slab,
// kDepth further slabs in flight in registers.  Both operands lie in LDS as [plane][mn][16 + 8] bf16: a row is twelve
// words, which spreads the 16-byte fragment reads, the 8-byte writes of k-contiguous operands and the 4-byte writes of
// transposed ones evenly over the banks.  An operand that is contiguous along mn is transposed on the way in: a
// thread holds two k-values of four neighbouring mn, and a bf16 pair along k costs the same to form as one along mn.
#pragma once

namespace tma {

constexpr int kSplitPerCu = 2;        // blocks per compute unit: two waves per SIMD of up to 256 registers
constexpr int kSlabK = 16;            // k-values per slab: one v_mfma_f32_32x32x16_bf16
constexpr int kSplitLd = kSlabK + 8;  // row pitch of a tile plane in bf16 values
constexpr int kFullLd = kSlabK + 4;   // row pitch in floats where a slab is staged unsplit
constexpr float kSplitScale = 0x1p24f, kSplitUnscale = 0x1p-48f;   // of both operands; of their product (see Range)

// two values -> their three parts as bf16 pairs (first value in the low half).  What a rounding left over is exact, and
// comes from one instruction: v - h as the dot product of the pair (h0, h1) with (-1, 0) or (0, -1), plus v.
struct SplitPair {
    typedef __bf16 Pair __attribute__((ext_vector_type(2)));
    uint32_t first, second;
    __device__ __forceinline__ SplitPair() : first(0x0000BF80u), second(0xBF800000u)
    {
        // held in registers: as an inline constant of this instruction -1.0 would stand in the other half
        asm("" : "+s"(first));
        asm("" : "+s"(second));
    }
    __device__ __forceinline__ float left(float v, uint32_t parts, uint32_t which) const
    {
        return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(Pair, parts), __builtin_bit_cast(Pair, which), v, false);
    }
    __device__ __forceinline__ void operator()(float x, float y, uint32_t &h, uint32_t &m, uint32_t &l) const
    {
        x *= kSplitScale;
        y *= kSplitScale;
        h = pack_bf16(x, y);
        x = left(x, h, first);
        y = left(y, h, second);
        m = pack_bf16(x, y);
        l = pack_bf16(left(x, m, first), left(y, m, second));
    }
};

// An optional member of an operand view: in_range(raw) is resolve(raw) for a k inside the operand; rows or columns past
// its end may then hold anything finite, since their results are not stored.
template <class View, class = void>
struct HasInRange : std::false_type {};
template <class View>
struct HasInRange<View, std::void_t<decltype(&View::in_range)>> : std::true_type {};
template <class View, bool kInRange>
__device__ __forceinline__ float4 operand_values(const typename View::Raw &r)
{
    if constexpr (kInRange && HasInRange<View>::value) return View::in_range(r);
    else return View::resolve(r);
}

// How the threads of a block share a slab of MN x 16 values of an operand: pieces of four k-values of one row, or of
// two k-values of four rows (64 consecutive threads then take 32 rows: 128-byte runs in memory, all banks in LDS).
template <class View, int MN, int NT>
struct SlabSlots {
    static constexpr int kPieces = View::kContigK ? MN * 4 : MN * 2;
    static constexpr int kSlots = (kPieces + NT - 1) / NT;
    static constexpr int kLoads = View::kContigK ? 1 : 2;
    static constexpr bool kEven = kPieces % NT == 0;
    static constexpr int kPlane = MN * kSplitLd;      // bf16 values of one plane
    typedef typename View::Raw Raws[kSlots][kLoads];

    typename View::Lane lane[kSlots];
    int mn[kSlots], k[kSlots];
    bool mine[kSlots];

    __device__ __forceinline__ void place(int tid)
    {
#pragma unroll
        for (int i = 0; i < kSlots; ++i) {
            const int p = tid + i * NT;
            mine[i] = kEven || p < kPieces;
            const int q = mine[i] ? p : 0;
            mn[i] = View::kContigK ? q / 4 : ((q / 32) * 4 + q % 4) * 4;
            k[i] = View::kContigK ? (q % 4) * 4 : ((q / 4) % 8) * 2;
        }
    }
    __device__ __forceinline__ void prepare(const View &v, int64_t mn0)
    {
#pragma unroll
        for (int i = 0; i < kSlots; ++i) lane[i] = v.prepare(mn0 + mn[i]);
    }
    template <bool kPlain>
    __device__ __forceinline__ void fetch(const View &v, int64_t kt, Raws &r) const
    {
#pragma unroll
        for (int i = 0; i < kSlots; ++i)
#pragma unroll
            for (int j = 0; j < kLoads; ++j)
                if constexpr (kPlain) r[i][j] = v.load_plain(lane[i], kt, k[i] + j);
                else r[i][j] = v.load(lane[i], kt + k[i] + j);
    }
    template <bool kInRange>
    __device__ __forceinline__ void stage(uint16_t *tile, const Raws &r, const SplitPair &split_pair) const
    {
#pragma unroll
        for (int i = 0; i < kSlots; ++i) {
            if (!mine[i]) continue;
            uint16_t *dst = tile + mn[i] * kSplitLd + k[i];
            const float4 v = operand_values<View, kInRange>(r[i][0]);
            if constexpr (View::kContigK) {
                uint2 h, m, l;
                split_pair(v.x, v.y, h.x, m.x, l.x);
                split_pair(v.z, v.w, h.y, m.y, l.y);
                *reinterpret_cast<uint2 *>(dst) = h;
                *reinterpret_cast<uint2 *>(dst + kPlane) = m;
                *reinterpret_cast<uint2 *>(dst + 2 * kPlane) = l;
            } else {
                const float4 w = operand_values<View, kInRange>(r[i][1]);
                const float lo[4] = {v.x, v.y, v.z, v.w}, hi[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    uint32_t h, m, l;
                    split_pair(lo[c], hi[c], h, m, l);
                    *reinterpret_cast<uint32_t *>(dst + c * kSplitLd) = h;
                    *reinterpret_cast<uint32_t *>(dst + c * kSplitLd + kPlane) = m;
                    *reinterpret_cast<uint32_t *>(dst + c * kSplitLd + 2 * kPlane) = l;
                }
            }
        }
    }
    __device__ __forceinline__ void stage_full(float *tile, const Raws &r) const   // the fp32 values as they are
    {
#pragma unroll
        for (int i = 0; i < kSlots; ++i) {
            if (!mine[i]) continue;
            float *dst = tile + mn[i] * kFullLd + k[i];
            const float4 v = View::resolve(r[i][0]);
            if constexpr (View::kContigK) {
                *reinterpret_cast<float4 *>(dst) = v;
            } else {
                const float4 w = View::resolve(r[i][1]);
                const float lo[4] = {v.x, v.y, v.z, v.w}, hi[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
                for (int c = 0; c < 4; ++c) *reinterpret_cast<float2 *>(dst + c * kFullLd) = make_float2(lo[c], hi[c]);
            }
        }
    }
};

// C[M,N] = A[M,K] B[K,N], k split into ranges of k_per_split; work items, their order over the dies, the fetch of the
// next tile's first slab ahead of the write-out and the unguarded loads of whole slabs as in gemm_bf16_kernel.
template <int BM, int BN, int WM, int WN, bool kColSum, class AL, class BL, class Epi>
__global__ __launch_bounds__(WM *WN * 64, kSplitPerCu) void gemm_split_kernel(AL a, BL b, Epi epi, int64_t M, int N, int64_t K,
                                                                    int64_t k_per_split, int n_tiles,
                                                                    int64_t tiles_per_split, int64_t total_work,
                                                                    float *__restrict__ colsum_partial)
{
    constexpr int NT = WM * WN * 64;
    // Slabs in flight in registers.  Two for a weight gradient, which streams both operands (us at 1,000,000 rows, one -> two:
    // 128 -> 128 335 -> 305, 128 -> 256 605 -> 545), and for the other products of four wavefronts in tiles below 128 x 128; one for the rest,
    // whose accumulators leave no registers for two (input gradient of 128 -> 128 401 with two, 383 with one, of 2 x 64 -> 100
    // with ReLU 493 and 474).  The unaligned views take registers of their own: one slab in the 128 x 128 tile (weight gradient of
    // 50 -> 128 at 125,237 rows 44 with two, 41 with one), and no set that lives across the barrier in the tiles of eight
    // wavefronts (47 -> 41 us the weight gradient of widths 90 -> 150 at 40,004 rows; the other views lose 5 to 20 % so).
    constexpr bool kUnaligned = std::is_same<typename AL::Raw, RawU>::value || std::is_same<typename BL::Raw, RawU>::value;
    constexpr int kDepth = (BM * BN < 128 * 128 && WM * WN == 4) || (kColSum && !(kUnaligned && WM * WN == 4)) ? 2 : 1;
    constexpr bool kLean = WM * WN == 8 && kUnaligned;
    constexpr int TM = BM / WM / 32;
    constexpr int TN = BN / WN / 32;
    typedef SlabSlots<AL, BM, NT> ASlots;
    typedef SlabSlots<BL, BN, NT> BSlots;
    static_assert(BM % (WM * 32) == 0 && BN % (WN * 32) == 0, "tile shape");
    static_assert(!kColSum || (!BL::kContigK && BSlots::kSlots == 1), "column sums are taken from a [k][n] operand");
    static_assert(kFullLd * sizeof(float) <= 2 * 3 * kSplitLd * sizeof(uint16_t), "an unsplit slab fits");

    __shared__ __attribute__((aligned(16))) uint16_t As[2][3 * ASlots::kPlane];
    __shared__ __attribute__((aligned(16))) uint16_t Bs[2][3 * BSlots::kPlane];
    __shared__ int odd_tile[WM * WN];
    float *const a_aux = reinterpret_cast<float *>(&As[0][0]);   // per-column / per-row epilogue inputs
    float *const b_aux = reinterpret_cast<float *>(&Bs[0][0]);

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int l31 = lane & 31;
    const int hi = lane >> 5;
    const int wave = tid >> 6;
    const int wm0 = (wave / WN) * (BM / WM);
    const int wn0 = (wave % WN) * (BN / WN);

    const SplitPair split_pair;
    ASlots as;
    BSlots bs;
    as.place(tid);
    bs.place(tid);

    const int64_t blocks_per_die = gridDim.x / kXcds;
    const int64_t per_die = (total_work + kXcds - 1) / kXcds;
    const int64_t die = blockIdx.x % kXcds;
    int64_t die_end = (die + 1) * per_die;
    if (die_end > total_work) die_end = total_work;

    struct Tile {
        int64_t m0;
        int n0, split;
        int64_t k_begin, k_end;
    };
    auto tile_of = [&](int64_t work) {
        Tile t;
        t.split = int(work / tiles_per_split);
        const int64_t tile = work % tiles_per_split;
        t.m0 = (tile / n_tiles) * BM;
        t.n0 = int(tile % n_tiles) * BN;
        t.k_begin = int64_t(t.split) * k_per_split;
        t.k_end = t.k_begin + k_per_split;
        if (t.k_end > K) t.k_end = K;
        return t;
    };
    auto fetch = [&](int64_t kt, typename ASlots::Raws &ar, typename BSlots::Raws &br) {   // any slab
        as.template fetch<false>(a, kt, ar);
        bs.template fetch<false>(b, kt, br);
    };
    auto fetch_whole = [&](int64_t kt, typename ASlots::Raws &ar, typename BSlots::Raws &br) {   // inside the k range
        as.template fetch<true>(a, kt, ar);
        bs.template fetch<true>(b, kt, br);
    };

    int64_t work = die * per_die + blockIdx.x / kXcds;
    if (work >= die_end) return;
    Tile t = tile_of(work);
    // first slab of the tile that comes next; the slabs inside a tile's main loop have registers of their own
    typename ASlots::Raws afirst;
    typename BSlots::Raws bfirst;
    as.prepare(a, t.m0);
    bs.prepare(b, t.n0);
    fetch(t.k_begin, afirst, bfirst);
    while (true) {
        floatx16 acc[TM][TN], rest[TM][TN];   // sums of the leading products, sums of the other five
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][j][r] = rest[i][j][r] = 0.0f;
        float4 colsum = zero4();
        const bool sums_columns = kColSum && t.m0 == 0;
        auto stage = [&](int buf, const typename ASlots::Raws &ar, const typename BSlots::Raws &br, auto in_range_tag) {
            constexpr bool kInRange = decltype(in_range_tag)::value;
            as.template stage<kInRange>(As[buf], ar, split_pair);
            bs.template stage<kInRange>(Bs[buf], br, split_pair);
            if constexpr (kColSum) {
                if (bs.mine[0]) {
                    const float4 v = BL::resolve(br[0][0]), w = BL::resolve(br[0][1]);
                    colsum.x += v.x + w.x;
                    colsum.y += v.y + w.y;
                    colsum.z += v.z + w.z;
                    colsum.w += v.w + w.w;
                }
            }
        };
        auto fragment = [](const uint16_t *p) { return __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(p)); };
        auto multiply = [&](int buf) {
            bf16x8 fa[3][TM], fb[3][TN];
#pragma unroll
            for (int p = 0; p < 3; ++p) {
#pragma unroll
                for (int i = 0; i < TM; ++i)
                    fa[p][i] = fragment(&As[buf][p * ASlots::kPlane + (wm0 + i * 32 + l31) * kSplitLd + 8 * hi]);
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    fb[p][j] = fragment(&Bs[buf][p * BSlots::kPlane + (wn0 + j * 32 + l31) * kSplitLd + 8 * hi]);
            }
            auto product = [&](int p, int q, floatx16(&c)[TM][TN]) {
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        c[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[p][i], fb[q][j], c[i][j], 0, 0, 0);
            };
            product(0, 0, acc);
            product(2, 0, rest);
            product(0, 2, rest);
            product(1, 1, rest);
            product(1, 0, rest);
            product(0, 1, rest);
        };

        __syncthreads();  // the previous tile's epilogue has finished reading LDS
        stage(0, afirst, bfirst, std::false_type{});
        __syncthreads();
        // Whole slabs: a body without branches, in which conversions and loads can pass behind the matrix work and every
        // wait counts exactly.
        const int n_whole = int((t.k_end - t.k_begin) / kSlabK);
        const bool tail = t.k_begin + int64_t(n_whole) * kSlabK < t.k_end;
        auto slab = [&](int s) { return t.k_begin + int64_t(s) * kSlabK; };
        int buf = 0;     // holds the slab that comes next
        if constexpr (kLean) {
            for (int s = 0; s + 1 < n_whole; ++s) {
                typename ASlots::Raws areg;
                typename BSlots::Raws breg;
                fetch_whole(slab(s + 1), areg, breg);
                multiply(buf);
                buf ^= 1;
                stage(buf, areg, breg, std::true_type{});
                __syncthreads();
            }
        } else if (n_whole > 1) {
            // Slab s >= 1 waits in register set (s - 1) % kDepth; its loads are issued kDepth iterations before it is staged.
            // Past the end the last slab is fetched again: steps without a fetch after the loop cost more (weight gradient of
            // 2 x 128 -> 256 at 125,237 rows 110 -> 119 us).
            typename ASlots::Raws areg[kDepth];
            typename BSlots::Raws breg[kDepth];
            auto at = [&](int s) { return slab(s < n_whole ? s : n_whole - 1); };
            static_for<kDepth>([&](auto d_tag) {
                constexpr int D = decltype(d_tag)::value;
                fetch_whole(at(D + 1), areg[D], breg[D]);
            });
            auto step = [&](int s, auto buf_tag, auto set_tag) {
                constexpr int kBuf = decltype(buf_tag)::value, kSet = decltype(set_tag)::value;
                multiply(kBuf);
                stage(1 - kBuf, areg[kSet], breg[kSet], std::true_type{});   // (last read before the previous barrier)
                fetch_whole(at(s + 1 + kDepth), areg[kSet], breg[kSet]);
                __syncthreads();
            };
            int s = 0;
            for (; s + 2 < n_whole; s += 2)
                static_for<2>([&](auto r_tag) {
                    constexpr int R = decltype(r_tag)::value;
                    step(s + R, std::integral_constant<int, R>{}, std::integral_constant<int, R % kDepth>{});
                });
            if (s + 1 < n_whole) step(s, std::integral_constant<int, 0>{}, std::integral_constant<int, 0>{});
            buf = (n_whole - 1) % 2;
        }
        if (n_whole > 0 && tail) {      // the last slab reaches past the end of k
            fetch(t.k_begin + int64_t(n_whole) * kSlabK, afirst, bfirst);
            multiply(buf);
            buf ^= 1;
            stage(buf, afirst, bfirst, std::false_type{});
            __syncthreads();
        }
        multiply(buf);
        __syncthreads();
        float odd = 0.0f;   // becomes NaN where a result is not finite
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    acc[i][j][r] = (acc[i][j][r] + rest[i][j][r]) * kSplitUnscale;
                    odd = fmaf(acc[i][j][r], 0.0f, odd);
                }
        bool stored_odd = false;
        if (__builtin_expect(__any(odd != 0.0f), 0)) {
            // Lanes outside the result do not count: they may hold sums of row padding, which nobody wrote (every tile of a
            // weight gradient of 150 columns in rows of 152 was multiplied twice for it).
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const bool in = t.n0 + wn0 + j * 32 + l31 < N &&
                                        t.m0 + wm0 + i * 32 + 8 * (r / 4) + 4 * hi + (r % 4) < M;
                        stored_odd |= in && acc[i][j][r] * 0.0f != 0.0f;
                    }
        }
        if (__any(stored_odd) && lane == 0) odd_tile[wave] = 1;
        else if (lane == 0) odd_tile[wave] = 0;
        __syncthreads();
        int redo = 0;
#pragma unroll
        for (int w = 0; w < WM * WN; ++w) redo |= odd_tile[w];
        if (__builtin_expect(redo, 0)) {
            float *const Af = reinterpret_cast<float *>(&As[0][0]);
            float *const Bf = reinterpret_cast<float *>(&Bs[0][0]);
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
#pragma unroll 1
            for (int64_t kt = t.k_begin; kt < t.k_end; kt += kSlabK) {
                typename ASlots::Raws ar;
                typename BSlots::Raws br;
                as.template fetch<false>(a, kt, ar);
                bs.template fetch<false>(b, kt, br);
                __syncthreads();
                as.stage_full(Af, ar);
                bs.stage_full(Bf, br);
                __syncthreads();
#pragma unroll
                for (int g = 0; g < kSlabK; g += 8) {   // the upper half of the wavefront takes the upper half of the group
                    float4 fa[TM], fb[TN];
#pragma unroll
                    for (int i = 0; i < TM; ++i)
                        fa[i] = *reinterpret_cast<const float4 *>(Af + (wm0 + i * 32 + l31) * kFullLd + g + 4 * hi);
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        fb[j] = *reinterpret_cast<const float4 *>(Bf + (wn0 + j * 32 + l31) * kFullLd + g + 4 * hi);
#pragma unroll
                    for (int i = 0; i < TM; ++i)
#pragma unroll
                        for (int j = 0; j < TN; ++j) {
                            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[i].x, fb[j].x, acc[i][j], 0, 0, 0);
                            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[i].y, fb[j].y, acc[i][j], 0, 0, 0);
                            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[i].z, fb[j].z, acc[i][j], 0, 0, 0);
                            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[i].w, fb[j].w, acc[i][j], 0, 0, 0);
                        }
                }
            }
            __syncthreads();
        }

        // Per-column / per-row epilogue inputs (bias, 1/deg) go through LDS (see gemm_bf16_kernel); the column sums'
        // eight parts (one per k-pair of the slab) meet there too.
        if (Epi::kColAux && tid < BN) a_aux[tid] = epi.col_aux(t.n0 + tid < N ? t.n0 + tid : N - 1);
        if (Epi::kRowAux && tid < BM) b_aux[tid] = epi.row_aux(t.m0 + tid < M ? t.m0 + tid : M - 1);
        if constexpr (kColSum) {
            static_assert(8 * BN * sizeof(float) <= 2 * 3 * BSlots::kPlane * sizeof(uint16_t) && !Epi::kRowAux, "sums fit");
            if (sums_columns && bs.mine[0]) *reinterpret_cast<float4 *>(b_aux + (bs.k[0] / 2) * BN + bs.mn[0]) = colsum;
        }
        if (Epi::kColAux || Epi::kRowAux || kColSum) __syncthreads();

        const Tile done = t;
        const int64_t next = work + blocks_per_die;
        const bool has_next = next < die_end;
        if (has_next) {   // its latency passes behind the write-out below
            t = tile_of(next);
            as.prepare(a, t.m0);
            bs.prepare(b, t.n0);
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
        if (kColSum && done.m0 == 0 && tid < BN && done.n0 + tid < N) {
            float s = 0.0f;
#pragma unroll
            for (int p = 0; p < 8; ++p) s += b_aux[p * BN + tid];
            colsum_partial[int64_t(done.split) * N + done.n0 + tid] = s;
        }
        if (!has_next) break;
        work = next;
    }
}

}  // namespace tma
