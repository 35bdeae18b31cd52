// The tile-product kernel template of libtma with its operand views, epilogues and launcher; included by the
// translation units that instantiate it (the GraphSAGE transforms, the dense / GCN transforms).
//
// Operands are described by small "view" structs that present concatenations ([H | M], [W_self ; W_neigh]), the ReLU
// mask and transposes as plain A[m][k], B[k][n], and results by an epilogue struct; three kernel templates take them:
// gemm_f32_kernel (gemm_f32.hpp) for the backward products of fp32 storage with few rows, gemm_split_kernel
// (gemm_split.hpp) for the other backward ones, gemm_bf16_kernel below for bf16 (v_mfma_f32_32x32x16_bf16, fp32 accumulation).
// The forward products of fp32 storage have a kernel with operands of its own (gemm_f32_async.hpp).
//
// Tiling of gemm_bf16_kernel.  BM x BN block tile, each wavefront owning a (BM/WM) x (BN/WN) patch of 32x32 MFMA
// tiles; k is consumed in slabs of BK through two LDS buffers (one barrier per slab) while the next slab's global
// loads are in flight in registers.  Every operand keeps in LDS the orientation it has in HBM, so all global->LDS
// traffic is 8-byte loads and 8-byte LDS writes:
//   k-contiguous operand : LDS [mn][BK+4]; a lane fetches eight k-values of its row with two 8-byte reads;
//   mn-contiguous operand: LDS [BK][MN+4]; a lane reads one element per k-value.
// Within a group of 16 k-values the lanes of the upper half take the upper half of the group, from both operands (any
// bijection of k is allowed as long as A and B agree).  Blocks are persistent and numbered so that the tiles sharing
// operand rows land on the same die (XCD) and hit its L2.
#pragma once
#include "kernels.hpp"

#include <string_view>
#include <type_traits>

namespace tma {

typedef float floatx16 __attribute__((ext_vector_type(16)));

// Which bf16 products keep two slabs in flight in registers (and then run two blocks per compute unit, 256 registers):
// the ones bound by streaming their operands.  Measured at n = 125,237 / 2,000,000 rows: forward 97 -> 79 us / 1.34 ->
// 1.06 ms, narrow input gradient 66 -> 48 us; the input-gradient product of the aggregate-first form loses with it
// (169 -> 190 us), which already runs two blocks per unit.
template <bool kColSum, bool kRowAux>
struct DeepPrefetch {
    static constexpr bool value = !kRowAux || kColSum;
};

// An operand that is contiguous along k and takes it from two arrays of different pitch
template <class View, class = void>
struct TwoSourcesAlongK : std::false_type {};
template <class View>
struct TwoSourcesAlongK<View, std::void_t<decltype(View::kTwoSources)>> : std::integral_constant<bool, View::kContigK> {};

constexpr int kPad = 4;   // LDS row padding in elements: keeps 8-byte alignment, spreads banks
constexpr int kXcds = 8;  // MI355X: 8 accelerator dies, workgroups are dealt round-robin to them

__device__ __forceinline__ float4 zero4() { return make_float4(0.0f, 0.0f, 0.0f, 0.0f); }

// f(integral_constant<int, 0>), ..., f(integral_constant<int, N - 1>): a loop whose index is a constant in the body
template <int N, class F>
__device__ __forceinline__ void static_for(F &&f)
{
    if constexpr (N > 0) {
        static_for<N - 1>(f);
        f(std::integral_constant<int, N - 1>{});
    }
}

struct PaddedRows;
struct CatWeightsRest;
struct RawU;
template <class View>
struct UnalignedGroups : std::is_same<typename View::Raw, RawU> {};
// Which bf16 products run the unrolled loop of gemm_bf16_kernel, three copies of whose body have to share the registers.
// Not views that load element by element (but for the weights of the 256-wide tile: its input gradient 256 -> 256 at
// 604,000 rows 914 against 779 us), which spill up to 900 registers there (us at 125,237 / 1,000,000 rows, the rolled
// loop against the unrolled one: weight gradient of 2 x 150 -> 150 with ReLU 357 / 3,090 against 964 / 8,960, of
// 2 x 90 -> 150 142 / 1,220 against 430 / 3,380); not PaddedRows (42 / 307 against 62 / 472, 130 -> 50); not gradients along k but for the
// 256-wide tile (input gradient of 128 -> 128 41 / 275 against 48 / 342, of 2 x 100 -> 128 with ReLU 57 / 410 against
// 72 / 524; the 256-wide one of 2 x 128 -> 256 with ReLU 73 / 515 against 68 / 484); not the forward product of two
// weight matrices with a rest of k (2 x 100 -> 128 36 / 271 against 45 / 315; without a rest, 2 x 64 -> 120, 34 / 226
// against 30 / 191); and not weights in unaligned groups in the 128 x 128 tile (forward 128 -> 150 46 / 191 against 64 / 281 at
// 125,237 / 600,000 rows).
template <int kBN, class AL, class BL>
struct SteadyLoop {
    static constexpr bool value = AL::kGroups && (BL::kGroups || kBN == 256) && !std::is_same<AL, PaddedRows>::value &&
                                  !std::is_same<BL, CatWeightsRest>::value && !(kBN == 128 && UnalignedGroups<BL>::value) &&
                                  !(AL::kMasks && AL::kContigK && kBN != 256);
};

// An optional member of an operand view: kPacksBf16 + packed(raw) say that the view's Raw already holds four bf16
// values the way a bf16 tile keeps them in LDS (bits unchanged), so a bf16 product stores them as they are instead
// of widening and rounding them again (the same bits either way).
template <class View, class = void>
struct PacksBf16 : std::false_type {};
template <class View>
struct PacksBf16<View, std::void_t<decltype(View::kPacksBf16)>> : std::integral_constant<bool, View::kPacksBf16> {};

// ---------------------------------------------------------------------------
// Storage types.  T = float (fp32 storage) or uint16_t (bf16 storage).  The
// views hand every operand over as fp32 quads (bf16 widened exactly); what sits
// in LDS is the kernel's business.  Results are rounded to bf16 (nearest even)
// on store.
// ---------------------------------------------------------------------------
template <typename T>
struct Pack4;
template <>
struct Pack4<float> {
    typedef float4 Packed;  // 16 bytes
    static __device__ __forceinline__ Packed load(const float *p)   // (the instruction needs 4-byte alignment only)
    {
        Packed v;
        __builtin_memcpy(&v, p, 16);
        return v;
    }
    static __device__ __forceinline__ float4 widen(const Packed &v) { return v; }
};
template <>
struct Pack4<uint16_t> {
    typedef uint2 Packed;  // 8 bytes
    static __device__ __forceinline__ Packed load(const uint16_t *p) { return *reinterpret_cast<const uint2 *>(p); }
    static __device__ __forceinline__ float4 widen(const Packed &v)
    {
        return make_float4(__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xFFFF0000u), __uint_as_float(v.y << 16),
                           __uint_as_float(v.y & 0xFFFF0000u));
    }
};
__device__ __forceinline__ float widen1(const float *p) { return *p; }
__device__ __forceinline__ float widen1(const uint16_t *p) { return bf16_to_f32(*p); }
__device__ __forceinline__ void narrow1(float *p, float v) { *p = v; }
__device__ __forceinline__ void narrow1(uint16_t *p, float v) { *p = f32_to_bf16(v); }

// ---------------------------------------------------------------------------
// Operand views.  A view presents its operand as X[mn][k].  Per thread and
// load slot the kernel calls prepare(mn) once per tile (everything that does
// not depend on k: row pointers, which half of a concatenation, validity), then
// load(lane, k) once per k-slab, which returns four consecutive elements along
// the view's contiguous direction (k when kContigK, else mn) as a Raw value;
// resolve(raw) turns it into fp32 operand values, zero outside the operand.
// The split lets the kernel issue the loads of the next slab before the MFMAs of
// the current one and touch the loaded registers (widening, ReLU mask, ragged
// tails) only afterwards, so no wait on global memory sits in front of the
// matrix work.  V = the vector path is legal (bases aligned to four elements,
// leading dimensions and inner extents multiples of 4); its loads are
// branch-free: an out-of-range position is clamped to a valid address and the
// value is discarded by resolve() through the `ok` flag.  fp32 loads need only
// the extents; alignment and leading dimension are free.  Without V the view
// loads element by element, guarded; fp32 operands whose extents are no
// multiples of four have views of their own (see RawU), and take that way only
// when an array is too small for those.
// ---------------------------------------------------------------------------
template <typename T, bool V>
struct RawV {
    typename Pack4<T>::Packed v;
    bool ok;
    __device__ __forceinline__ float4 get() const
    {
        const float4 f = Pack4<T>::widen(v);
        return make_float4(ok ? f.x : 0.0f, ok ? f.y : 0.0f, ok ? f.z : 0.0f, ok ? f.w : 0.0f);
    }
    __device__ __forceinline__ float4 any() const { return Pack4<T>::widen(v); }
};
template <typename T>
struct RawV<T, false> {  // element-wise path: already fp32, already zero outside
    float4 v;
    bool ok;
    __device__ __forceinline__ float4 get() const { return v; }
    __device__ __forceinline__ float4 any() const { return v; }
};

// fp32 arrays whose rows are not multiples of four (F_out = 47): four consecutive elements starting at
// element e of an array of `count` >= 4 elements, fetched with one 16-byte load from a base that is
// only 4-byte aligned (the load instruction needs no more), unconditionally.  A group that would run past the
// end of the array is fetched `shift` elements earlier and moved back in registers; `valid` leading elements are
// kept, the rest read as zero.
struct RawU {
    float4 v;
    int meta;  // valid (0..4) | shift (0..3) << 4
    __device__ __forceinline__ float4 get() const
    {
        const int valid = meta & 15;
        float4 t = v;
        if (meta & 16) t = make_float4(t.y, t.z, t.w, 0.0f);
        if (meta & 32) t = make_float4(t.z, t.w, 0.0f, 0.0f);
        return make_float4(valid > 0 ? t.x : 0.0f, valid > 1 ? t.y : 0.0f, valid > 2 ? t.z : 0.0f, valid > 3 ? t.w : 0.0f);
    }
};
__device__ __forceinline__ RawU load_unaligned4(const float *base, int e, int count, int valid)
{
    const int over = e + 4 - count;
    const int shift = over > 0 ? over : 0;
    RawU r;
    __builtin_memcpy(&r.v, base + (e - shift), 16);
    r.meta = (valid < 4 ? valid : 4) | (shift << 4);
    return r;
}
// the same from p, of whose row `room` elements are left in the array (past the end of a row that is not the last one
// the group runs into the next row)
__device__ __forceinline__ RawU load_unaligned4_at(const float *p, int room, int valid)
{
    const int shift = room < 4 ? 4 - room : 0;
    RawU r;
    __builtin_memcpy(&r.v, p - shift, 16);
    r.meta = (valid < 0 ? 0 : valid < 4 ? valid : 4) | (shift << 4);
    return r;
}
enum : int { kElementwise = 0, kAligned4 = 1, kUnaligned4 = 2 };   // how a weight view fetches its groups of four

template <typename T, bool V>
struct CatRows {  // A[m][k] = k < F ? H[m][k] : M[m][k-F]  for k < Kv, zero beyond    (contiguous along k)
    static constexpr bool kContigK = true;
    static constexpr bool kMasks = false;
    static constexpr bool kGroups = V;
    typedef RawV<T, V> Raw;
    struct Lane {
        const T *p0, *p1;  // row pointers such that element k is p0[k] (k < F) or p1[k] (k >= F)
        bool ok;
    };
    const T *H;
    int64_t ldh;
    const T *Mx;
    int64_t ldm;
    int F;
    int64_t rows;
    int Kv;  // extent of k: 2F for the concatenation, F when only the first part is used (Mx is then never read)
    static __device__ __forceinline__ float4 resolve(const Raw &r) { return r.get(); }
    static constexpr bool kPacksBf16 = V && sizeof(T) == 2;
    static __device__ __forceinline__ uint2 packed(const Raw &r)
    {
        if constexpr (kPacksBf16) return make_uint2(r.ok ? r.v.x : 0u, r.ok ? r.v.y : 0u);
        else return make_uint2(0u, 0u);
    }
    __device__ __forceinline__ Lane prepare(int64_t m) const
    {
        const int64_t mm = m < rows ? m : 0;
        return Lane{H + mm * ldh, Mx + mm * ldm - F, m < rows};
    }
    __device__ __forceinline__ float at(const Lane &l, int k) const
    {
        return k < Kv ? (k < F ? widen1(l.p0 + k) : widen1(l.p1 + k)) : 0.0f;
    }
    __device__ __forceinline__ Raw load(const Lane &l, int64_t k64) const
    {
        const int k = int(k64);
        Raw r;
        r.ok = l.ok && k < Kv;
        if constexpr (V) {
            const int kc = k < Kv ? k : 0;
            r.v = Pack4<T>::load((kc < F ? l.p0 : l.p1) + kc);
        } else {
            r.v = r.ok ? make_float4(at(l, k), at(l, k + 1), at(l, k + 2), at(l, k + 3)) : zero4();
        }
        return r;
    }
    __device__ __forceinline__ Raw load_plain(const Lane &l, int64_t kt, int dk) const
    {
        if constexpr (V) {
            const int k = int(kt) + dk;
            Raw r;
            r.ok = l.ok;
            r.v = Pack4<T>::load((k < F ? l.p0 : l.p1) + k);
            return r;
        } else {
            return load(l, kt + dk);
        }
    }
};

// bf16 rows whose width is no multiple of four, in rows padded to one: the padding comes in with the last group and is
// masked there, whatever it holds (against the zero rows of the other operand a NaN would still be one).
struct PaddedRows {  // A[m][k] = H[m][k] for k < F, zero beyond    (contiguous along k)
    static constexpr bool kContigK = true;
    static constexpr bool kMasks = false;
    static constexpr bool kGroups = true;
    static constexpr bool kPacksBf16 = true;
    struct Raw {
        uint2 v;
        int valid;   // leading elements that are inside the operand (<= 0: none)
    };
    struct Lane {
        const uint16_t *p;
        bool ok;
    };
    const uint16_t *H;
    int64_t ldh;
    int F;
    int64_t rows;
    static __device__ __forceinline__ uint2 packed(const Raw &r)
    {
        return make_uint2(r.v.x & (r.valid > 1 ? ~0u : r.valid > 0 ? 0xFFFFu : 0u),
                          r.v.y & (r.valid > 3 ? ~0u : r.valid > 2 ? 0xFFFFu : 0u));
    }
    static __device__ __forceinline__ float4 resolve(const Raw &r) { return Pack4<uint16_t>::widen(packed(r)); }
    __device__ __forceinline__ Lane prepare(int64_t m) const { return Lane{H + (m < rows ? m : 0) * ldh, m < rows}; }
    __device__ __forceinline__ Raw load(const Lane &l, int64_t k64) const
    {
        const int k = int(k64);
        return Raw{Pack4<uint16_t>::load(l.p + (k < F ? k : 0)), l.ok ? F - k : 0};
    }
    __device__ __forceinline__ Raw load_plain(const Lane &l, int64_t kt, int dk) const
    {
        return Raw{Pack4<uint16_t>::load(l.p + kt + dk), l.ok ? 4 : 0};
    }
};

template <typename T, bool V>
struct CatRowsT {  // A[m][k] = m < F ? H[k][m] : M[k][m-F]  for m < Mv   (contiguous along m); k = node
    static constexpr bool kContigK = false;
    static constexpr bool kMasks = false;
    static constexpr bool kGroups = V;
    typedef RawV<T, V> Raw;
    struct Lane {
        const T *p;  // column pointer: element of node k is p[k * ld]
        int64_t ld;
        int m;
        bool ok;
    };
    const T *H;
    int64_t ldh;
    const T *Mx;
    int64_t ldm;
    int F;
    int64_t rows;
    int Mv;  // extent of m: 2F for the concatenation, F when only the first part is used (Mx is then never read)
    static __device__ __forceinline__ float4 resolve(const Raw &r) { return r.get(); }
    static __device__ __forceinline__ float4 in_range(const Raw &r) { return r.any(); }
    __device__ __forceinline__ Lane prepare(int64_t m64) const
    {
        const int m = int(m64);
        if (m < F) return Lane{H + m, ldh, m, true};
        if (m < Mv) return Lane{Mx + (m - F), ldm, m, true};
        return Lane{H, ldh, m, false};   // (the first column, and discarded)
    }
    __device__ __forceinline__ float at(int64_t node, int m) const
    {
        if (m < F) return widen1(H + node * ldh + m);
        if (m < Mv) return widen1(Mx + node * ldm + (m - F));
        return 0.0f;
    }
    __device__ __forceinline__ Raw load(const Lane &l, int64_t node) const
    {
        Raw r;
        r.ok = l.ok && node < rows;
        if constexpr (V) {
            r.v = Pack4<T>::load(l.p + (node < rows ? node : 0) * l.ld);
        } else {
            r.v = r.ok ? make_float4(at(node, l.m), at(node, l.m + 1), at(node, l.m + 2), at(node, l.m + 3)) : zero4();
        }
        return r;
    }
    __device__ __forceinline__ Raw load_plain(const Lane &l, int64_t kt, int dk) const
    {
        if constexpr (V) {
            Raw r;
            r.ok = l.ok;
            r.v = Pack4<T>::load(l.p + (kt + dk) * l.ld);
            return r;
        } else {
            return load(l, kt + dk);
        }
    }
};

template <bool V>
struct CatWeights {  // B[k][n] = k < F ? W_self[k][n] : W_neigh[k-F][n]  (contiguous along n); fp32 master weights
    static constexpr bool kContigK = false;
    static constexpr bool kGroups = V;
    typedef RawV<float, V> Raw;
    struct Lane {
        int n;
    };
    const float *Ws;
    const float *Wn;
    int F;
    int N;
    static __device__ __forceinline__ float4 resolve(const Raw &r) { return r.get(); }
    __device__ __forceinline__ Lane prepare(int64_t n) const { return Lane{int(n)}; }
    __device__ __forceinline__ Raw load(const Lane &l, int64_t k64) const
    {
        const int n = l.n, k = int(k64);
        Raw r;
        r.ok = k < 2 * F && n < N;
        const int kc = k < 2 * F ? k : 0;
        const float *row = kc < F ? Ws + int64_t(kc) * N : Wn + int64_t(kc - F) * N;
        if constexpr (V) {
            r.v = Pack4<float>::load(row + (n < N ? n : 0));
        } else if (r.ok) {
            r.v.x = row[n];
            r.v.y = n + 1 < N ? row[n + 1] : 0.0f;
            r.v.z = n + 2 < N ? row[n + 2] : 0.0f;
            r.v.w = n + 3 < N ? row[n + 3] : 0.0f;
        } else {
            r.v = zero4();
        }
        return r;
    }
    __device__ __forceinline__ Raw load_plain(const Lane &l, int64_t kt, int dk) const
    {
        if constexpr (V) {
            Raw r;
            r.ok = l.n < N;
            const int64_t e = kt * N + (dk * N + (l.n < N ? l.n : 0));   // (rows of a slab: below 2^31 elements)
            r.v = Pack4<float>::load((kt + dk < F ? Ws : Wn - int64_t(F) * N) + e);
            return r;
        } else {
            return load(l, kt + dk);
        }
    }
};

struct CatWeightsRest : CatWeights<true> {};   // the same for a k that is no multiple of a slab: see SteadyLoop

template <bool V>
struct CatWeightsT {  // B[k][n] = n < F ? W_self[n][k] : W_neigh[n-F][k]  (contiguous along k); k = output feature
    static constexpr bool kContigK = true;
    static constexpr bool kGroups = V;
    typedef RawV<float, V> Raw;
    struct Lane {
        const float *row;
        bool ok;
    };
    const float *Ws;
    const float *Wn;
    int F;
    int Fo;
    static __device__ __forceinline__ float4 resolve(const Raw &r) { return r.get(); }
    static __device__ __forceinline__ float4 in_range(const Raw &r) { return r.any(); }
    __device__ __forceinline__ Lane prepare(int64_t n64) const
    {
        const int n = int(n64);
        if (n < F) return Lane{Ws + int64_t(n) * Fo, true};
        return Lane{Wn + int64_t(n < 2 * F ? n - F : 0) * Fo, n < 2 * F};
    }
    __device__ __forceinline__ Raw load(const Lane &l, int64_t k64) const
    {
        const int k = int(k64);
        Raw r;
        r.ok = l.ok && k < Fo;
        if constexpr (V) {
            r.v = Pack4<float>::load(l.row + (k < Fo ? k : 0));
        } else if (r.ok) {
            r.v.x = l.row[k];
            r.v.y = k + 1 < Fo ? l.row[k + 1] : 0.0f;
            r.v.z = k + 2 < Fo ? l.row[k + 2] : 0.0f;
            r.v.w = k + 3 < Fo ? l.row[k + 3] : 0.0f;
        } else {
            r.v = zero4();
        }
        return r;
    }
    __device__ __forceinline__ Raw load_plain(const Lane &l, int64_t kt, int dk) const
    {
        if constexpr (V) {
            Raw r;
            r.ok = l.ok;
            r.v = Pack4<float>::load(l.row + kt + dk);
            return r;
        } else {
            return load(l, kt + dk);
        }
    }
};

// dZ = dHnext (.) [Hnext > 0] (ReLU) or dHnext (identity); rows = nodes, [rows, Fo] with leading dimension ld.
// kAsA: used as A[m=node][k=o] (contiguous along k).  Otherwise as B[k=node][n=o] (contiguous along n).
// The vector path may read up to three padding elements past Fo inside a row (ld is a multiple of 4);
// resolve() discards them.
template <bool kAsA, typename T, bool V, bool kRelu>
struct MaskedGrad {
    static constexpr bool kContigK = kAsA;
    static constexpr bool kMasks = true;
    static constexpr bool kGroups = V;
    typedef typename std::conditional<V, typename Pack4<T>::Packed, float4>::type Quad;
    struct RawRelu {
        Quad g, h;
        int nv;  // leading elements that are inside the operand (<= 0: none)
    };
    struct RawPlain {
        Quad g;
        int nv;
    };
    typedef typename std::conditional<kRelu, RawRelu, RawPlain>::type Raw;
    struct Lane {
        int64_t off;  // kAsA: node * ld ; else: o
        bool ok;
    };
    const T *dHn;
    const T *Hn;  // forward output; read only with ReLU
    int Fo;
    int64_t ld;
    int64_t rows;
    static __device__ __forceinline__ float4 quad(const Quad &q)
    {
        if constexpr (V) return Pack4<T>::widen(q);
        else return q;
    }
    static __device__ __forceinline__ float4 resolve(const Raw &r)
    {
        const float4 g = quad(r.g);
        if constexpr (kRelu) {
            const float4 h = quad(r.h);
            return make_float4((r.nv > 0 && h.x > 0.0f) ? g.x : 0.0f, (r.nv > 1 && h.y > 0.0f) ? g.y : 0.0f,
                               (r.nv > 2 && h.z > 0.0f) ? g.z : 0.0f, (r.nv > 3 && h.w > 0.0f) ? g.w : 0.0f);
        } else {
            return make_float4(r.nv > 0 ? g.x : 0.0f, r.nv > 1 ? g.y : 0.0f, r.nv > 2 ? g.z : 0.0f,
                               r.nv > 3 ? g.w : 0.0f);
        }
    }
    __device__ __forceinline__ Lane prepare(int64_t mn) const
    {
        if (kAsA) return Lane{(mn < rows ? mn : 0) * ld, mn < rows};
        return Lane{mn < Fo ? mn : 0, mn < Fo};
    }
    __device__ __forceinline__ Raw load(const Lane &l, int64_t k) const
    {
        Raw r;
        const int o = int(kAsA ? k : l.off);
        const bool inside = kAsA ? (l.ok && o < Fo) : (l.ok && k < rows);
        r.nv = inside ? Fo - o : 0;
        if constexpr (V) {
            const int64_t e = kAsA ? l.off + (o < Fo ? o : 0) : (k < rows ? k : 0) * ld + o;
            r.g = Pack4<T>::load(dHn + e);
            if constexpr (kRelu) r.h = Pack4<T>::load(Hn + e);
        } else {
            r.g = zero4();
            if constexpr (kRelu) r.h = zero4();
            if (inside) {
                const int64_t e = kAsA ? l.off + o : k * ld + o;
                r.g.x = widen1(dHn + e);
                if (o + 1 < Fo) r.g.y = widen1(dHn + e + 1);
                if (o + 2 < Fo) r.g.z = widen1(dHn + e + 2);
                if (o + 3 < Fo) r.g.w = widen1(dHn + e + 3);
                if constexpr (kRelu) {
                    r.h.x = widen1(Hn + e);
                    if (o + 1 < Fo) r.h.y = widen1(Hn + e + 1);
                    if (o + 2 < Fo) r.h.z = widen1(Hn + e + 2);
                    if (o + 3 < Fo) r.h.w = widen1(Hn + e + 3);
                }
            }
        }
        return r;
    }
    __device__ __forceinline__ Raw load_plain(const Lane &l, int64_t kt, int dk) const
    {
        if constexpr (V) {
            Raw r;
            int64_t e;
            if (kAsA) {   // k = output feature, whole groups of four inside [0, Fo)
                r.nv = l.ok ? 4 : 0;
                e = l.off + kt + dk;
            } else {      // k = node
                r.nv = l.ok ? Fo - int(l.off) : 0;
                e = kt * ld + (dk * ld + l.off);
            }
            r.g = Pack4<T>::load(dHn + e);
            if constexpr (kRelu) r.h = Pack4<T>::load(Hn + e);
            return r;
        } else {
            return load(l, kt + dk);
        }
    }
};

// ---------------------------------------------------------------------------
// Views for the transform-before-aggregate form of the layer (F_out much smaller
// than F_in):  Y = H [W_self | W_neigh],  H' = act(Y_self + Abar Y_neigh + b).
// The two halves of the concatenation are padded to Fp = F_out rounded up to the
// 16-byte element count, so that a group of four never straddles the halves;
// positions c >= F_out inside a half read as zero.
// ---------------------------------------------------------------------------
template <int kMode>
struct SideWeights {  // B[k][n] = n < Fp ? W_self[k][n] : W_neigh[k][n-Fp]   (contiguous along n)
    static constexpr bool kContigK = false;
    static constexpr bool kGroups = kMode != kElementwise;
    static constexpr bool V = kMode == kAligned4;
    typedef typename std::conditional<kMode == kUnaligned4, RawU, RawV<float, V>>::type Raw;
    struct Lane {
        const float *col;  // element of row k is col[k * Fo]  (kUnaligned4: the matrix, and c = first column)
        int nv;            // valid elements from this column on (<= 0: padding)
        int c;
    };
    const float *Ws;
    const float *Wn;
    int F;   // rows (= F_in)
    int Fo;  // valid columns per half
    int Fp;  // padded columns per half
    static __device__ __forceinline__ float4 resolve(const Raw &r) { return r.get(); }
    __device__ __forceinline__ Lane prepare(int64_t n64) const
    {
        const int n = int(n64);
        const bool second = n >= Fp;
        const int c = n - (second ? Fp : 0);
        const bool ok = n < 2 * Fp && c < Fo;
        if constexpr (kMode == kUnaligned4) return Lane{second ? Wn : Ws, ok ? Fo - c : 0, ok ? c : 0};
        else return Lane{(second ? Wn : Ws) + (ok ? c : 0), ok ? Fo - c : 0, 0};
    }
    __device__ __forceinline__ Raw load(const Lane &l, int64_t k64) const
    {
        const int k = int(k64);
        if constexpr (kMode == kUnaligned4) {
            return load_unaligned4(l.col, (k < F ? k : 0) * Fo + l.c, F * Fo, (l.nv > 0 && k < F) ? l.nv : 0);
        } else {
            Raw r;
            r.ok = l.nv > 0 && k < F;
            const float *p = l.col + int64_t(k < F ? k : 0) * Fo;
            if constexpr (V) {
                r.v = *reinterpret_cast<const float4 *>(p);
            } else if (r.ok) {
                r.v.x = p[0];
                r.v.y = l.nv > 1 ? p[1] : 0.0f;
                r.v.z = l.nv > 2 ? p[2] : 0.0f;
                r.v.w = l.nv > 3 ? p[3] : 0.0f;
            } else {
                r.v = zero4();
            }
            return r;
        }
    }
    __device__ __forceinline__ Raw load_plain(const Lane &l, int64_t kt, int dk) const
    {
        if constexpr (V) {
            Raw r;
            r.ok = l.nv > 0;
            r.v = *reinterpret_cast<const float4 *>(l.col + kt * Fo + dk * Fo);
            return r;
        } else {
            return load(l, kt + dk);
        }
    }
};

template <int kMode>
struct SideWeightsT {  // B[k][n] = k < Fp ? W_self[n][k] : W_neigh[n][k-Fp]   (contiguous along k); n = input feature
    static constexpr bool kContigK = true;
    static constexpr bool kGroups = kMode != kElementwise;
    static constexpr bool V = kMode == kAligned4;
    typedef typename std::conditional<kMode == kUnaligned4, RawU, RawV<float, V>>::type Raw;
    struct Lane {
        const float *rs, *rn;  // rows such that element k is rs[k] (first half) or rn[k] (second half)
        int row;               // first element of the row inside its matrix
        bool ok;
    };
    const float *Ws;
    const float *Wn;
    int F;  // rows of W (= F_in) = extent of n
    int Fo;
    int Fp;
    static __device__ __forceinline__ float4 resolve(const Raw &r) { return r.get(); }
    __device__ __forceinline__ Lane prepare(int64_t n64) const
    {
        const int n = int(n64 < F ? n64 : 0);
        return Lane{Ws + int64_t(n) * Fo, Wn + int64_t(n) * Fo - Fp, n * Fo, n64 < F};
    }
    __device__ __forceinline__ Raw load(const Lane &l, int64_t k64) const
    {
        const int k = int(k64);
        const bool second = k >= Fp;
        const int c = k - (second ? Fp : 0);
        const bool ok = l.ok && k < 2 * Fp && c < Fo;
        if constexpr (kMode == kUnaligned4) {
            return load_unaligned4(second ? Wn : Ws, l.row + (ok ? c : 0), F * Fo, ok ? Fo - c : 0);
        } else {
            Raw r;
            r.ok = ok;
            const float *p = (second ? l.rn : l.rs) + (r.ok ? k : (second ? Fp : 0));
            if constexpr (V) {
                r.v = *reinterpret_cast<const float4 *>(p);
            } else if (r.ok) {
                r.v.x = p[0];
                r.v.y = c + 1 < Fo ? p[1] : 0.0f;
                r.v.z = c + 2 < Fo ? p[2] : 0.0f;
                r.v.w = c + 3 < Fo ? p[3] : 0.0f;
            } else {
                r.v = zero4();
            }
            return r;
        }
    }
    __device__ __forceinline__ Raw load_plain(const Lane &l, int64_t kt, int dk) const
    {
        if constexpr (V) {
            const int k = int(kt) + dk;
            const bool second = k >= Fp;
            Raw r;
            r.ok = l.ok && k - (second ? Fp : 0) < Fo;      // (Fo < Fp: padding inside the halves)
            r.v = *reinterpret_cast<const float4 *>((second ? l.rn : l.rs) + (r.ok ? k : second ? Fp : 0));
            return r;
        } else {
            return load(l, kt + dk);
        }
    }
};

// [dZ | dYn]: first half = dHnext (.) act'(Hnext) (leading dimension ld, Fo valid columns),
// second half = dYn (leading dimension ldy, Fp columns, padding already zero).
// kAsA: A[m=node][k] (contiguous along k); otherwise B[k=node][n] (contiguous along n).
template <bool kAsA, typename T, bool V, bool kRelu>
struct SideGrad {
    static constexpr bool kContigK = kAsA;
    static constexpr bool kMasks = true;
    static constexpr bool kGroups = V;
    static constexpr bool kTwoSources = true;
    typedef typename std::conditional<V, typename Pack4<T>::Packed, float4>::type Quad;
    struct Raw {
        Quad g, h;
        int nv;
        bool second;
    };
    struct Lane {
        int64_t a, b;  // kAsA: node*ld, node*ldy ; else: column inside its half, unused
        bool ok, second;
    };
    const T *dHn;
    const T *Hn;
    const T *dYn;
    int Fo, Fp;
    int64_t ld, ldy;
    int64_t rows;
    static __device__ __forceinline__ float4 quad(const Quad &q)
    {
        if constexpr (V) return Pack4<T>::widen(q);
        else return q;
    }
    static __device__ __forceinline__ float4 resolve(const Raw &r)
    {
        const float4 g = quad(r.g);
        bool o0 = r.nv > 0, o1 = r.nv > 1, o2 = r.nv > 2, o3 = r.nv > 3;
        if constexpr (kRelu) {
            const float4 h = quad(r.h);
            o0 = o0 && (r.second || h.x > 0.0f);
            o1 = o1 && (r.second || h.y > 0.0f);
            o2 = o2 && (r.second || h.z > 0.0f);
            o3 = o3 && (r.second || h.w > 0.0f);
        }
        return make_float4(o0 ? g.x : 0.0f, o1 ? g.y : 0.0f, o2 ? g.z : 0.0f, o3 ? g.w : 0.0f);
    }
    __device__ __forceinline__ Lane prepare(int64_t mn) const
    {
        if (kAsA) {
            const int64_t node = mn < rows ? mn : 0;
            return Lane{node * ld, node * ldy, mn < rows, false};
        }
        const bool second = mn >= Fp;
        const int64_t c = mn - (second ? Fp : 0);
        const bool ok = mn < 2 * Fp && (second || c < Fo);
        return Lane{ok ? c : 0, 0, ok, second};
    }
    __device__ __forceinline__ Raw load(const Lane &l, int64_t k) const
    {
        Raw r;
        bool second, inside;
        int c;
        int64_t eg, ey;
        if (kAsA) {
            second = k >= Fp;
            c = int(k - (second ? Fp : 0));
            inside = l.ok && k < 2 * Fp && (second || c < Fo);
            if (!inside) c = 0;
            eg = l.a + (c < Fo ? c : 0);       // (a half is padded to Fp, dZ's rows end at Fo)
            ey = l.b + c;
        } else {
            second = l.second;
            c = int(l.a);
            inside = l.ok && k < rows;
            const int64_t node = k < rows ? k : 0;
            eg = node * ld + (c < Fo ? c : 0);
            ey = node * ldy + c;
        }
        r.second = second;
        r.nv = inside ? (second ? Fp : Fo) - c : 0;
        if constexpr (V) {
            r.g = Pack4<T>::load(second ? dYn + ey : dHn + eg);
            if constexpr (kRelu) r.h = Pack4<T>::load(Hn + eg);
            else r.h = r.g;
        } else {
            r.g = zero4();
            r.h = zero4();
            if (inside) {
                const T *pg = second ? dYn + ey : dHn + eg;
                const int lim = r.nv;
                r.g.x = widen1(pg);
                if (lim > 1) r.g.y = widen1(pg + 1);
                if (lim > 2) r.g.z = widen1(pg + 2);
                if (lim > 3) r.g.w = widen1(pg + 3);
                if (kRelu && !second) {
                    const T *ph = Hn + eg;
                    r.h.x = widen1(ph);
                    if (lim > 1) r.h.y = widen1(ph + 1);
                    if (lim > 2) r.h.z = widen1(ph + 2);
                    if (lim > 3) r.h.w = widen1(ph + 3);
                }
            }
        }
        return r;
    }
    __device__ __forceinline__ Raw load_plain(const Lane &l, int64_t kt, int dk) const
    {
        if constexpr (V) {
            Raw r;
            int64_t eg, ey;
            if (kAsA) {   // k = position in [dZ | dYn]
                const int64_t k = kt + dk;
                r.second = k >= Fp;
                const int c = int(k - (r.second ? Fp : 0));
                r.nv = !l.ok ? 0 : r.second ? 4 : Fo - c;       // (Fo < Fp: padding at the end of dZ's half)
                eg = l.a + (c < Fo ? c : 0);
                ey = l.b + c;
            } else {      // k = node
                r.second = l.second;
                const int c = int(l.a);
                r.nv = l.ok ? (r.second ? Fp : Fo) - c : 0;
                eg = kt * ld + (dk * ld + (c < Fo ? c : 0));
                ey = kt * ldy + (dk * ldy + c);
            }
            r.g = Pack4<T>::load(r.second ? dYn + ey : dHn + eg);
            if constexpr (kRelu) r.h = Pack4<T>::load(Hn + eg);
            else r.h = r.g;
            return r;
        } else {
            return load(l, kt + dk);
        }
    }
};

// ---------------------------------------------------------------------------
// fp32 operands of backward products whose inner extent F is not a multiple of four.  Groups along a concatenation are padded to
// Fq = F rounded up to four, so that no group of four straddles the halves; the padding reads as zero in both operands.  Groups are
// fetched whole from 4-byte-aligned addresses: past the end of a row lies the next one, and in the last row the group is
// fetched `shift` elements earlier (RawU).  See rows_u_ok for the arrays this takes.
// ---------------------------------------------------------------------------
struct CatRowsTU {  // A[m][k] = (m < Fq ? H[k][m] : M[k][m-Fq])   (contiguous along m); k = node
    static constexpr bool kContigK = false;
    static constexpr bool kGroups = true;
    typedef RawU Raw;
    struct Lane {
        const float *p;   // column pointer: element of node k is p[k * ld]
        int64_t ld;
        int left;         // elements of the row from this column on (<= 0: padding)
    };
    const float *H;
    int64_t ldh;
    const float *Mx;
    int64_t ldm;
    int F, Fq;
    int64_t rows;
    static __device__ __forceinline__ float4 resolve(const Raw &r) { return r.get(); }
    __device__ __forceinline__ Lane prepare(int64_t m64) const
    {
        const int m = int(m64);
        const bool second = m >= Fq && m < 2 * Fq;
        const int c = m - (second ? Fq : 0);
        return Lane{(second ? Mx : H) + (c < F ? c : 0), second ? ldm : ldh, F - c};
    }
    __device__ __forceinline__ Raw load(const Lane &l, int64_t node) const
    {
        const bool ok = node < rows && l.left > 0;
        const int64_t at = node < rows ? node : 0;
        // (a padding lane fetches from column 0)
        return load_unaligned4_at(l.p + at * l.ld, at == rows - 1 ? (l.left > 0 ? l.left : F) : 4, ok ? l.left : 0);
    }
    __device__ __forceinline__ Raw load_plain(const Lane &l, int64_t kt, int dk) const { return load(l, kt + dk); }
};

struct CatWeightsTU {  // B[k][n] = n < F ? W_self[n][k] : W_neigh[n-F][k]  (contiguous along k); k = output feature
    static constexpr bool kContigK = true;
    static constexpr bool kGroups = true;
    typedef RawU Raw;
    struct Lane {
        const float *W;
        int row;      // first element of the row
        bool ok;
    };
    const float *Ws;
    const float *Wn;
    int F;
    int Fo;
    static __device__ __forceinline__ float4 resolve(const Raw &r) { return r.get(); }
    __device__ __forceinline__ Lane prepare(int64_t n64) const
    {
        const int n = int(n64);
        if (n < F) return Lane{Ws, n * Fo, true};
        return Lane{Wn, (n < 2 * F ? n - F : 0) * Fo, n < 2 * F};
    }
    __device__ __forceinline__ Raw load(const Lane &l, int64_t k64) const
    {
        const int k = int(k64);
        return load_unaligned4(l.W, l.row + (k < Fo ? k : 0), F * Fo, l.ok ? (k < Fo ? Fo - k : 0) : 0);
    }
    __device__ __forceinline__ Raw load_plain(const Lane &l, int64_t kt, int dk) const { return load(l, kt + dk); }
};

// ---------------------------------------------------------------------------
// Epilogues.  col_aux / row_aux are fetched once per tile column / row with a
// clamped (always valid) index; value() is pure arithmetic on registers.
// ---------------------------------------------------------------------------
// Two-byte results: an epilogue that can name the address of an element (at) and vouches that columns 2c and 2c + 1
// of a row are one aligned 4-byte word (pairs_ok) lets neighbouring lanes trade every other value, so that each
// lane stores two columns of one row in one instruction instead of one column of two rows in two.
template <class E, class = void>
struct StoresPairs : std::false_type {};
template <class E>
struct StoresPairs<E, std::void_t<decltype(&E::pairs_ok)>> : std::bool_constant<E::kPairs> {};

__device__ __forceinline__ bool word_aligned(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 3) == 0; }

template <class E>
__device__ __forceinline__ bool pairs_ok_of(const E &e)
{
    if constexpr (StoresPairs<E>::value) return e.pairs_ok();
    else return false;
}
template <class E>
__device__ __forceinline__ void store_pair(const E &e, int64_t row, int col, uint32_t word)
{
    if constexpr (StoresPairs<E>::value) *reinterpret_cast<uint32_t *>(e.at(row, col)) = word;
}

template <typename T>
struct FwdEpilogue {  // H' = act(acc + b)
    static constexpr bool kColAux = true, kRowAux = false;
    T *out;
    int64_t ld;
    const float *bias;
    bool relu;
    __device__ __forceinline__ float col_aux(int col) const { return bias[col]; }
    __device__ __forceinline__ const float *col_at(int col) const { return bias + col; }
    __device__ __forceinline__ const float *row_at(int64_t) const { return nullptr; }
    __device__ __forceinline__ bool padding(int) const { return false; }
    __device__ __forceinline__ float row_aux(int64_t) const { return 0.0f; }
    __device__ __forceinline__ float value(float v, float caux, float, int) const
    {
        v += caux;
        if (relu) v = v > 0.0f ? v : 0.0f;
        return v;
    }
    __device__ __forceinline__ void store(int64_t row, int col, float v, int) const { narrow1(out + row * ld + col, v); }
    static constexpr bool kPairs = sizeof(T) == 2;
    __device__ __forceinline__ bool pairs_ok() const { return ld % 2 == 0 && word_aligned(out); }
    __device__ __forceinline__ T *at(int64_t row, int col) const { return out + row * ld + col; }
};

template <typename T>
struct BwdDataEpilogue {  // columns [0,F): dH_self (leading dimension ldh) ; [F,2F): inv_deg[row] * dM (dense)
    static constexpr bool kColAux = false, kRowAux = true;
    T *dH;
    int64_t ldh;
    T *dMs;
    const float *inv_deg;
    int F;
    __device__ __forceinline__ float col_aux(int) const { return 0.0f; }
    __device__ __forceinline__ float row_aux(int64_t row) const { return inv_deg[row]; }
    __device__ __forceinline__ const float *col_at(int) const { return nullptr; }
    __device__ __forceinline__ const float *row_at(int64_t row) const { return inv_deg + row; }
    __device__ __forceinline__ bool padding(int) const { return false; }
    __device__ __forceinline__ float value(float v, float, float raux, int col) const { return col < F ? v : v * raux; }
    __device__ __forceinline__ void store(int64_t row, int col, float v, int) const
    {
        if (col < F) narrow1(dH + row * ldh + col, v);
        else narrow1(dMs + row * F + (col - F), v);
    }
    static constexpr bool kPairs = sizeof(T) == 2;
    __device__ __forceinline__ bool pairs_ok() const
    {
        return ldh % 2 == 0 && F % 2 == 0 && word_aligned(dH) && word_aligned(dMs);
    }
    __device__ __forceinline__ T *at(int64_t row, int col) const
    {
        return col < F ? dH + row * ldh + col : dMs + row * F + (col - F);
    }
};

template <typename T>
struct HalvesEpilogue {  // columns [0,Fp): Y_self ; [Fp,2Fp): Y_neigh ; both [rows, ldy], of which Fo are not padding
    static constexpr bool kColAux = false, kRowAux = false;
    T *Ys;
    T *Yn;
    int64_t ldy;
    int Fp, Fo;
    __device__ __forceinline__ bool padding(int col) const { return col - (col < Fp ? 0 : Fp) >= Fo; }
    __device__ __forceinline__ const float *col_at(int) const { return nullptr; }
    __device__ __forceinline__ const float *row_at(int64_t) const { return nullptr; }
    __device__ __forceinline__ float col_aux(int) const { return 0.0f; }
    __device__ __forceinline__ float row_aux(int64_t) const { return 0.0f; }
    __device__ __forceinline__ float value(float v, float, float, int) const { return v; }
    __device__ __forceinline__ void store(int64_t row, int col, float v, int) const
    {
        if (col < Fp) narrow1(Ys + row * ldy + col, v);
        else narrow1(Yn + row * ldy + (col - Fp), v);
    }
    static constexpr bool kPairs = sizeof(T) == 2;
    __device__ __forceinline__ bool pairs_ok() const
    {
        return ldy % 2 == 0 && Fp % 2 == 0 && word_aligned(Ys) && word_aligned(Yn);
    }
    __device__ __forceinline__ T *at(int64_t row, int col) const
    {
        return col < Fp ? Ys + row * ldy + col : Yn + row * ldy + (col - Fp);
    }
};

template <typename T>
struct RowsEpilogue {  // plain [rows, ld] output
    static constexpr bool kColAux = false, kRowAux = false;
    T *out;
    int64_t ld;
    __device__ __forceinline__ const float *col_at(int) const { return nullptr; }
    __device__ __forceinline__ const float *row_at(int64_t) const { return nullptr; }
    __device__ __forceinline__ bool padding(int) const { return false; }
    __device__ __forceinline__ float col_aux(int) const { return 0.0f; }
    __device__ __forceinline__ float row_aux(int64_t) const { return 0.0f; }
    __device__ __forceinline__ float value(float v, float, float, int) const { return v; }
    __device__ __forceinline__ void store(int64_t row, int col, float v, int) const { narrow1(out + row * ld + col, v); }
    static constexpr bool kPairs = sizeof(T) == 2;
    __device__ __forceinline__ bool pairs_ok() const { return ld % 2 == 0 && word_aligned(out); }
    __device__ __forceinline__ T *at(int64_t row, int col) const { return out + row * ld + col; }
};

struct SplitEpilogue {  // partial products, one slab per split
    static constexpr bool kColAux = false, kRowAux = false;
    float *partial;
    int64_t Mtot;
    int N;
    __device__ __forceinline__ float col_aux(int) const { return 0.0f; }
    __device__ __forceinline__ float row_aux(int64_t) const { return 0.0f; }
    __device__ __forceinline__ float value(float v, float, float, int) const { return v; }
    __device__ __forceinline__ void store(int64_t row, int col, float v, int split) const
    {
        partial[(int64_t(split) * Mtot + row) * N + col] = v;
    }
};

struct SplitEpiloguePad {  // the same from [H | M] with halves padded to Fq columns, which are left out
    static constexpr bool kColAux = false, kRowAux = false;
    float *partial;
    int F, Fq;
    int N;
    __device__ __forceinline__ float col_aux(int) const { return 0.0f; }
    __device__ __forceinline__ float row_aux(int64_t) const { return 0.0f; }
    __device__ __forceinline__ float value(float v, float, float, int) const { return v; }
    __device__ __forceinline__ void store(int64_t row, int col, float v, int split) const
    {
        const bool second = row >= Fq;
        const int64_t c = row - (second ? Fq : 0);
        if (c < F) partial[(int64_t(split) * 2 * F + c + (second ? F : 0)) * N + col] = v;
    }
};

// ---------------------------------------------------------------------------
// bf16 fragments.  A group of 16 k-values is ONE v_mfma_f32_32x32x16_bf16 (the instruction this chip adds; the
// 32x32x8 one runs at half its rate): lane l holds row l%32 and the eight k-values 8*(l/32) .. +7.  Activations
// stored in bf16 pass through LDS unchanged, fp32 weights are rounded to nearest even on their way in.
// ---------------------------------------------------------------------------
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// A lane's values of two rows R and R + 1 of its column -> neighbouring columns of one row: an even lane gets (column, column + 1) of row R,
// an odd one (column - 1, column) of row R + 1.  `select`: traded_bytes(lane).
__device__ __forceinline__ uint32_t traded_bytes(int lane) { return lane & 1 ? 0x03020706u : 0x05040100u; }
__device__ __forceinline__ uint32_t traded_pair(float v0, float v1, uint32_t select)
{
    const uint32_t own = pack_bf16(v0, v1);
    const uint32_t other = __builtin_amdgcn_mov_dpp(own, 0xB1, 0xF, 0xF, true);   // quad_perm [1, 0, 3, 2]: the neighbouring lane's
    return __builtin_amdgcn_perm(other, own, select);
}

constexpr int kGroupK = 16;
__device__ __forceinline__ void put_bf16(uint16_t *dst, const float4 &v)
{
    *reinterpret_cast<uint2 *>(dst) = make_uint2(pack_bf16(v.x, v.y), pack_bf16(v.z, v.w));
}
__device__ __forceinline__ bf16x8 fragment_along(const uint16_t *p)   // (tile rows are 8-byte aligned, not 16)
{
    const uint2 lo = *reinterpret_cast<const uint2 *>(p), hi = *reinterpret_cast<const uint2 *>(p + 4);
    return __builtin_bit_cast(bf16x8, make_uint4(lo.x, lo.y, hi.x, hi.y));
}
__device__ __forceinline__ bf16x8 fragment_strided(const uint16_t *p, int ld)
{
    uint4 w;
    w.x = uint32_t(p[0]) | (uint32_t(p[ld]) << 16);
    w.y = uint32_t(p[2 * ld]) | (uint32_t(p[3 * ld]) << 16);
    w.z = uint32_t(p[4 * ld]) | (uint32_t(p[5 * ld]) << 16);
    w.w = uint32_t(p[6 * ld]) | (uint32_t(p[7 * ld]) << 16);
    return __builtin_bit_cast(bf16x8, w);
}

// ---------------------------------------------------------------------------
// C[M,N] = A[M,K] B[K,N], k split into ranges of k_per_split, bf16 MFMA.
// Work item = (split, m-tile, n-tile), numbered split-major then m then n.
// Persistent blocks: the grid is 8 x (blocks per die); the block with id b sits
// on die b % 8 and walks the work items  die*per_die + b/8, + blocks_per_die, ...
// so that at any time the blocks of a die work on neighbouring items (the n-tiles
// of one row block, the output tiles of one node range) and share them in its L2.
// The first slab of a block's next tile is fetched before the results of the
// current one are written out, so that its latency passes behind the stores.
// Whole slabs are fetched with unguarded loads (addresses affine in k: one
// addition per load and slab instead of clamps and 64-bit multiplications) where
// the operands' views have them; a tile that lies wholly
// inside the result is written out without per-element bounds tests, which also
// gives the compiler a fixed number of stores to count its waits against.
// ---------------------------------------------------------------------------
template <int BM, int BN, int BK, int WM, int WN, bool kColSum, class AL, class BL, class Epi>
__global__ __launch_bounds__(WM *WN * 64, 2) void gemm_bf16_kernel(AL a, BL b, Epi epi, int64_t M, int N, int64_t K,
                                                                 int64_t k_per_split, int n_tiles,
                                                                 int64_t tiles_per_split, int64_t total_work,
                                                                 float *__restrict__ colsum_partial)
{
    constexpr int NT = WM * WN * 64;
    constexpr int kDepth = DeepPrefetch<kColSum, Epi::kRowAux>::value ? 2 : 1;   // slabs in flight in registers
    // 8 accumulator tiles, or the two sources of [dZ | dYn], leave registers for one, and not across the barrier
    constexpr bool kLean = (BM / WM / 32) * (BN / WN / 32) > 4 || TwoSourcesAlongK<AL>::value;
    constexpr bool kSteady = !kLean && SteadyLoop<BN, AL, BL>::value;
    constexpr int TM = BM / WM / 32;
    constexpr int TN = BN / WN / 32;
    constexpr int A_Q = BM * BK / 4, B_Q = BN * BK / 4;   // pieces (four values) of a slab
    constexpr int A_V = (A_Q + NT - 1) / NT;              // load slots per thread; when the pieces do not divide
    constexpr int B_V = (B_Q + NT - 1) / NT;              // evenly the last slots repeat the last piece (same value)
    typedef bf16x8 Frag;
    constexpr int GK = kGroupK;
    constexpr int KG = BK / GK;
    constexpr int A_LD = AL::kContigK ? BK + kPad : BM + kPad;
    constexpr int B_LD = BL::kContigK ? BK + kPad : BN + kPad;
    constexpr int A_WORDS = AL::kContigK ? BM * A_LD : BK * A_LD;
    constexpr int B_WORDS = BL::kContigK ? BN * B_LD : BK * B_LD;
    static_assert(BM % (WM * 32) == 0 && BN % (WN * 32) == 0 && BK % GK == 0, "tile shape");
    static_assert(!kColSum || !BL::kContigK, "column sums are taken from a [k][n] tile");
    static_assert(A_WORDS * sizeof(uint16_t) >= BN * sizeof(float) && B_WORDS * sizeof(uint16_t) >= BM * sizeof(float),
                  "epilogue staging fits");

    __shared__ __attribute__((aligned(16))) uint16_t As[2][A_WORDS];
    __shared__ __attribute__((aligned(16))) uint16_t Bs[2][B_WORDS];
    float *const a_aux = reinterpret_cast<float *>(&As[0][0]);   // per-column / per-row epilogue inputs
    float *const b_aux = reinterpret_cast<float *>(&Bs[0][0]);

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

    typename AL::Lane alane[A_V];
    typename BL::Lane blane[B_V];
    // first slab of the tile that comes next; the slabs inside a tile's main loop have registers of their own
    typename AL::Raw afirst[A_V];
    typename BL::Raw bfirst[B_V];
    auto prepare = [&](const Tile &t) {
#pragma unroll
        for (int i = 0; i < A_V; ++i) alane[i] = a.prepare(t.m0 + a_mn[i]);
#pragma unroll
        for (int i = 0; i < B_V; ++i) blane[i] = b.prepare(t.n0 + b_mn[i]);
    };
    // guarded: any position, clamped and flagged; plain: the caller knows the whole slab lies inside the
    // operands' k range, so the addresses are affine in k and cost one addition per slab
    auto fetch = [&](int64_t kt, typename AL::Raw(&ar)[A_V], typename BL::Raw(&br)[B_V]) {
#pragma unroll
        for (int i = 0; i < A_V; ++i) ar[i] = a.load(alane[i], kt + a_k[i]);
#pragma unroll
        for (int i = 0; i < B_V; ++i) br[i] = b.load(blane[i], kt + b_k[i]);
    };
    auto fetch_plain = [&](int64_t kt, typename AL::Raw(&ar)[A_V], typename BL::Raw(&br)[B_V]) {
#pragma unroll
        for (int i = 0; i < A_V; ++i) ar[i] = a.load_plain(alane[i], kt, a_k[i]);
#pragma unroll
        for (int i = 0; i < B_V; ++i) br[i] = b.load_plain(blane[i], kt, b_k[i]);
    };
    auto stage = [&](int buf, const typename AL::Raw(&ar)[A_V], const typename BL::Raw(&br)[B_V]) {
#pragma unroll
        for (int i = 0; i < A_V; ++i) {
            if constexpr (PacksBf16<AL>::value) *reinterpret_cast<uint2 *>(&As[buf][a_lds[i]]) = AL::packed(ar[i]);
            else put_bf16(&As[buf][a_lds[i]], AL::resolve(ar[i]));
        }
#pragma unroll
        for (int i = 0; i < B_V; ++i) {
            if constexpr (PacksBf16<BL>::value) *reinterpret_cast<uint2 *>(&Bs[buf][b_lds[i]]) = BL::packed(br[i]);
            else put_bf16(&Bs[buf][b_lds[i]], BL::resolve(br[i]));
        }
    };
    // This lane's k-values of group g (the upper half of the wavefront holds the upper half of the group) of its
    // row/column.
    auto frag_a = [&](int buf, int g, int i) -> Frag {
        const int mn = wm0 + i * 32 + l31;
        const int k = g * GK + (GK / 2) * hi;
        if (AL::kContigK) return fragment_along(&As[buf][mn * A_LD + k]);
        return fragment_strided(&As[buf][k * A_LD + mn], A_LD);
    };
    auto frag_b = [&](int buf, int g, int j) -> Frag {
        const int mn = wn0 + j * 32 + l31;
        const int k = g * GK + (GK / 2) * hi;
        if (BL::kContigK) return fragment_along(&Bs[buf][mn * B_LD + k]);
        return fragment_strided(&Bs[buf][k * B_LD + mn], B_LD);
    };

    int64_t work = die * per_die + blockIdx.x / kXcds;
    if (work >= die_end) return;
    Tile t = tile_of(work);
    prepare(t);
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
            Frag fa[2][TM], fb[2][TN];
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
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[cur][i], fb[cur][j], acc[i][j], 0, 0, 0);
            }
            if (kColSum && t.m0 == 0 && tid < BN) {
#pragma unroll
                for (int k = 0; k < BK; ++k) colsum += bf16_to_f32(Bs[buf][k * B_LD + tid]);
            }
        };
        int buf = 0;     // holds the slab that comes next
        auto one_loop = [&](auto plain_tag) {      // few registers: nothing but the next slab's loads, one multiply in the code
            typename AL::Raw areg[A_V];
            typename BL::Raw breg[B_V];
            for (int64_t kt = t.k_begin; kt < t.k_end; kt += BK) {
                const bool more = kt + BK < t.k_end;
                if (more) {  // in flight while this slab is multiplied
                    if constexpr (decltype(plain_tag)::value) fetch_plain(kt + BK, areg, breg);
                    else fetch(kt + BK, areg, breg);
                }
                multiply(buf);
                if (more) stage(buf ^ 1, areg, breg);  // the other buffer was last read before the previous barrier
                __syncthreads();
                buf ^= 1;
            }
        };
        // two slabs in flight in registers (slab s >= 1 waits in set (s - 1) % kDepth), whole slabs only
        auto two_loop = [&]() {
            typename AL::Raw areg[kDepth][A_V];
            typename BL::Raw breg[kDepth][B_V];
            const int64_t n_slabs = (t.k_end - t.k_begin) / BK;
            static_for<kDepth>([&](auto d_tag) {
                constexpr int D = decltype(d_tag)::value;
                if (n_slabs > D + 1) fetch_plain(t.k_begin + (D + 1) * BK, areg[D], breg[D]);
            });
            for (int64_t sl0 = 0; sl0 < n_slabs; sl0 += kDepth)
                static_for<kDepth>([&](auto r_tag) {
                    constexpr int R = decltype(r_tag)::value;
                    const int64_t sl = sl0 + R;
                    if (sl < n_slabs) {      // the same for every thread
                        multiply(buf);
                        if (sl + 1 < n_slabs) stage(buf ^ 1, areg[R], breg[R]);
                        if (sl + 1 + kDepth < n_slabs) fetch_plain(t.k_begin + (sl + 1 + kDepth) * BK, areg[R], breg[R]);
                        __syncthreads();
                        buf ^= 1;
                    }
                });
        };
        if constexpr (!kSteady) {
            // guarded loads: (two sources) they need no more registers than the others and fewer in all, 41 us against 50;
            // (element by element, unaligned groups) they are the only ones; (rows of no multiple of four) no range of theirs is whole slabs
            if constexpr (TwoSourcesAlongK<AL>::value || !AL::kGroups || !BL::kGroups || UnalignedGroups<BL>::value ||
                          std::is_same<AL, PaddedRows>::value)
                one_loop(std::false_type{});
            else if ((t.k_end - t.k_begin) % BK != 0) one_loop(std::false_type{});
            else if constexpr (kLean || kDepth == 1) one_loop(std::true_type{});
            else two_loop();
        } else {
            // Whole slabs, in a body without branches, so that the waits ahead of a slab's staging count the younger slabs'
            // loads exactly and leave them in flight (a conditional fetch had made every wait drain them: forward 2 x 256 ->
            // 256 at 2,000,000 rows 1,228 -> 1,114 us, its input gradient 1,950 -> 1,801 us).
            const int64_t n_whole = (t.k_end - t.k_begin) / BK;
            const bool tail = t.k_begin + n_whole * BK < t.k_end;
            auto slab = [&](int64_t s) { return t.k_begin + s * BK; };
            if (n_whole > 1) {
                // Slab s >= 1 waits in register set (s - 1) % kDepth; its loads are issued kDepth iterations before it is
                // staged.  The last steps, with nothing or less to fetch, come after the loop.
                typename AL::Raw areg[kDepth][A_V];
                typename BL::Raw breg[kDepth][B_V];
                static_for<kDepth>([&](auto d_tag) {
                    constexpr int D = decltype(d_tag)::value;
                    if (D + 1 < n_whole) fetch_plain(slab(D + 1), areg[D], breg[D]);
                });
                int64_t s = 0;
                for (; s + 2 + kDepth < n_whole; s += 2)
                    static_for<2>([&](auto r_tag) {
                        constexpr int R = decltype(r_tag)::value;
                        multiply(R);
                        stage(1 - R, areg[R % kDepth], breg[R % kDepth]);   // (last read before the previous barrier)
                        fetch_plain(slab(s + R + 1 + kDepth), areg[R % kDepth], breg[R % kDepth]);
                        __syncthreads();
                    });
                static_for<kDepth + 1>([&](auto r_tag) {
                    constexpr int R = decltype(r_tag)::value;
                    if (s + R + 1 < n_whole) {
                        multiply(R % 2);
                        stage(1 - R % 2, areg[R % kDepth], breg[R % kDepth]);
                        if (s + R + 1 + kDepth < n_whole) fetch_plain(slab(s + R + 1 + kDepth), areg[R % kDepth], breg[R % kDepth]);
                        __syncthreads();
                    }
                });
                buf = int((n_whole - 1) % 2);
            }
            if (n_whole > 0 && tail) {      // the last slab reaches past the end of k
                fetch(t.k_begin + n_whole * BK, afirst, bfirst);
                multiply(buf);
                buf ^= 1;
                stage(buf, afirst, bfirst);
                __syncthreads();
            }
            multiply(buf);
            __syncthreads();
        }

        // Per-column / per-row epilogue inputs (bias, 1/deg) go through LDS: they are loaded from
        // global memory once, here, before any store is in flight.  Fetched into registers directly they
        // would make the compiler guard every store below with a wait on the memory counter, which
        // also waits for the earlier stores and serialises the whole write-out.
        if (Epi::kColAux && tid < BN) a_aux[tid] = epi.col_aux(t.n0 + tid < N ? t.n0 + tid : N - 1);
        if (Epi::kRowAux && tid < BM) b_aux[tid] = epi.row_aux(t.m0 + tid < M ? t.m0 + tid : M - 1);
        if (Epi::kColAux || Epi::kRowAux) __syncthreads();

        // The first slab of this block's next tile is fetched now, so that its latency passes while the
        // results below are written out.
        const Tile done = t;
        const float done_colsum = colsum;
        const int64_t next = work + blocks_per_die;
        const bool has_next = next < die_end;
        if (has_next) {
            t = tile_of(next);
            prepare(t);
            fetch(t.k_begin, afirst, bfirst);
        }

        // MFMA 32x32 result layout: register r of lane l holds row 8*(r/4) + 4*(l/32) + r%4, column l%32.
        float caux[TN];
#pragma unroll
        for (int j = 0; j < TN; ++j) caux[j] = Epi::kColAux ? a_aux[wn0 + j * 32 + l31] : 0.0f;
        auto write_out = [&](auto inside_tag) {
            constexpr bool kInside = decltype(inside_tag)::value;   // the whole tile lies inside the result
            bool pairs = false;
            if constexpr (kInside && StoresPairs<Epi>::value) pairs = pairs_ok_of(epi);   // the same for every lane
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                float raux[16];
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    raux[r] = Epi::kRowAux ? b_aux[wm0 + i * 32 + 8 * (r / 4) + 4 * hi + (r % 4)] : 0.0f;
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    const int col = done.n0 + wn0 + j * 32 + l31;
                    if constexpr (kInside && StoresPairs<Epi>::value) {
                        if (pairs) {
                            // registers r and r + 1 are rows R and R + 1 of this lane's column
                            const int odd = l31 & 1;
                            const uint32_t select = traded_bytes(l31);
#pragma unroll
                            for (int r = 0; r < 16; r += 2) {
                                const int64_t row = done.m0 + wm0 + i * 32 + 8 * (r / 4) + 4 * hi + (r % 4);
                                const float v0 = epi.value(acc[i][j][r], caux[j], raux[r], col);
                                const float v1 = epi.value(acc[i][j][r + 1], caux[j], raux[r + 1], col);
                                store_pair(epi, row + odd, col - odd, traded_pair(v0, v1, select));
                            }
                            continue;
                        }
                    }
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
#include "gemm_f32.hpp"
#include "gemm_f32_async.hpp"
#include "gemm_split.hpp"
namespace tma {

template <typename T>
static bool vec4_ok(const T *p, int64_t ld) { return aligned(p, 4 * sizeof(T)) && ld % 4 == 0; }
// groups of four inside rows of F elements may be fetched whole: fp32 needs no alignment for it
template <typename T>
static bool groups_ok(const T *p, int64_t ld, int F)
{
    return F % 4 == 0 && (sizeof(T) == 4 || vec4_ok(p, ld));
}
// the same for a gradient or activation whose rows may have padding after F elements (then read, and discarded)
template <typename T>
static bool padded_groups_ok(const T *p, int64_t ld, int F) { return vec4_ok(p, ld) || groups_ok(p, ld, F); }
// what the views of RawU need: four elements at least, a group that starts in one row ends in the next at the latest
// (one row has none), and element numbers of weights in 32 bits
static inline bool rows_u_ok(int64_t n, int64_t ld, int F) { return (n - 1) * ld + F >= 4 && (n == 1 || ld >= 3); }
static inline bool weights_u_ok(int64_t F_in, int64_t F_out) { return F_in * F_out >= 4 && F_in * F_out <= INT32_MAX; }
static inline int pad4(int F) { return (F + 3) / 4 * 4; }

// BK: k-values per slab of the bf16 kernel (gemm_split_kernel, CT = float, has its own).
template <int BM, int BN, int BK, int WM, int WN, bool kColSum, typename CT = float, int kBlocks = 0, class AL, class BL, class Epi>
static void launch_gemm(const char *name, const AL &a, const BL &b, const Epi &e, int64_t M, int N, int64_t K,
                        int64_t k_per_split, int n_splits, float *colsum_partial, hipStream_t s)
{
    if (M <= 0 || N <= 0 || K <= 0) return;   // an empty product: callers zero-fill what they need
    const int n_tiles = int(ceil_div(N, BN));
    const int64_t tiles = ceil_div(M, BM) * n_tiles;
    const int64_t total = tiles * n_splits;
    // resident blocks per compute unit follow from the kernel's LDS footprint (160 KB per unit) and its
    // register budget (launch bounds: two waves per SIMD); 256 units in 8 dies
    constexpr int kLdsBytes = 2 * 2 * ((AL::kContigK ? BM * (BK + kPad) : BK * (BM + kPad)) + (BL::kContigK ? BN * (BK + kPad) : BK * (BN + kPad)));
    constexpr int kByWaves = 2 * 4 / (WM * WN) > 0 ? 2 * 4 / (WM * WN) : 1;
    constexpr int kByLds = 160 * 1024 / kLdsBytes > 0 ? 160 * 1024 / kLdsBytes : 1;
    constexpr int kPerCu = kBlocks ? kBlocks : sizeof(CT) == 4 ? kSplitPerCu * 4 / (WM * WN) : kByWaves < kByLds ? kByWaves : kByLds;
    int64_t blocks_per_die = ceil_div(total, kXcds);
    if (blocks_per_die > 32 * kPerCu) blocks_per_die = 32 * kPerCu;
    const dim3 grid(unsigned(blocks_per_die * kXcds)), block(WM * WN * 64);
    TMA_TIMED(name, s);
    if constexpr (sizeof(CT) == 4)
        hipLaunchKernelGGL((gemm_split_kernel<BM, BN, WM, WN, kColSum, AL, BL, Epi>), grid, block, 0, s, a, b, e, M, N, K,
                           k_per_split, n_tiles, tiles, total, colsum_partial);
    else
        hipLaunchKernelGGL((gemm_bf16_kernel<BM, BN, BK, WM, WN, kColSum, AL, BL, Epi>), grid, block, 0, s, a, b, e, M, N, K,
                           k_per_split, n_tiles, tiles, total, colsum_partial);
}

// Kernel names for the timing hook: <what>_<tile>[_bf16][_generic]; "generic" = a streaming operand is
// on the element-wise path (the name does not say how the weights are read: aligned groups, unaligned groups
// or element by element, which costs a transform-first product about a tenth of its time).
template <typename T>
static const char *kname(const char *f32_vec, const char *f32_gen, const char *bf16_vec, const char *bf16_gen, bool vec)
{
    if (sizeof(T) == 4) return vec ? f32_vec : f32_gen;
    return vec ? bf16_vec : bf16_gen;
}

// A product with few 128x128 output tiles (a sampled block, a small part) would leave compute units without a
// workgroup or with a single one: below this many tiles (256 compute units) the narrower tile is taken, for twice
// as many workgroups.
#ifndef TMA_GEMM_FEW_TILES
#define TMA_GEMM_FEW_TILES 384
#endif
constexpr int64_t kFewTiles = TMA_GEMM_FEW_TILES;
static inline bool few_tiles(int64_t M, int64_t N, int n_splits = 1)
{
    return ceil_div(M, int64_t(128)) * ceil_div(N, int64_t(128)) * n_splits < kFewTiles;
}

// A bf16 product of few rows (see few_rows) in tiles of 64 x 64, three blocks to a compute unit: where the fullest unit then has less to do, by
// `price` hundredths more a value, than with tiles of `rows` x `width`.  Forward products of layers that aggregate first (price 120); forward
// products, input and weight gradients of dense layers, and forward products and weight gradients of layers that transform first (110).
// Geometric mean of 72 products each of 1,700 to 60,000 rows, 64 to 256 columns in and 48 to 256 out: forward 0.89 of the time, input gradients of
// dense layers 0.88 and weight gradients of those two 0.93.  us at 5,000 rows, 2 x 256 -> 64 forward 9.5 -> 7.2, dense input gradient of 128 from 256 9.8 -> 7.1; at
// 40,004, 2 x 64 -> 48 forward 7.6 -> 6.4, dense input gradient of 64 from 256 14.5 -> 11.7; as before: 40,004 rows, 2 x 256 -> 256 forward
// 31 (64 x 64: 34).  Five blocks to a unit or k in slabs of 64 gain nothing on three.
// The other backward products, whose tiles are chosen in their own places, were not measured so: input and weight gradients of layers that aggregate
// first and input gradients of those that transform first have tiles of 128 rows at any number of them.
static inline bool few_rows_narrow(int64_t of_rows, int64_t M, int N, int n_splits, int rows, int width, int price)
{
    const auto fullest = [&](int r, int w) { return ceil_div(ceil_div(M, int64_t(r)) * ceil_div(N, w) * n_splits, int64_t(256)) * r * w; };
    return few_rows(of_rows) && fullest(64, 64) * price < fullest(rows, width) * 100;
}

// A product of fp32 storage on the fp32 instruction (gemm_f32.hpp), up to kPerCu blocks to a compute unit.
template <int BM, int BN, int BK, int WM, int WN, int kPerCu, bool kColSum, class AL, class BL, class Epi>
static void launch_f32(const char *name, const AL &a, const BL &b, const Epi &e, int64_t M, int N, int64_t K, int64_t k_per_split,
                       int n_splits, float *colsum_partial, hipStream_t s)
{
    if (M <= 0 || N <= 0 || K <= 0) return;   // an empty product: callers zero-fill what they need
    const int n_tiles = int(ceil_div(N, BN));
    const int64_t tiles = ceil_div(M, BM) * n_tiles;
    const int64_t total = tiles * n_splits;
    constexpr int kLdsBytes = 2 * 4 * ((AL::kContigK ? BM * (BK + kPad) : BK * (BM + kPad)) + (BL::kContigK ? BN * (BK + kPad) : BK * (BN + kPad)));
    static_assert(kPerCu * kLdsBytes <= 160 * 1024, "blocks per compute unit");
    int64_t blocks_per_die = ceil_div(total, kXcds);
    if (blocks_per_die > 32 * kPerCu) blocks_per_die = 32 * kPerCu;
    TMA_TIMED(name, s);
    hipLaunchKernelGGL((gemm_f32_kernel<BM, BN, BK, WM, WN, kColSum, AL, BL, Epi>), dim3(unsigned(blocks_per_die * kXcds)),
                       dim3(WM * WN * 64), 0, s, a, b, e, M, N, K, k_per_split, n_tiles, tiles, total, colsum_partial);
}

// A forward product of fp32 storage (gemm_f32_async.hpp).  The tile: the one that gives the fullest of 256 compute units least to do, a value
// of it, padding included, priced at what that tile takes for one where units have many, and at up to two fifths more where
// they have one at most, whose waits nothing then covers.  (The shorter k, the more of the time is writing, whose rate
// is the chip's and not a unit's: below 96 the mean over the units counts in proportion.)  Prices from 400,000 x 256 (us per
// column: 64 wide 1.86, 96 1.66, 128 1.67, 160 1.61).  1,560 products of 1,700 to 400,000 rows, 41 to 300 columns and
// k of 32 to 512 take 0.979 of what they take by padding and a count of tiles alone, 99 in 100 at most 1.05 of it, the best
// tile for each 0.971.  us, by padding -> so:
//   40,004 rows, k 256, 150 columns 51.0 (128 x 160, 313 tiles) -> 39.8 (128 x 64);  k 180, 200 columns 48.0 (128 x 128, 626) -> 40.5 (64 x 128)
//   70,000 rows, k 256, 100 columns 53.4 (128 x 128, 547 tiles) -> 45.2 (64 x 64);  125,237 rows, k 256, 256 columns: 128 x 128 as before
// 64 x 64 of 5,000 rows, 256 -> 256 and 128: 13.2 and 9.5, 64 x 128 14.0 and 13.5, 128 wide 22.0 and 21.7.
template <class BL, class Epi>
static void launch_fwd_f32(const char *name, const AsyncRows &a, const BL &b, const Epi &e, int64_t M, int N, hipStream_t s)
{
    if (M <= 0 || N <= 0 || a.K <= 0) return;
    if (N <= 32) return launch_async<64, 32, 2, 1, 3, 4>(name, a, b, e, M, N, s);   // 64 -> 32, 125,237 rows: 15.2 -> 12.6 us
    struct Tile { int rows, width, price, alone; };   // per cent
    constexpr Tile tiles[] = {{64, 64, 110, 110}, {64, 128, 105, 125}, {128, 64, 105, 125}, {128, 96, 100, 130}, {128, 128, 100, 140}, {128, 160, 97, 137}};
    constexpr int64_t kLongK = 96;
    const int64_t k = a.K < kLongK ? a.K : kLongK;
    int best = 0;
    int64_t least = 0;
    for (int i = 0; i < 6; ++i) {
        const Tile &t = tiles[i];
        const int64_t items = ceil_div(M, int64_t(t.rows)) * ceil_div(N, t.width);
        const int64_t load = items <= 256 ? 256 * kLongK : ceil_div(items, int64_t(256)) * 256 * k + items * (kLongK - k);
        const int64_t cost = load * t.rows * t.width * (items <= 256 ? t.alone : t.price);
        if (i == 0 || cost < least) best = i, least = cost;
    }
    switch (best) {
    case 0: return launch_async<64, 64, 2, 2, 3, 5>(name, a, b, e, M, N, s);
    case 1: return launch_async<64, 128, 2, 2, 3, 4>(name, a, b, e, M, N, s);
    case 2: return launch_async<128, 64, 4, 1, 3, 4>(name, a, b, e, M, N, s);
    case 3: return launch_async<128, 96, 4, 1, 3, 3>(name, a, b, e, M, N, s);
    case 4: return launch_async<128, 128, 2, 2, 3, 3>(name, a, b, e, M, N, s);
    default: return launch_async<128, 160, 4, 1, 3, 2>(name, a, b, e, M, N, s);
    }
}

// fp32 products with more than 96 columns.  The 256-wide tile of eight wavefronts reads the operand it is wide across
// once instead of twice and converts a quarter fewer values per product; it is taken where it pads no more than two
// tiles of 128 would, across the columns for a product whose rows are nodes and across the rows for a weight gradient.
// Measured, 128 x 128 -> 256-wide, n = 125,237 / 1,000,000, 2 x 128 -> 256: input gradient 166 -> 142 / 1,210 -> 1,031 us,
// weight gradient 125 -> 117 / 901 -> 840 us.
template <bool kColSum, class AL, class BL, class Epi>
static void launch_split_128(const char *name, const AL &a, const BL &b, const Epi &e, int64_t M, int N, int64_t K,
                             int64_t kps, int n_splits, float *colsum, hipStream_t s)
{
    if constexpr (kColSum) {
        if (ceil_div(M, int64_t(128)) % 2 == 0)
            return launch_gemm<256, 128, 32, 4, 2, true, float>(name, a, b, e, M, N, K, kps, n_splits, colsum, s);
    } else {
        if (ceil_div(N, 128) % 2 == 0)
            return launch_gemm<128, 256, 32, 2, 4, false, float>(name, a, b, e, M, N, K, kps, n_splits, colsum, s);
    }
    launch_gemm<128, 128, 32, 2, 2, kColSum, float>(name, a, b, e, M, N, K, kps, n_splits, colsum, s);
}

// A backward product of few rows (see few_rows).  us, from bf16 parts -> so, weight gradient of 128 -> 128 and input gradient of
// 2 x 128 -> 256: 5,000 rows 14 -> 14 and 16 -> 18, 60,000 rows 34 -> 47 and 60 -> 86.
//
// Its loads, LDS passes and instructions take turns inside a block, so what counts is how many blocks a unit has to
// choose from, and how evenly the units are loaded.  Tiles of 64 x 64, five blocks to a unit (k in slabs of 16; of 32, half
// the barriers, where each unit has one tile at most): by what the fullest unit has to do they go before wider tiles, which
// read less, unless they cost it a tenth more; a unit with a single tile of 128 rows idles through every barrier.
// us, by width as before (128 x 64 below 384 tiles, 128 x 96, 128 x 128, two blocks to a unit) -> 64 x 64:
//   weight gradients with ReLU, 5,000 rows 2 x 100 -> 150 14.5 -> 12.9; 40,004 rows 2 x 90 -> 150 62 -> 43, 2 x 160 -> 150 79 -> 56;
//   input gradients, 14,600 rows 150 from 150 20.5 -> 16.8; 40,004 rows 150 from 100 41 -> 27, 64 from 48 10.4 -> 8.0;
//   where 128 x 128 stays: 40,004 rows 512 from 256 104 (64 x 64: 118), weight gradient 2 x 128 -> 256 56 (60)
template <bool kColSum, class AL, class BL, class Epi>
static void launch_few_rows(const char *name, const AL &a, const BL &b, const Epi &e, int64_t M, int N, int64_t K, int64_t kps,
                            int n_splits, float *colsum, hipStream_t s)
{
    const auto items = [&](int rows, int width) { return ceil_div(M, int64_t(rows)) * ceil_div(N, width) * n_splits; };
    const auto fullest = [&](int rows, int width) { return ceil_div(items(rows, width), int64_t(256)) * rows * width; };
    const int64_t narrow = fullest(64, 64) * 11;
    if (items(64, 64) <= 256)
        launch_f32<64, 64, 32, 2, 2, 2, kColSum>(name, a, b, e, M, N, K, kps, n_splits, colsum, s);
    else if (N > 64 && N <= 96 && items(128, 96) > 256 && fullest(128, 96) * 10 < narrow)
        launch_f32<128, 96, 32, 4, 1, 2, kColSum>(name, a, b, e, M, N, K, kps, n_splits, colsum, s);
    else if (N > 96 && items(128, 128) > 256 && fullest(128, 128) * 10 < narrow)
        launch_f32<128, 128, 16, 2, 2, 2, kColSum>(name, a, b, e, M, N, K, kps, n_splits, colsum, s);
    else launch_f32<64, 64, 16, 2, 2, 5, kColSum>(name, a, b, e, M, N, K, kps, n_splits, colsum, s);
}

// Every backward product of fp32 storage.  kWide: the operands are fetched in groups of four.
template <bool kColSum, bool kWide, class AL, class BL, class Epi>
static void launch_split(const char *name, const AL &a, const BL &b, const Epi &e, int64_t M, int N, int64_t K, int64_t kps,
                         int n_splits, float *colsum, hipStream_t s)
{
    if (few_rows(kColSum ? K : M)) return launch_few_rows<kColSum>(name, a, b, e, M, N, K, kps, n_splits, colsum, s);
    if constexpr (!kWide) {   // rare, and bound by its loads: one tile is enough
        launch_gemm<128, 64, 32, 4, 1, kColSum, float>(name, a, b, e, M, N, K, kps, n_splits, colsum, s);
    } else {
        if (N <= 64) launch_gemm<128, 64, 32, 4, 1, kColSum, float>(name, a, b, e, M, N, K, kps, n_splits, colsum, s);
        else if (N <= 96) launch_gemm<128, 96, 32, 4, 1, kColSum, float>(name, a, b, e, M, N, K, kps, n_splits, colsum, s);
        else launch_split_128<kColSum>(name, a, b, e, M, N, K, kps, n_splits, colsum, s);
    }
}

template <typename CT, int BK, bool kColSum, bool kWide, class AL, class BL, class Epi>
static void launch_by_width(const char *name, const AL &a, const BL &b, const Epi &e, int64_t M, int N, int64_t K,
                            int64_t kps, int n_splits, float *colsum, hipStream_t s)
{
    if constexpr (sizeof(CT) == 4) launch_split<kColSum, kWide>(name, a, b, e, M, N, K, kps, n_splits, colsum, s);
    else {
        const int width = N <= 64 || few_tiles(M, N, n_splits) ? 64 : N <= 96 ? 96 : 128;
        if (few_rows_narrow(kColSum ? K : M, M, N, n_splits, 128, width, 110)) {
            const std::string_view whole(name), what = whole.substr(0, whole.find("_bf16"));
            char tiled[64];
            snprintf(tiled, sizeof(tiled), "%.*s_64x64%s", int(what.size()), name, name + what.size());
            launch_gemm<64, 64, BK, 2, 2, kColSum, CT, 3>(tiled, a, b, e, M, N, K, kps, n_splits, colsum, s);
        } else if (width == 64) launch_gemm<128, 64, BK, 4, 1, kColSum, CT>(name, a, b, e, M, N, K, kps, n_splits, colsum, s);
        else if (width == 96) launch_gemm<128, 96, BK, 4, 1, kColSum, CT>(name, a, b, e, M, N, K, kps, n_splits, colsum, s);
        else launch_gemm<128, 128, BK, 2, 2, kColSum, CT>(name, a, b, e, M, N, K, kps, n_splits, colsum, s);
    }
}

}  // namespace tma
