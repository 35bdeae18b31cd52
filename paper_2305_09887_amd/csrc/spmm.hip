// Mean aggregation  M = Abar H  (paper Thm. 1, first equation of its proof) and
// the plain row gather-sum used by the backward pass.  HBM/gather bound: the
// flops (2 per gathered element) are negligible.
//
// Mapping.  A feature row is cut into 16-byte chunks; G lanes (one per chunk; any
// G up to the 64-lane wavefront, 64 / G rows share a wavefront) own one row and
// each lane keeps its chunk of the running sum in registers, so every neighbour
// row is fetched with one coalesced 16-byte load per lane.
//
// Local graphs under random assignment are very sparse (mean local degree 2-5)
// with a power-law tail.  Two things follow.  (1) A row is too short to hide a
// memory latency by itself, so a lane group walks through its rows as one
// stream of steps of up to four neighbours and runs that stream as a three-stage
// pipeline: the neighbour ids of step s+2, the feature loads of step s+1 and the
// additions of step s are in flight together, across row boundaries.  (2) A
// group can only pull a few loads per latency, so a long row would become the
// tail of the launch: rows longer than a threshold (a multiple of the mean
// degree) are deferred and then summed by all groups of the workgroup together,
// each taking one contiguous share, with a fixed-order combine through LDS.  The
// result of a row depends only on its own neighbour list and the mean degree, never
// on scheduling.
//
// Every load of the pipeline but a finished row's own (see row_extra) is issued unconditionally (an unused slot
// repeats an address that was just fetched): the wait counters are then exact and a wait for step s never also
// waits for the loads of step s+1.
//
// Dense graphs whose rows sit in the caches are bound by the vector units: 35 instructions a slot of 256 bf16 columns,
// 16 of them the sum's, kept these 94 % busy.  So a group has a multiple of four lanes (those past the last chunk repeat
// it): each fetches one of a step's four ids and multiplies it by the pitch, and takes the other lanes' products by lane
// permutes; a slot that is not used is skipped by the lane mask; and bounds are read one row ahead.  us, before -> so, means: 150,000 rows of 50
// entries in communities of 1,000, bf16, 256 columns 255 -> 190, 128 159 -> 130, 64 98 -> 69, 48 105 -> 82, fp32, 128 columns 247 -> 179, 48 110 -> 99; 400,000
// rows of 3.3 random ones, bound by memory, 131 -> 125, 72 -> 66, 44 -> 39, 50 -> 48, 125 -> 125 and 64 -> 64.  Groups fill a wavefront less well so (rows of 9, 10 and 21 pieces:
// five, five and two of them instead of seven, six and three), which rows in memory do not notice, 125,000 of 3.3 random ones, 9 and 21 fp32 pieces
// 21 -> 20 and 36.5 -> 34.9, nor dense ones; a power law's long rows do, 125,000 of 3.3, 9, 10 and 21 pieces 26.3 -> 26.1, 24.6 -> 25.5 and 40.5 -> 42.8.
#include "kernels.hpp"

#include <utility>

namespace tma {

constexpr int kSpmmThreads = 256;
constexpr int kDies = 8;           // accelerator dies (XCDs) of the chip
constexpr int kRowsPerGroup = 4;   // rows a lane group walks through per block
constexpr int kHubDegree = 48;     // rows longer than this are summed by the whole workgroup

__device__ __forceinline__ float load_elem(const float *p) { return *p; }
__device__ __forceinline__ float load_elem(const uint16_t *p) { return bf16_to_f32(*p); }
__device__ __forceinline__ void store_elem(float *p, float v) { *p = v; }
__device__ __forceinline__ void store_elem(uint16_t *p, float v) { *p = f32_to_bf16(v); }

// U neighbour rows (entries j .. j+U-1 of the run whose ids sit in `mine`) fetched together, then added in order.
template <typename T, int G, int CPL, int U>
__device__ __forceinline__ void gather_batch(const T *__restrict__ in, int64_t ld, int32_t mine, int j, int sub,
                                             int n_chunks, const float *__restrict__ edge_scale,
                                             float (&acc)[CPL][Chunk<T>::kElems])
{
    constexpr int E = Chunk<T>::kElems;
    float v[U][CPL][E];
    float w[U];
#pragma unroll
    for (int q = 0; q < U; ++q) {
        const int32_t id = __shfl(mine, j + q, G);
        w[q] = edge_scale ? edge_scale[id] : 1.0f;
        const T *row = in + int64_t(id) * ld;
#pragma unroll
        for (int c = 0; c < CPL; ++c)
            if (sub + c * G < n_chunks) Chunk<T>::load(row + (sub + c * G) * E, v[q][c]);
    }
#pragma unroll
    for (int q = 0; q < U; ++q)
#pragma unroll
        for (int c = 0; c < CPL; ++c)
            if (sub + c * G < n_chunks)
#pragma unroll
                for (int i = 0; i < E; ++i) acc[c][i] += edge_scale ? w[q] * v[q][c][i] : v[q][c][i];
}

// Adds the rows colidx[e] for e = beg, beg+1, ... in runs of G entries that start
// `run_stride` entries apart.  Every lane of the group gets the same trip counts.
// kDeep: up to 16 rows in flight per lane (long rows are latency bound: a 500-entry
// row walked four loads at a time sets the kernel's tail).
template <typename T, int G, int CPL, bool kDeep>
__device__ __forceinline__ void gather_sum(const T *__restrict__ in, int64_t ld, const int32_t *__restrict__ colidx,
                                           int32_t beg, int32_t end, int32_t run_stride, int sub, int n_chunks,
                                           const float *__restrict__ edge_scale,
                                           float (&acc)[CPL][Chunk<T>::kElems])
{
    for (int32_t e0 = beg; e0 < end; e0 += run_stride) {
        const int cnt = (end - e0) < G ? (end - e0) : G;
        const int32_t mine = sub < cnt ? colidx[e0 + sub] : 0;
        int j = 0;
        if constexpr (kDeep && CPL == 1 && G >= 16)
            for (; j + 16 <= cnt; j += 16) gather_batch<T, G, CPL, 16>(in, ld, mine, j, sub, n_chunks, edge_scale, acc);
        for (; j + 4 <= cnt; j += 4) gather_batch<T, G, CPL, 4>(in, ld, mine, j, sub, n_chunks, edge_scale, acc);
        for (; j < cnt; ++j) gather_batch<T, G, CPL, 1>(in, ld, mine, j, sub, n_chunks, edge_scale, acc);
    }
}

// 16 bytes from and to 4-byte-aligned addresses (the instructions need no more)
template <typename T>
__device__ __forceinline__ uint4 load_chunk(const T *p)
{
    uint4 v;
    __builtin_memcpy(&v, __builtin_assume_aligned(p, 4), 16);
    return v;
}
__device__ __forceinline__ uint4 load_global_chunk(uint64_t address)   // (a number says nothing of where it points)
{
    typedef uint32_t Words __attribute__((ext_vector_type(4), aligned(4)));
    const Words v = *(const __attribute__((address_space(1))) Words *)address;
    return make_uint4(v.x, v.y, v.z, v.w);
}
template <typename T>
__device__ __forceinline__ void store_chunk(T *p, const float (&v)[Chunk<T>::kElems])
{
    uint4 w;
    Chunk<T>::store(reinterpret_cast<T *>(&w), v);
    __builtin_memcpy(__builtin_assume_aligned(p, 4), &w, 16);
}

// What happens to a finished row sum s_v:
//   out_v = act( scale_v * s_v  [+ out_v]  [+ self_v]  [+ bias] )
//   out_v = act( scale_v * (s_v  [+ out_v]  [+ self_v])  [+ bias] )      with scale_all
// With edge_scale the sum is s_v = sum_u edge_scale[u] in_u and self_v stands for edge_scale[v] self_v
// (GCN aggregation S (A + I) S H in one pass over the unscaled H).
// scale_v = inv_deg[v] (mean) or 1; "+ out_v" accumulates onto what is there (backward: on top of
// dZ W_self^T); "+ self_v + bias" and the activation turn the gather into the layer output when the
// transform ran before the aggregation.
template <typename T>
struct SpmmOut {
    T *out;
    int64_t ld_out;
    const float *inv_deg;
    int accumulate;
    const T *self;
    int64_t ld_self;
    const float *bias;
    int F;  // valid elements of a row (bias is not applied to padding)
    int relu;
    int scale_all;  // the scale multiplies the sum with "+ out_v" / "+ self_v" already added (GCN: s_v (sum + self_v))
    const float *edge_scale;  // neighbour u enters the sum as edge_scale[u] * in_u, and self_v as edge_scale[v] * self_v
    int clear_padding;        // elements from F on come out as zeros whatever the gathered rows hold there
    EntryGate gate;
};

__device__ __forceinline__ bool shut(const EntryGate &gate, const int32_t *__restrict__ rowptr, int64_t n)
{
    return gate.side != EntryGate::kAlways && (rowptr[n] > gate.entries) != (gate.side == EntryGate::kAbove);
}

// last_col: see launch_typed (the first column of a row's last chunk)
template <typename T, int G, int CPL>
__device__ __forceinline__ void finish_row(int64_t v, const SpmmOut<T> &o, int sub, int n_chunks, int last_col,
                                           float (&acc)[CPL][Chunk<T>::kElems])
{
    constexpr int E = Chunk<T>::kElems;
    const float scale = o.inv_deg ? o.inv_deg[v] : 1.0f;
#pragma unroll
    for (int c = 0; c < CPL; ++c)
        if (sub + c * G < n_chunks) {
            const int f0 = (sub + c * G) * E < last_col ? (sub + c * G) * E : last_col;
            T *dst = o.out + v * o.ld_out + f0;
            float r[E];
#pragma unroll
            for (int i = 0; i < E; ++i) r[i] = o.scale_all ? acc[c][i] : acc[c][i] * scale;
            if (o.accumulate) {
                float old[E];
                Chunk<T>::load(dst, old);
#pragma unroll
                for (int i = 0; i < E; ++i) r[i] += old[i];
            }
            if (o.self) {
                float sv[E];
                Chunk<T>::widen(load_chunk(o.self + v * o.ld_self + f0), sv);
                const float ws = o.edge_scale ? o.edge_scale[v] : 1.0f;
#pragma unroll
                for (int i = 0; i < E; ++i) r[i] += ws * sv[i];
            }
            if (o.scale_all) {
#pragma unroll
                for (int i = 0; i < E; ++i) r[i] *= scale;
            }
            if (o.bias) {
#pragma unroll
                for (int i = 0; i < E; ++i) r[i] += (f0 + i < o.F) ? o.bias[f0 + i] : 0.0f;
            }
            if (o.relu) {
#pragma unroll
                for (int i = 0; i < E; ++i) r[i] = r[i] > 0.0f ? r[i] : 0.0f;
            }
            if (o.clear_padding) {
#pragma unroll
                for (int i = 0; i < E; ++i) r[i] = f0 + i < o.F ? r[i] : 0.0f;
            }
            store_chunk(dst, r);
        }
}

// ---------------------------------------------------------------------------------------------------
// Rows of at most 64 chunks: the streaming kernel.

constexpr int kStreamU = 4;              // neighbours per step
constexpr int kMinDefer = 24;            // rows up to this length are never deferred
constexpr int kMinDeferOverlap = 256;    // the same for fp32 rows with an overlapping last piece (see launch_typed)
constexpr int kDeferFactor = 4;          // ... nor rows up to this multiple of the mean degree
constexpr int kMaxRowsPerBlock = 512;    // rows of one workgroup (their bounds, scales and the deferred-row list sit in LDS;
// groups of four lanes, rows of up to four pieces, so have 8 rows at most: 12,500,000 rows of 3.3 entries, 1 and 4 pieces 937 and 1,128 us, of 1,024 rows 961 and 1,147)
// LDS for the partial sums of deferred rows: room for five workgroups to a compute unit instead of the seven of 16 KB, and more hubs pass at a time.  us, 16 KB ->
// 24, means: power law, 125,000 rows of 3.3 entries, 8 bf16 columns 95 -> 75, fp32, 12 and 36 columns 26.1 -> 22.9 and 28.8 -> 25.8, 1,000,000 of 20, 128 columns
// 1,289 -> 1,280, of 3.3 345 -> 359; bf16, 256 columns, 150,000 of 50 in communities and 1,000,000 of 20 random ones 205 and 1,454, either way.
constexpr int kPartialBytes = 24576;

// (A choice between two arrays: without the name of their memory a load from it would wait for all others and be waited for.)
typedef const __attribute__((address_space(1))) int32_t *GlobalIds;

// One step of a group's stream: add the rows ids[lo .. lo + count) (at most kStreamU) to the running sum of
// segment `seg`; `last` closes the segment.  seg < 0: nothing left (the loads of such a step are dummies).
struct Step {
    int32_t lo, count, seg;
    bool last;
};

// What lane q of every four lanes holds.  (Additions in assembler that take another lane's word as an operand are one instruction less an
// address, but their carry has to be waited for, which only the compiler does by itself: with the waits written out they are as fast as this,
// within 1.5 % at 1 to 64 pieces a row, dense and sparse.)
template <int q>
__device__ __forceinline__ uint32_t of_quad(uint32_t x)
{
    return uint32_t(__builtin_amdgcn_update_dpp(0, int32_t(x), q * 0x55, 0xF, 0xF, true));
}
// (words side by side: shifted and joined they would be added one by one)
template <int q>
__device__ __forceinline__ uint64_t of_quad(uint64_t x)
{
    typedef uint32_t Words __attribute__((ext_vector_type(2)));
    const Words mine = __builtin_bit_cast(Words, x);
    Words there;
    there.x = of_quad<q>(mine.x);
    there.y = of_quad<q>(mine.y);
    return __builtin_bit_cast(uint64_t, there);
}
template <typename Fn, int... q>
__device__ __forceinline__ void unrolled(Fn &&fn, std::integer_sequence<int, q...>)
{
    (fn(std::integral_constant<int, q>{}), ...);
}
template <typename Fn>
__device__ __forceinline__ void for_each_slot(Fn &&fn)
{
    unrolled(fn, std::make_integer_sequence<int, kStreamU>{});
}

// The id that this lane fetches for its four.  An unused slot repeats the step's last entry, a step without entries the
// entry before it: rows that this group fetched a moment ago.
__device__ __forceinline__ int32_t step_id(GlobalIds ids, const Step &s)
{
    const int32_t k = int32_t(threadIdx.x) & 3;
    const int32_t at = s.lo + (k < s.count - 1 ? k : s.count - 1);
    return ids[uint32_t(at > 0 ? at : 0)];
}

// The rows of a matrix as a lane reads them: its chunk of row 0, and the rows' pitch in bytes.  Ids are not negative and a
// pitch fits 32 bits (launch_typed), so that a row is one 32 x 32 bit multiplication away, of a quarter of the rate.
struct LaneRows {
    const char *first;
    uint32_t pitch;
};

// The rows of a step and, with kEdge, the weight of the row whose id this lane fetched.
template <typename T, bool kEdge>
struct StepRows {
    uint4 chunk[kStreamU];
    float weight;
    __device__ __forceinline__ void issue(const LaneRows &in, const float *__restrict__ edge_scale, int32_t id)
    {
        const uint64_t mine = uint64_t(uint32_t(id)) * in.pitch, first = reinterpret_cast<uint64_t>(in.first);
        for_each_slot([&](auto q) { chunk[q] = load_global_chunk(first + of_quad<q>(mine)); });
        if constexpr (kEdge) weight = edge_scale[uint32_t(id)];
    }
};

// How a weighted neighbour row enters the sum: its product with the weight rounded on its own, or inside the addition.
// A forward sum is compared with zero further on, where a unit within a rounding of it is worth 1e-4 of a small batch's
// gradient and more: which of the two, and the order of the additions, is part of the result (see launch_typed).
enum class Weighting { kNone, kRounded, kFused };

template <typename T, Weighting kW, bool kFull>
__device__ __forceinline__ void consume(const Step &s, const StepRows<T, kW != Weighting::kNone> &rows, float (&acc)[Chunk<T>::kElems])
{
#pragma clang fp contract(off)
    constexpr int E = Chunk<T>::kElems;
    for_each_slot([&](auto q) {
        float w = 1.0f;
        if constexpr (kW != Weighting::kNone) w = __uint_as_float(of_quad<q>(__float_as_uint(rows.weight)));
        if (kFull || q < s.count) {   // kFull: no group of the wavefront has an unused slot
            float v[E];
            Chunk<T>::widen(rows.chunk[q], v);
#pragma unroll
            for (int i = 0; i < E; ++i) {
                if constexpr (kW == Weighting::kFused) acc[i] = fmaf(w, v[i], acc[i]);
                else if constexpr (kW == Weighting::kRounded) acc[i] += w * v[i];
                else acc[i] += v[i];
            }
        }
    });
}

// What a row's output needs besides the sum, fetched together with the row's last gathers.
struct RowExtra {
    uint4 raw;
};

// Runs the steps that `gen` hands out through the ids -> gathers -> additions pipeline.  `extra(seg, X)`
// issues the loads a closing step needs (or nothing); `emit(seg, acc, X)` takes a finished segment.
template <typename T, Weighting kW, typename Gen, typename Extra, typename Emit>
__device__ __forceinline__ void stream_segments(const LaneRows &in, GlobalIds ids,
                                                const float *__restrict__ edge_scale, bool few_groups, Gen &&gen, Extra &&extra, Emit &&emit)
{
    constexpr int E = Chunk<T>::kElems;
    using Rows = StepRows<T, kW != Weighting::kNone>;
    Rows V0, V1;
    RowExtra X0, X1;
    float acc[E];
#pragma unroll
    for (int i = 0; i < E; ++i) acc[i] = 0.0f;

    Step a = gen();
    int32_t I0 = step_id(ids, a);
    Step b = gen();
    int32_t I1 = step_id(ids, b);
    V0.issue(in, edge_scale, I0);
    extra(a, X0);
    // entering a half: step a has its gathers in flight (V0/X0 in the first half), step b its ids (I1)
    auto half = [&](int32_t &Ia, int32_t &Ib, Rows &Va, Rows &Vb, RowExtra &Xa, RowExtra &Xb) __attribute__((always_inline)) {
        const Step c = gen();
        Ia = step_id(ids, c);
        Vb.issue(in, edge_scale, Ib);
        extra(b, Xb);
        // (steps without an unused slot, where most of them are: wide bf16 rows of dense graphs, two groups or four to a wavefront;
        // 128 columns, 150,000 rows of 50 entries, 3 % less.  fp32 rows, of half the additions a slot, gain nothing.)
        if (sizeof(T) == 2 && few_groups && __all(a.count == kStreamU)) consume<T, kW, true>(a, Va, acc);
        else consume<T, kW, false>(a, Va, acc);
        if (a.last) {
            emit(a.seg, acc, Xa);
#pragma unroll
            for (int i = 0; i < E; ++i) acc[i] = 0.0f;
        }
        a = b;
        b = c;
    };
    while (a.seg >= 0) {
        half(I0, I1, V0, V1, X0, X1);
        if (a.seg < 0) break;
        half(I1, I0, V1, V0, X1, X0);
    }
}

static __device__ const int32_t kNoEntry = 0;   // what stands for the ids of a graph without entries: steps without a row read it

// kExtra: 0 = nothing, 1 = "+ self_v", 2 = "+ out_v" (accumulate).  kScale: multiply by inv_deg[v].
// kW: weighted neighbours (and self row), see SpmmOut::edge_scale.
template <typename T, int kExtra, bool kScale, Weighting kW>
__global__ __launch_bounds__(kSpmmThreads) void spmm_stream_kernel(int64_t n, const int32_t *__restrict__ rowptr,
                                                                   const int32_t *__restrict__ colidx,
                                                                   const T *__restrict__ in, int64_t ld_in,
                                                                   SpmmOut<T> o, int n_chunks, int G, int rows_per_group,
                                                                   int min_defer, int last_col)
{
    constexpr int E = Chunk<T>::kElems;
    constexpr int U = kStreamU;
    constexpr bool kEdge = kW != Weighting::kNone;
    constexpr int kHubsPerPass = kPartialBytes / (kSpmmThreads * E * int(sizeof(float)));
    if (shut(o.gate, rowptr, n)) return;
    __shared__ int32_t bounds[kMaxRowsPerBlock + 2];   // rowptr of the workgroup's rows
    __shared__ float scales[kScale ? kMaxRowsPerBlock : 1];
    __shared__ uint16_t deferred[kMaxRowsPerBlock];
    __shared__ int32_t n_deferred;
    __shared__ float partial[kPartialBytes / sizeof(float)];

    const int lane = threadIdx.x % kWave;
    const int gpw = kWave / G;                       // groups per wavefront
    const int gl = lane / G;
    const bool live = gl < gpw;                      // lanes past the last whole group idle
    const int sub = lane - gl * G;
    const int col = sub * E < last_col ? sub * E : last_col;   // first column of this lane's chunk
    const int NG = (kSpmmThreads / kWave) * gpw;
    const int grp = (threadIdx.x / kWave) * gpw + gl;

    const int rows_per_block = NG * rows_per_group;  // <= kMaxRowsPerBlock
    // Workgroups are dealt round-robin to the 8 dies, each with an L2 of its own.  Die d takes the d-th eighth of
    // the row range (the grid is a multiple of 8): rows with neighbouring ids, which on a clustered graph gather
    // from the same few hundred rows, then share one L2 instead of filling all eight with the same lines.
    const int64_t per_die = gridDim.x / kDies;
    const int64_t base = (int64_t(blockIdx.x % kDies) * per_die + blockIdx.x / kDies) * rows_per_block;
    if (base >= n) return;
    const int block_rows = int((n - base) < rows_per_block ? (n - base) : rows_per_block);   // >= 1
    // Entries are counted from the first one, so that the entry before one, where there is none, is at worst the first.
    const int32_t first_entry = rowptr[0], nnz = rowptr[n];
    for (int i = threadIdx.x; i <= block_rows; i += kSpmmThreads) bounds[i] = rowptr[base + i] - first_entry;
    if (kScale)
        for (int i = threadIdx.x; i < block_rows; i += kSpmmThreads) scales[i] = o.inv_deg[base + i];
    if (threadIdx.x == 0) n_deferred = 0;
    if (o.bias)   // where the deferred rows' sums come later
        for (int i = threadIdx.x; i < G * E; i += kSpmmThreads) partial[i] = i < o.F ? o.bias[i] : 0.0f;
    __syncthreads();
    const GlobalIds ids = nnz > first_entry ? GlobalIds(colidx + first_entry) : GlobalIds(&kNoEntry);
    const int64_t by_mean = int64_t(kDeferFactor) * (int64_t(nnz - first_entry) / n);
    const int32_t defer_above = by_mean > min_defer ? int32_t(by_mean < INT32_MAX ? by_mean : INT32_MAX) : min_defer;

    // ---- the group's own rows, block-local indices [r, r_end): entries [e, end) of row r are still to come
    int r = live ? grp * rows_per_group : block_rows;
    const int r_end = (r + rows_per_group) < block_rows ? (r + rows_per_group) : block_rows;
    const int r_first = r < block_rows ? r : 0;
    int32_t e = bounds[r_first], end = bounds[r_first + 1], next_end = bounds[r_first + 2];   // (the last may not be one: unused then)
    auto skip_long_rows = [&]() {
        while (r < r_end && end - e > defer_above) {
            if (sub == 0) deferred[atomicAdd(&n_deferred, 1)] = uint16_t(r);
            ++r;
            e = end;
            end = next_end;
            next_end = bounds[r < r_end ? r + 2 : 0];
        }
    };
    skip_long_rows();
    auto next_row_step = [&]() {
        Step s;
        const bool open = r < r_end;
        s.seg = open ? r : -1;
        s.lo = e;
        s.count = !open ? 0 : (end - e < U ? end - e : U);
        e += s.count;
        s.last = open && e == end;
        if (s.last) {
            ++r;
            end = next_end;
            next_end = bounds[r < r_end ? r + 2 : 0];
            skip_long_rows();
        }
        return s;
    };
    auto row_extra = [&](const Step &s, RowExtra &X) {
        if (kExtra == 0 || !__any(s.last)) return;   // (for all groups of a wavefront or none)
        const int64_t v = base + (s.seg >= 0 ? s.seg : r_first);
        if constexpr (kExtra == 1) X.raw = load_chunk(o.self + v * o.ld_self + col);
        if constexpr (kExtra == 2) X.raw = load_chunk(o.out + v * o.ld_out + col);
    };
    auto finish = [&](int32_t seg, const float (&acc)[E], const RowExtra &X) {
        const int64_t v = base + seg;
        const int f0 = col;
        const float scale = kScale ? scales[seg] : 1.0f;
        float res[E];
#pragma unroll
        for (int i = 0; i < E; ++i) res[i] = acc[i];
        if (kScale && !o.scale_all) {
#pragma unroll
            for (int i = 0; i < E; ++i) res[i] *= scale;
        }
        if constexpr (kExtra != 0) {
            float x[E];
            Chunk<T>::widen(X.raw, x);
#pragma unroll
            for (int i = 0; i < E; ++i) res[i] += (kEdge && kExtra == 1) ? scale * x[i] : x[i];
        }
        if (kScale && o.scale_all) {
#pragma unroll
            for (int i = 0; i < E; ++i) res[i] *= scale;
        }
        if (o.bias) {
#pragma unroll
            for (int i = 0; i < E; ++i) res[i] += partial[f0 + i];
        }
        if (o.relu) {
#pragma unroll
            for (int i = 0; i < E; ++i) res[i] = res[i] > 0.0f ? res[i] : 0.0f;
        }
        if constexpr (kEdge && kExtra == 0) {
#pragma unroll
            for (int i = 0; i < E; ++i) res[i] = (o.clear_padding && f0 + i >= o.F) ? 0.0f : res[i];
        }
        if (sub < n_chunks) store_chunk(o.out + v * o.ld_out + f0, res);
    };
    const LaneRows rows{reinterpret_cast<const char *>(in + col), uint32_t(ld_in) * uint32_t(sizeof(T))};
    stream_segments<T, kW>(rows, ids, o.edge_scale, gpw <= 4, next_row_step, row_extra, finish);
    __syncthreads();

    // ---- deferred rows, some at a time: the groups sum the shares of each, then one group each combines them in order.  A row's
    // shares, and so the order of its sum, are the groups of n_chunks lanes that a workgroup has room for, whatever its groups are.
    const int n_hubs = n_deferred;
    const int n_shares = (kSpmmThreads / kWave) * (kWave / n_chunks);   // >= NG
    const int width = n_chunks * E;                  // floats of one partial row
    const int per_pass = kHubsPerPass < NG ? kHubsPerPass : NG;
    for (int h0 = 0; h0 < n_hubs; h0 += per_pass) {
        const int h_end = (h0 + per_pass) < n_hubs ? (h0 + per_pass) : n_hubs;
        if (live) {
            int h = h0, part = grp;
            int32_t pos = 0, stop = 0;
            bool open = false;
            auto next_share_step = [&]() {
                Step s{pos, 0, -1, false};
                if (h >= h_end) return s;
                if (!open) {
                    const int row = deferred[h];
                    const int32_t beg = bounds[row], end = bounds[row + 1];
                    const int32_t share = int32_t((int64_t(end - beg) + int64_t(n_shares) * U - 1) / (int64_t(n_shares) * U)) * U;
                    const int64_t lo = int64_t(beg) + int64_t(part) * share;
                    pos = lo < end ? int32_t(lo) : end;
                    stop = (lo + share) < end ? int32_t(lo + share) : end;
                    open = true;
                }
                s.seg = (h - h0) * n_shares + part;
                s.lo = pos;
                s.count = (stop - pos > U) ? U : stop - pos;
                pos += s.count;
                s.last = pos == stop;
                if (s.last) {
                    open = false;
                    part += NG;
                    if (part >= n_shares) {
                        part -= n_shares;
                        ++h;
                    }
                }
                return s;
            };
            auto no_extra = [](const Step &, RowExtra &) {};
            auto to_lds = [&](int32_t seg, const float (&acc)[E], const RowExtra &) {
                if (sub >= n_chunks) return;
#pragma unroll
                for (int i = 0; i < E; ++i) partial[seg * width + sub * E + i] = acc[i];
            };
            stream_segments<T, kW>(rows, ids, o.edge_scale, gpw <= 4, next_share_step, no_extra, to_lds);
        }
        __syncthreads();
        if (live && sub < n_chunks && grp < h_end - h0) {
            const int64_t v = base + deferred[h0 + grp];
            float acc[E];
#pragma unroll
            for (int i = 0; i < E; ++i) acc[i] = 0.0f;
            for (int g = 0; g < n_shares; ++g)   // fixed order
#pragma unroll
                for (int i = 0; i < E; ++i) acc[i] += partial[(grp * n_shares + g) * width + sub * E + i];
            float one[1][E];
#pragma unroll
            for (int i = 0; i < E; ++i) one[0][i] = acc[i];
            finish_row<T, 1, 1>(v, o, sub, n_chunks, last_col, one);
        }
        __syncthreads();
    }
}

// Rows wider than 64 chunks (1 KB): the whole wavefront owns one row, CPL chunks per lane; rows one after
// the other, rows of more than kHubDegree entries by the whole workgroup.
template <typename T, int G, int CPL>
__global__ __launch_bounds__(kSpmmThreads) void spmm_rows_kernel(int64_t n, const int32_t *__restrict__ rowptr,
                                                                 const int32_t *__restrict__ colidx,
                                                                 const T *__restrict__ in, int64_t ld_in,
                                                                 SpmmOut<T> o, int n_chunks)
{
    constexpr int E = Chunk<T>::kElems;
    constexpr int NG = kSpmmThreads / G;
    constexpr int R = kRowsPerGroup;
    constexpr int RPB = NG * R;
    if (shut(o.gate, rowptr, n)) return;
    __shared__ int32_t hub_rows[RPB];
    __shared__ int32_t hub_count;
    __shared__ float partial[NG][G * CPL * E];

    const int sub = threadIdx.x % G;
    const int grp = threadIdx.x / G;
    if (threadIdx.x == 0) hub_count = 0;
    __syncthreads();

    // the group owns R consecutive rows v0 .. v0+R-1
    const int64_t base = int64_t(blockIdx.x) * RPB;
    const int64_t v0 = base + int64_t(grp) * R;
    for (int r = 0; r < R; ++r) {
        const int64_t v = v0 + r;
        if (v >= n) break;
        const int32_t beg = rowptr[v], end = rowptr[v + 1];
        if (end - beg > kHubDegree) {
            if (sub == 0) hub_rows[atomicAdd(&hub_count, 1)] = int32_t(v - base);
            continue;
        }
        float acc[CPL][E];
#pragma unroll
        for (int c = 0; c < CPL; ++c)
#pragma unroll
            for (int k = 0; k < E; ++k) acc[c][k] = 0.0f;
        gather_sum<T, G, CPL, false>(in, ld_in, colidx, beg, end, G, sub, n_chunks, o.edge_scale, acc);
        finish_row<T, G, CPL>(v, o, sub, n_chunks, INT32_MAX, acc);
    }
    __syncthreads();

    const int n_hubs = hub_count;
    for (int h = 0; h < n_hubs; ++h) {
        const int64_t v = base + hub_rows[h];
        const int32_t beg = rowptr[v], end = rowptr[v + 1];
        float acc[CPL][E];
#pragma unroll
        for (int c = 0; c < CPL; ++c)
#pragma unroll
            for (int k = 0; k < E; ++k) acc[c][k] = 0.0f;
        if (beg + grp * G < end) gather_sum<T, G, CPL, true>(in, ld_in, colidx, beg + grp * G, end, NG * G, sub, n_chunks, o.edge_scale, acc);
#pragma unroll
        for (int c = 0; c < CPL; ++c)
#pragma unroll
            for (int k = 0; k < E; ++k) partial[grp][(c * G + sub) * E + k] = acc[c][k];
        __syncthreads();
        if (grp == 0) {
#pragma unroll
            for (int c = 0; c < CPL; ++c)
#pragma unroll
                for (int k = 0; k < E; ++k) {
                    float s = 0.0f;
                    for (int g = 0; g < NG; ++g) s += partial[g][(c * G + sub) * E + k];  // fixed order
                    acc[c][k] = s;
                }
            finish_row<T, G, CPL>(v, o, sub, n_chunks, INT32_MAX, acc);
        }
        __syncthreads();
    }
}

// Any F, any alignment: one wavefront per row, lane owns elements lane, lane+64, ...
template <typename T>
__global__ __launch_bounds__(kSpmmThreads) void spmm_rows_generic_kernel(int64_t n, const int32_t *__restrict__ rowptr,
                                                                         const int32_t *__restrict__ colidx,
                                                                         const T *__restrict__ in, int64_t ld_in,
                                                                         SpmmOut<T> o, int F)
{
    if (shut(o.gate, rowptr, n)) return;
    constexpr int kPer = 8;  // elements per lane per sweep: 512 features per sweep
    const int lane = threadIdx.x % kWave;
    const int64_t v = int64_t(blockIdx.x) * (kSpmmThreads / kWave) + threadIdx.x / kWave;
    if (v >= n) return;
    const int32_t beg = rowptr[v], end = rowptr[v + 1];
    const float scale = o.inv_deg ? o.inv_deg[v] : 1.0f;
    for (int f0 = 0; f0 < F; f0 += kWave * kPer) {
        float acc[kPer];
#pragma unroll
        for (int k = 0; k < kPer; ++k) acc[k] = 0.0f;
        for (int32_t e = beg; e < end; ++e) {
            const int32_t u = colidx[e];
            const T *row = in + int64_t(u) * ld_in;
            const float w = o.edge_scale ? o.edge_scale[u] : 1.0f;
#pragma unroll
            for (int k = 0; k < kPer; ++k) {
                const int f = f0 + k * kWave + lane;
                if (f < F) acc[k] += w * load_elem(row + f);
            }
        }
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const int f = f0 + k * kWave + lane;
            if (f < F) {
                T *dst = o.out + v * o.ld_out + f;
                float r = o.scale_all ? acc[k] : acc[k] * scale;
                if (o.accumulate) r += load_elem(dst);
                if (o.self) r += (o.edge_scale ? o.edge_scale[v] : 1.0f) * load_elem(o.self + v * o.ld_self + f);
                if (o.scale_all) r *= scale;
                if (o.bias && f < o.F) r += o.bias[f];
                if (o.relu) r = r > 0.0f ? r : 0.0f;
                if (o.clear_padding && f >= o.F) r = 0.0f;
                store_elem(dst, r);
            }
        }
    }
}

template <typename T, int G, int CPL>
static void launch_wide_rows(int64_t n, const int32_t *rowptr, const int32_t *colidx, const T *in, int64_t ld_in,
                             const SpmmOut<T> &o, int n_chunks, hipStream_t s)
{
    constexpr int RPB = (kSpmmThreads / G) * kRowsPerGroup;
    char name[48];
    snprintf(name, sizeof(name), "%s%s_%s_g%dx%d", o.gate.side ? "gated_" : "", o.self ? "spmm_combine" : (o.inv_deg ? "spmm_mean" : "spmm_sum"),
             sizeof(T) == 4 ? "f32" : "bf16", G, CPL);
    TMA_TIMED(name, s);
    hipLaunchKernelGGL((spmm_rows_kernel<T, G, CPL>), dim3(unsigned(ceil_div(n, RPB))), dim3(kSpmmThreads), 0, s, n,
                       rowptr, colidx, in, ld_in, o, n_chunks);
}

template <typename T, int kExtra, bool kScale, Weighting kW = Weighting::kNone>
static void launch_stream(int64_t n, const int32_t *rowptr, const int32_t *colidx, const T *in, int64_t ld_in,
                          const SpmmOut<T> &o, int n_chunks, int last_col, int min_defer, hipStream_t s)
{
    const int G = int(round_up(size_t(n_chunks), 4));
    // rows per group: long enough a stream for the pipeline to pay, short enough to leave the chip
    // several workgroups per compute unit
    const int NG = (kSpmmThreads / kWave) * (kWave / G);
    // Rows per lane group: enough blocks to fill the chip six times over, 4 to 8 rows each; a group's pipeline
    // costs two extra steps to fill and drain, so on very long row ranges (millions of rows: every block runs many
    // rounds anyway) 16 rows per group amortise it better (12.5 M rows: -7 %), while on a dense cache-resident
    // graph (mean degree 44, 144 k rows) longer groups only lengthen the tail (+15 %).
    // Rows of 512 bytes and more, below four million of them: 6 rows at most, of fewer than 2^18 5.  What counts there is how many rows a die has at
    // hand at a time, in whose neighbours, where these are near, its 4 MB of L2 have to hold.  us, means over 512-byte fp32 rows, 8 rows / 8 with a
    // workgroup less to a unit / 6 / 5 or 4: communities of 1,000 rows, 150,000 of 50 entries 226 / 204 / 191 / 175 (4), 125,000 of 20 86 / - / 77 / 73, 40,000 of 3.3
    // 11.9 / 14.7 / 12.0 / 11.9 (4), 1,000,000 of 20 785 / 771 / 768 / 755 (4); random ones, 125,000 of 3.3 42.0 / - / 42.5 / 41.4, 400,000 124.8 / 130.5 / 124.8 / 127.6 (4);
    // power law, 125,000 of 3.3 44.1 / - / 46.2 / 43.8, 700,000 244 / 264 / 254 / 269 (4); 1 KB rows, communities, 150,000 of 50 439 / 399 / 378 / 355 (4),
    // power law, 60,000 of 3.3 43.0 / - / 46.2 / 44.7.
    int64_t rpg = ceil_div(n, int64_t(NG) * 256 * 6);
    const int64_t rpg_max = n >= (int64_t(1) << 22) ? 16 : n_chunks < 32 ? 8 : n >= (int64_t(1) << 18) ? 6 : 5;
    rpg = rpg < 4 ? 4 : (rpg > rpg_max ? rpg_max : rpg);
    if (rpg * NG > kMaxRowsPerBlock) rpg = kMaxRowsPerBlock / NG;
    char name[48];
    snprintf(name, sizeof(name), "%s%s_%s_g%dx1", o.gate.side ? "gated_" : "",
             kW != Weighting::kNone ? "spmm_weighted" : (kExtra == 1 ? "spmm_combine" : (kScale ? "spmm_mean" : "spmm_sum")),
             sizeof(T) == 4 ? "f32" : "bf16", n_chunks);
    TMA_TIMED(name, s);
    const dim3 grid(unsigned(round_up(size_t(ceil_div(n, rpg * NG)), kDies)));
    hipLaunchKernelGGL((spmm_stream_kernel<T, kExtra, kScale, kW>), grid, dim3(kSpmmThreads), 0, s, n, rowptr,
                       colidx, in, ld_in, o, n_chunks, G, int(rpg), min_defer, last_col);
}

template <typename T>
static int launch_typed(int64_t n, const int32_t *rowptr, const int32_t *colidx, const T *in, int64_t ld_in, int32_t F,
                        const SpmmOut<T> &o, hipStream_t s)
{
    // A row is walked in whole 16-byte pieces.  A width that is no multiple of 16 bytes (100 bf16 elements) still
    // takes this path when every pitch leaves room for the last piece: the piece's tail then reads and writes
    // padding elements inside the rows (never memory outside them).
    const size_t row_bytes = round_up(size_t(F) * sizeof(T), 16);
    const bool vec_ok = (size_t(ld_in) * sizeof(T)) % 16 == 0 && size_t(ld_in) * sizeof(T) >= row_bytes &&
                        (size_t(o.ld_out) * sizeof(T)) % 16 == 0 && size_t(o.ld_out) * sizeof(T) >= row_bytes &&
                        aligned(in, 16) && aligned(o.out, 16) &&
                        (!o.self || ((size_t(o.ld_self) * sizeof(T)) % 16 == 0 && aligned(o.self, 16) &&
                                     size_t(o.ld_self) * sizeof(T) >= row_bytes)) &&
                        row_bytes / 16 <= 256 && !(o.self && o.accumulate);
    // Rows that leave no such room (90 fp32 elements side by side) take it with their last piece moved back to the
    // row's end: it then covers some elements of the piece before a second time, with the same sums, stored twice.
    // Not on top of what is there (accumulate), which would be added twice; the pieces need 4-byte alignment.  A mean
    // over 90 fp32 features on 40,004 rows: 38 us element by element, 17 us so.
    constexpr int E = Chunk<T>::kElems;
    const auto words = [](const void *p, int64_t ld) { return aligned(p, 4) && (size_t(ld) * sizeof(T)) % 4 == 0; };
    const bool overlap = !vec_ok && F >= E && (size_t(F) * sizeof(T)) % 4 == 0 && row_bytes / 16 <= 64 && !o.accumulate &&
                         words(in, ld_in) && words(o.out, o.ld_out) && (!o.self || words(o.self, o.ld_self));
    const int last_col = overlap ? F - E : int(row_bytes / sizeof(T)) - E;
    // The order of the additions is kept as it was before such rows came here (element by element, in neighbour order):
    // fp32 rows are cut into shares only where one group would take longer than the rest of the launch (means over 90
    // features of a power-law graph, never / above 256 / above 24 entries: 110 / 68 / 32 us at 40,000 nodes, 611 / 359 /
    // 347 us at 300,000), which no sampled block and fewer than one row in a thousand of a power-law graph reaches.
    const int min_defer = overlap && sizeof(T) == 4 ? kMinDeferOverlap : kMinDefer;
    // the streaming kernel's weighted forms: with the self weight from the row scale it already holds, or without
    // self, scale and accumulation
    const bool edge_self = o.edge_scale && o.self && o.inv_deg == o.edge_scale;
    const bool edge_plain = o.edge_scale && !o.self && !o.inv_deg && !o.accumulate;
    const bool far = size_t(ld_in) * sizeof(T) > UINT32_MAX;   // (see LaneRows)
    if ((!vec_ok && !overlap) || (far && row_bytes / 16 <= 64) || (o.edge_scale && !edge_self && !edge_plain && row_bytes / 16 <= 64)) {
        TMA_TIMED(o.gate.side ? "gated_spmm_generic" : o.self ? "spmm_combine_generic" : (o.inv_deg ? "spmm_mean_generic" : "spmm_sum_generic"), s);
        hipLaunchKernelGGL((spmm_rows_generic_kernel<T>), dim3(unsigned(ceil_div(n, kSpmmThreads / kWave))),
                           dim3(kSpmmThreads), 0, s, n, rowptr, colidx, in, ld_in, o, F);
        return check_launch("spmm (generic)");
    }
    const int nc = int(row_bytes / 16);
    if (nc <= 64) {
        const int extra = o.self ? 1 : (o.accumulate ? 2 : 0);
#define TMA_SPMM_STREAM(X, S) launch_stream<T, X, S>(n, rowptr, colidx, in, ld_in, o, nc, last_col, min_defer, s)
        if (edge_self) {
            if (overlap) launch_stream<T, 1, true, Weighting::kFused>(n, rowptr, colidx, in, ld_in, o, nc, last_col, min_defer, s);
            else launch_stream<T, 1, true, Weighting::kRounded>(n, rowptr, colidx, in, ld_in, o, nc, last_col, min_defer, s);
        } else if (edge_plain) {
            launch_stream<T, 0, false, Weighting::kFused>(n, rowptr, colidx, in, ld_in, o, nc, last_col, min_defer, s);
        } else if (o.inv_deg) {
            if (extra == 0) TMA_SPMM_STREAM(0, true);
            else if (extra == 1) TMA_SPMM_STREAM(1, true);
            else TMA_SPMM_STREAM(2, true);
        } else {
            if (extra == 0) TMA_SPMM_STREAM(0, false);
            else if (extra == 1) TMA_SPMM_STREAM(1, false);
            else TMA_SPMM_STREAM(2, false);
        }
#undef TMA_SPMM_STREAM
    } else if (nc <= 128) {
        launch_wide_rows<T, 64, 2>(n, rowptr, colidx, in, ld_in, o, nc, s);
    } else {
        launch_wide_rows<T, 64, 4>(n, rowptr, colidx, in, ld_in, o, nc, s);
    }
    return check_launch("spmm");
}

template <typename T>
static int spmm_any(int64_t n, const int32_t *rowptr, const int32_t *colidx, const float *inv_deg, const void *in,
                    int64_t ld_in, int32_t F, void *out, int64_t ld_out, bool accumulate, const void *self,
                    int64_t ld_self, const float *bias, int32_t F_valid, bool relu, bool scale_all,
                    const float *edge_scale, EntryGate gate, hipStream_t stream)
{
    SpmmOut<T> o{static_cast<T *>(out), ld_out, inv_deg, accumulate ? 1 : 0, static_cast<const T *>(self), ld_self,
                 bias, F_valid, relu ? 1 : 0, (scale_all && inv_deg) ? 1 : 0, edge_scale, F_valid < F ? 1 : 0, gate};
    return launch_typed<T>(n, rowptr, colidx, static_cast<const T *>(in), ld_in, F, o, stream);
}

int launch_spmm(int64_t n, const int32_t *rowptr, const int32_t *colidx, const float *inv_deg, const void *in,
                int64_t ld_in, int32_t F, int32_t dtype, void *out, int64_t ld_out, bool accumulate,
                hipStream_t stream, EntryGate gate)
{
    return launch_spmm_combine(n, rowptr, colidx, inv_deg, in, ld_in, F, dtype, out, ld_out, accumulate, nullptr, 0,
                               nullptr, F, false, false, nullptr, stream, gate);
}

int launch_spmm_combine(int64_t n, const int32_t *rowptr, const int32_t *colidx, const float *inv_deg, const void *in,
                        int64_t ld_in, int32_t F, int32_t dtype, void *out, int64_t ld_out, bool accumulate,
                        const void *self, int64_t ld_self, const float *bias, int32_t F_valid, bool relu,
                        bool scale_all, const float *edge_scale, hipStream_t stream, EntryGate gate)
{
    if (n == 0 || F == 0) return TMA_OK;
    if (dtype == TMA_F32)
        return spmm_any<float>(n, rowptr, colidx, inv_deg, in, ld_in, F, out, ld_out, accumulate, self, ld_self, bias,
                               F_valid, relu, scale_all, edge_scale, gate, stream);
    if (dtype == TMA_BF16)
        return spmm_any<uint16_t>(n, rowptr, colidx, inv_deg, in, ld_in, F, out, ld_out, accumulate, self, ld_self,
                                  bias, F_valid, relu, scale_all, edge_scale, gate, stream);
    return fail(TMA_ERR_UNSUPPORTED_DTYPE, "spmm: dtype %d", dtype);
}

// dst_v = inv_deg[v] * g_v (.) [h_v > 0]   (rows of F elements; padding up to F_pad is zeroed).  Whole 16-byte pieces of dst a
// thread (us, element by element -> so: 150,000 rows of 47 bf16 17.4 -> 11.7, 40,004 of 41 fp32 6.6 -> 5.3); `fetched`: pieces of g and h inside a row are.
template <typename T>
__global__ __launch_bounds__(256) void scale_mask_rows_kernel(int64_t n, int F, int pieces, const T *__restrict__ g,
                                                              const T *__restrict__ h, int64_t ld, bool fetched,
                                                              const float *__restrict__ inv_deg, int relu,
                                                              T *__restrict__ dst, int64_t ld_dst,
                                                              const int32_t *__restrict__ rowptr, EntryGate gate)
{
    if (shut(gate, rowptr, n)) return;
    constexpr int E = Chunk<T>::kElems;
    const int64_t total = n * pieces;
    const int64_t stride = int64_t(gridDim.x) * 256;
    for (int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x; i < total; i += stride) {
        const int64_t v = i / pieces;
        const int f0 = int(i - v * pieces) * E;
        const T *gv = g + v * ld + f0, *hv = h + v * ld + f0;
        float x[E], m[E];
        if (fetched && f0 + E <= F) {
            const uint4 gw = load_chunk(gv), hw = relu ? load_chunk(hv) : gw;
            Chunk<T>::widen(gw, x);
            Chunk<T>::widen(hw, m);
        } else {
#pragma unroll
            for (int j = 0; j < E; ++j) {
                const bool there = f0 + j < F;
                x[j] = there ? load_elem(gv + j) : 0.0f;
                m[j] = there && relu ? load_elem(hv + j) : 0.0f;
            }
        }
        const float scale = inv_deg[v];
#pragma unroll
        for (int j = 0; j < E; ++j) x[j] = f0 + j < F && !(relu && !(m[j] > 0.0f)) ? x[j] * scale : 0.0f;
        store_chunk(dst + v * ld_dst + f0, x);
    }
}

int launch_scale_mask_rows(int64_t n, int32_t F, int32_t F_pad, const void *g, const void *h, int64_t ld,
                           const float *inv_deg, bool relu, int32_t dtype, void *dst, int64_t ld_dst,
                           hipStream_t stream, const int32_t *rowptr, EntryGate gate)
{
    if (n == 0 || F_pad == 0) return TMA_OK;
    const size_t bytes = (dtype == TMA_BF16 ? 2 : 4);
    const int pieces = int(size_t(F_pad) * bytes / 16);
    // (callers' rows are whole pieces; loads of 16 bytes need 4-byte-aligned rows)
    const bool fetched = (size_t(ld) * bytes) % 4 == 0 && aligned(g, 4) && (!relu || aligned(h, 4));
    int64_t blocks = ceil_div(n * pieces, 256);
    if (blocks > 256 * 32) blocks = 256 * 32;
    TMA_TIMED(gate.side ? "gated_scale_mask_rows" : "scale_mask_rows", stream);
    if (dtype == TMA_F32)
        hipLaunchKernelGGL(scale_mask_rows_kernel<float>, dim3(unsigned(blocks)), dim3(256), 0, stream, n, F, pieces,
                           static_cast<const float *>(g), static_cast<const float *>(h), ld, fetched, inv_deg, relu ? 1 : 0,
                           static_cast<float *>(dst), ld_dst, rowptr, gate);
    else
        hipLaunchKernelGGL(scale_mask_rows_kernel<uint16_t>, dim3(unsigned(blocks)), dim3(256), 0, stream, n, F, pieces,
                           static_cast<const uint16_t *>(g), static_cast<const uint16_t *>(h), ld, fetched, inv_deg,
                           relu ? 1 : 0, static_cast<uint16_t *>(dst), ld_dst, rowptr, gate);
    return check_launch("scale_mask_rows");
}

}  // namespace tma

extern "C" int tma_mean_aggregate(int64_t n, const int32_t *rowptr, const int32_t *colidx, const float *inv_deg,
                                  const void *H, int64_t ldh, int32_t F, int32_t dtype, void *M_out, int64_t ldm,
                                  tma_stream_t stream)
{
    using namespace tma;
    const char *fn = "tma_mean_aggregate";
    TMA_REQUIRE(n >= 0 && n <= INT32_MAX && F >= 0, TMA_ERR_INVALID_ARG, "%s: bad n or F", fn);
    TMA_REQUIRE(dtype == TMA_F32 || dtype == TMA_BF16, TMA_ERR_UNSUPPORTED_DTYPE, "%s: dtype %d", fn, dtype);
    if (n == 0 || F == 0) return TMA_OK;
    TMA_REQUIRE(rowptr && inv_deg && H && M_out, TMA_ERR_INVALID_ARG, "%s: NULL argument", fn);
    TMA_REQUIRE(ldh >= F && ldm >= F, TMA_ERR_BAD_SHAPE, "%s: leading dimension smaller than F", fn);
    TMA_REQUIRE(H != M_out, TMA_ERR_INVALID_ARG, "%s: in-place aggregation is not supported", fn);
    return launch_spmm(n, rowptr, colidx, inv_deg, H, ldh, F, dtype, M_out, ldm, false, as_stream(stream));
}
