// Runs the operand views of the products on the host, over every position a tile can ask for, on arrays that end (or begin)
// at a page that may not be read.  The last line printed names the case; a read outside an array ends the process there.
//   view_bounds F_in F_out n
#include <hip/hip_runtime.h>
#undef __device__
#define __device__ __attribute__((host)) __attribute__((device))
#define __uint_as_float(x) __builtin_bit_cast(float, uint32_t(x))
#define __float_as_uint(x) __builtin_bit_cast(uint32_t, float(x))
#include "gemm_core.hpp"

#include <sys/mman.h>
#include <unistd.h>

#include <cstdio>
#include <cstdlib>

using namespace tma;

template <typename T>
struct Guarded {   // `count` elements between two unreadable pages, at the end or at the beginning of what lies between
    char *base;
    size_t bytes;
    T *p;
    Guarded(int64_t count, bool at_end)
    {
        const size_t page = size_t(sysconf(_SC_PAGESIZE));
        bytes = round_up(size_t(count) * sizeof(T), page);
        base = static_cast<char *>(mmap(nullptr, bytes + 2 * page, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0));
        if (base == MAP_FAILED) exit(3);
        mprotect(base, page, PROT_NONE);
        mprotect(base + page + bytes, page, PROT_NONE);
        p = reinterpret_cast<T *>(base + page + (at_end ? bytes - size_t(count) * sizeof(T) : 0));
        bytes += 2 * page;
    }
    Guarded(const Guarded &) = delete;
    ~Guarded() { munmap(base, bytes); }
};

template <class Raw>
static void wanted(const Raw &r) { asm volatile("" : : "r"(&r) : "memory"); }   // (all of it: no part of a load is left out)
template <class View>
static void every_position(const char *name, const View &v, int64_t mn_extent, int64_t k_extent)
{
    printf("%s\n", name);
    fflush(stdout);
    const int mn_step = View::kContigK ? 1 : 4, k_step = View::kContigK ? 4 : 1;
    for (int64_t mn = 0; mn < int64_t(round_up(size_t(mn_extent), 256)); mn += mn_step) {
        const typename View::Lane lane = v.prepare(mn);
        for (int64_t k = 0; k < int64_t(round_up(size_t(k_extent), 32)); k += k_step) {
            wanted(v.load(lane, k));
            if (k < k_extent / 16 * 16) wanted(v.load_plain(lane, k / 16 * 16, int(k % 16)));
        }
    }
}

// Rows with room up to `pitch`; where the views leave the padding alone the array ends with the last row's elements.
template <typename T>
static void rows_of(const char *type, int64_t n, int F_in, int F_out, int64_t ldh, int64_t ldg, bool at_end)
{
    char name[160];
    const bool h_padded = vec4_ok(static_cast<const T *>(nullptr), ldh), g_padded = vec4_ok(static_cast<const T *>(nullptr), ldg);
    const Guarded<T> H(h_padded && F_in % 4 ? n * ldh : (n - 1) * ldh + F_in, at_end);
    const Guarded<T> G(g_padded && F_out % 4 ? n * ldg : (n - 1) * ldg + F_out, at_end);
    const int Fp = int(round_up(size_t(F_out), sizeof(T) == 4 ? 4 : 8));
    const Guarded<T> Y(n * Fp, at_end);
#define RUN(V_, MN_, K_)                                                                                              \
    do {                                                                                                              \
        snprintf(name, sizeof(name), "%s n=%ld F_in=%d F_out=%d ldh=%ld ldg=%ld end=%d: " #V_, type, long(n), F_in, F_out, \
                 long(ldh), long(ldg), int(at_end));                                                                  \
        every_position(name, V_, MN_, K_);                                                                            \
    } while (0)
    // gradients: as A (k = output feature) and as B (k = node)
    if (padded_groups_ok(G.p, ldg, F_out)) {
        RUN((MaskedGrad<true, T, true, true>{G.p, G.p, F_out, ldg, n}), n, F_out);
        RUN((MaskedGrad<false, T, true, true>{G.p, G.p, F_out, ldg, n}), F_out, n);
        RUN((SideGrad<true, T, true, true>{G.p, G.p, Y.p, F_out, Fp, ldg, Fp, n}), n, 2 * Fp);
        RUN((SideGrad<false, T, true, true>{G.p, G.p, Y.p, F_out, Fp, ldg, Fp, n}), 2 * Fp, n);
    }
    RUN((MaskedGrad<true, T, false, true>{G.p, G.p, F_out, ldg, n}), n, F_out);
    RUN((MaskedGrad<false, T, false, true>{G.p, G.p, F_out, ldg, n}), F_out, n);
    RUN((SideGrad<false, T, false, true>{G.p, G.p, Y.p, F_out, Fp, ldg, Fp, n}), 2 * Fp, n);
    // layer inputs: [H | M] in the aggregate-first form, H alone otherwise
    if (groups_ok(H.p, ldh, F_in)) {
        RUN((CatRows<T, true>{H.p, ldh, H.p, ldh, F_in, n, 2 * F_in}), n, 2 * F_in);
        RUN((CatRowsT<T, true>{H.p, ldh, H.p, ldh, F_in, n, 2 * F_in}), 2 * F_in, n);
    }
    if (padded_groups_ok(H.p, ldh, F_in)) {
        if constexpr (sizeof(T) == 2) RUN((PaddedRows{H.p, ldh, F_in, n}), n, F_in);
        RUN((CatRowsT<T, true>{H.p, ldh, H.p, ldh, F_in, n, F_in}), F_in, n);
    }
    RUN((CatRows<T, false>{H.p, ldh, H.p, ldh, F_in, n, 2 * F_in}), n, 2 * F_in);
    RUN((CatRowsT<T, false>{H.p, ldh, H.p, ldh, F_in, n, 2 * F_in}), 2 * F_in, n);
    RUN((CatRowsT<T, false>{H.p, ldh, H.p, ldh, F_in, n, F_in}), F_in, n);
    if constexpr (sizeof(T) == 4)
        if (rows_u_ok(n, ldh, F_in)) RUN((CatRowsTU{H.p, ldh, H.p, ldh, F_in, pad4(F_in), n}), 2 * pad4(F_in), n);
}

static void weights_of(int F_in, int F_out, bool at_end)
{
    char name[160];
    const int64_t n = 0, ldh = 0, ldg = 0;
    const char *type = "weights";
    const Guarded<float> W(int64_t(F_in) * F_out, at_end), V(int64_t(F_in) * F_out, at_end);
    const int Fp = int(round_up(size_t(F_out), 8));
    if (F_out % 4 == 0) {
        RUN((CatWeights<true>{W.p, V.p, F_in, F_out}), F_out, 2 * F_in);
        RUN((CatWeightsT<true>{W.p, V.p, F_in, F_out}), 2 * F_in, F_out);
    }
    RUN((CatWeights<false>{W.p, V.p, F_in, F_out}), F_out, 2 * F_in);
    RUN((CatWeightsT<false>{W.p, V.p, F_in, F_out}), 2 * F_in, F_out);
    if (F_out % 4 == 0 && aligned(W.p, 16)) {
        RUN((SideWeights<kAligned4>{W.p, V.p, F_in, F_out, Fp}), 2 * Fp, F_in);
        RUN((SideWeightsT<kAligned4>{W.p, V.p, F_in, F_out, Fp}), F_in, 2 * Fp);
    }
    RUN((SideWeights<kElementwise>{W.p, V.p, F_in, F_out, Fp}), 2 * Fp, F_in);
    if (weights_u_ok(F_in, F_out)) {
        RUN((CatWeightsTU{W.p, V.p, F_in, F_out}), 2 * F_in, F_out);
        RUN((SideWeights<kUnaligned4>{W.p, V.p, F_in, F_out, Fp}), 2 * Fp, F_in);
        RUN((SideWeightsT<kUnaligned4>{W.p, V.p, F_in, F_out, Fp}), F_in, 2 * Fp);
    }
}

int main(int argc, char **argv)
{
    if (argc != 4) return 2;
    const int F_in = atoi(argv[1]), F_out = atoi(argv[2]);
    const int64_t n = atoll(argv[3]);
    for (int at_end = 0; at_end < 2; ++at_end) {
        weights_of(F_in, F_out, at_end);
        for (int pitch = 0; pitch < 9; ++pitch) {
            rows_of<float>("fp32", n, F_in, F_out, F_in + pitch, F_out + pitch, at_end);
            rows_of<uint16_t>("bf16", n, F_in, F_out, F_in + pitch, F_out + pitch, at_end);
        }
    }
    printf("done\n");
    return 0;
}
