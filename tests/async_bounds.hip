// Every address that the operands of the fp32 forward products and of the bf16 products over many nodes hand out lies inside their
// arrays, and every element comes from its place: walked on the host as the kernels walk them, over arrays of exactly their size.
#include "gemm_core.hpp"
#include "gemm_bf16_async.hpp"

#include <cstdio>
#include <cstdlib>

namespace tma {
KernelTimer::KernelTimer(const char *, hipStream_t) {}
KernelTimer::~KernelTimer() {}
}  // namespace tma
using namespace tma;

static int wrong = 0;
static void expect(bool ok, const char *what, int a, int b, int c)
{
    if (!ok && ++wrong < 20) printf("%s at %d %d %d\n", what, a, b, c);
}

static void rows(int n, int F, int pitch, bool two)
{
    const int ld = F + pitch, K = two ? 2 * F : F;
    const int64_t count = int64_t(n - 1) * ld + F;
    float *H = static_cast<float *>(malloc(count * 4)), *M = static_cast<float *>(malloc(count * 4)), zero[4];
    const AsyncRows a(H, ld, M, ld, F, K, n);
    const auto check = [&](const float *p, int m, int k, int e) {
        const float *want = k < F ? H + int64_t(m) * ld + k : M + int64_t(m) * ld + (k - F), *base = k < F ? H : M;
        expect(p == want && p >= base && p + e <= base + count, "row", m, k, e);
    };
    for (int m = 0; m < n; ++m)
        for (int kt = 0; kt < K; kt += kAsyncK) {
            if (a.run(kt) > 0) {
                const float *base = kt < F ? H + kt : M + (kt - F);
                for (int k = kt; k < kt + kAsyncK; k += 4) check(base + int64_t(m) * ld + (k - kt), m, k, 4);
            }
            const int step = a.pieces() ? 4 : 1;
            for (int k = kt; k < kt + kAsyncK; k += step) {
                const float *p = a.at(m, k, zero);
                if (k < K) check(p, m, k, step);
                else expect(p == zero, "past k", m, k, step);
            }
        }
    expect(a.at(n + 3, 0, zero) == a.at(n - 1, 0, zero), "past the rows", n, F, K);
    free(H);
    free(M);
}

template <bool kSide>
static void weights(int R, int N, bool two)
{
    const int Np = (N + 3) / 4 * 4, K = kSide || !two ? R : 2 * R, columns = kSide ? 2 * Np : N;
    const int64_t count = int64_t(R) * N;
    float *W = static_cast<float *>(malloc(count * 4)), *V = static_cast<float *>(malloc(count * 4)), zero[4];
    const AsyncWeights<kSide> b{W, V, R, N, K, kSide ? Np : 0};
    for (int n = 0; n < (columns + 255) / 128 * 128; ++n)
        for (int kt = 0; kt < K; kt += kAsyncK)
            for (int k = kt; k < kt + kAsyncK; ++k) {
                const int c = n - (kSide && n >= Np ? Np : 0);
                const bool inside = n < columns && c < N;
                const float *base = (kSide ? n >= Np && n < columns : k >= R) ? V : W;
                const float *want = base + int64_t(!kSide && k >= R ? k - R : k) * N + c;
                if (b.run(kt) > 0 && n % 4 == 0) {
                    const float *p = kSide ? (b.half(n) ? V : W) + int64_t(k) * N + b.column(n) : b.first(kt) + int64_t(k - kt) * N + b.column(n);
                    expect(p >= base && p + 4 <= base + count && (!inside || p == want), "piece", k, n, N);
                }
                const int step = b.pieces() ? 4 : 1;
                if (n % step) continue;
                const float *p = b.at(k, n, zero);
                if (k >= K) expect(p == zero, "past k", k, n, N);
                else expect(p >= base && p + step <= base + count && (!inside || p == want), "element", k, n, N);
            }
    free(W);
    free(V);
}

// rows of bf16: the whole slabs of a run and the pairs of the others, as Fetch16 walks them
static void rows16(int n, int F, int Fv, int pitch, bool two)
{
    const int ld = F + pitch, K = two ? 2 * F : F;
    const int64_t count = int64_t(n - 1) * ld + F;      // (padding up to an even width is the rows' own)
    uint16_t *H = static_cast<uint16_t *>(malloc(count * 2)), *M = static_cast<uint16_t *>(malloc(count * 2)), zero[8];
    const AsyncRows16 a{H, ld, M, ld, F, Fv, K, n};
    expect(a.ok(), "form", n, F, ld);
    for (int m = 0; m < n + 2; ++m)
        for (int kt = 0; kt < K; kt += kAsyncK16) {
            const int row = m < n ? m : n - 1;
            const uint16_t *base = kt < F ? H : M;
            if (a.run(kt) > 0) {
                const uint16_t *p = base + int64_t(row) * ld + (kt < F ? kt : kt - F);
                expect(kt + kAsyncK16 <= (kt < F ? Fv : K) && p >= base && p + kAsyncK16 <= base + count, "slab", m, kt, F);
            }
            for (int k = kt; k < kt + kAsyncK16; k += 2) {
                const uint16_t *p = a.at(m, k, zero);
                if (k >= K || (k >= Fv && k < F)) expect(p == zero, "outside", m, k, F);
                else expect(p == (k < F ? H + int64_t(row) * ld + k : M + int64_t(row) * ld + (k - F)) && p + 2 <= (k < F ? H : M) + count, "pair", m, k, F);
            }
        }
    free(H);
    free(M);
}

// columns of bf16 nodes as FetchCols16 walks them: whole slabs before the one that holds the last node, pairs in that one
template <int COLS>
static void cols16(int n, int F, int pitch, bool two)
{
    typedef FetchCols16<COLS, 4> Fetch;
    const int ld = F + F % 2 + pitch, Fq = (F + 7) / 8 * 8, width = two ? 2 * Fq : Fq;
    const int64_t count = int64_t(n - 1) * ld + F + F % 2;
    uint16_t *H = static_cast<uint16_t *>(malloc(count * 2)), *M = static_cast<uint16_t *>(malloc(count * 2)), zero[8];
    const AsyncCols16 x{H, ld, M, ld, F, Fq, width, n};
    expect(x.ok(), "form", n, F, ld);
    for (int c0 = 0; c0 < width; c0 += COLS)
        for (int k = 0; k < n; k += kAsyncK16)
            for (int place = 0; place < COLS * kAsyncK16 / 8; ++place) {
                const int node = k + place / Fetch::kPieces, c = c0 + ((place % Fetch::kPieces) ^ (4 * (place / Fetch::kPieces & 3))) * 8;
                const bool second = c >= Fq && c < width, inside = c < width && c - (second ? Fq : 0) < F;
                const uint16_t *base = second ? M : H, *want = base + int64_t(node) * ld + (c - (second ? Fq : 0));
                if (k + kAsyncK16 < n) {
                    const uint16_t *p = x.piece(node, c);
                    expect(p >= base && p + 8 <= base + count && (!inside || p == want), "piece", node, c, F);
                } else {
                    for (int e = 0; e < 8; e += 2) {
                        const uint16_t *p = x.at(node, c + e, zero);
                        const bool own = c < width && c + e - (second ? Fq : 0) < F;
                        if (node >= n) expect(p == zero, "past the nodes", node, c, F);
                        else expect(p >= base && p + 2 <= base + count && (!own || p == want + e), "pair", node, c, F);
                    }
                }
            }
    free(H);
    free(M);
}

// the mask of a ReLU, for every value of it
static void positive()
{
    for (uint32_t h = 0; h < 65536; ++h) {
        const bool above = __builtin_bit_cast(float, h << 16) > 0.0f;
        expect(where_positive(0xABCD8001u, h << 16 | (65535 - h)) >> 16 == (above ? 0xABCDu : 0u), "mask, upper half", int(h), 0, 0);
        expect((where_positive(0xABCD8001u, (65535 - h) << 16 | h) & 0xFFFFu) == (above ? 0x8001u : 0u), "mask, lower half", int(h), 0, 0);
    }
}

int main()
{
    positive();
    for (int F : {8, 9, 30, 47, 48, 64, 100, 128, 150, 256, 300})
        for (int n : {1, 31, 32, 33, 64, 97})
            for (int pitch : {0, 2, 6}) {
                cols16<256>(n, F, pitch, false);
                cols16<256>(n, F, pitch, true);
                cols16<128>(n, F, pitch, true);
            }
    for (int F : {2, 8, 16, 30, 32, 34, 48, 50, 64, 96, 100, 150, 256})
        for (int n : {1, 3})
            for (int pitch : {0, 2, 6})
                for (int less : {0, 1, 7}) {
                    if (less < F) rows16(n, F, F - less, pitch, true);
                    rows16(n, F, F, pitch, false);
                }
    for (int F : {1, 2, 3, 4, 5, 7, 8, 12, 15, 16, 17, 20, 31, 32, 33, 48, 50, 63, 64, 90, 100, 128, 150}) {
        for (int n : {1, 2, 5})
            for (int pitch : {0, 1, 3, 4}) rows(n, F, pitch, false), rows(n, F, pitch, true);
        for (int N : {1, 2, 3, 4, 5, 6, 7, 8, 31, 41, 47, 48, 64, 97, 130}) {
            weights<false>(F, N, false);
            weights<false>(F, N, true);
            weights<true>(F, N, false);
        }
    }
    printf("%d wrong\n", wrong);
    return wrong ? 1 : 0;
}
