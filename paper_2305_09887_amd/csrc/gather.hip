// Row gather  dst[i,:] = src[l2g[i],:]  -- how a trainer takes its part of the
// feature matrix and the label vector (Alg. 2, set-up line).  Pure data
// movement, HBM bound: row_bytes read + row_bytes written per local node.
#include "common.hpp"

#include <type_traits>

namespace tma {

constexpr int kCopies = 4;   // pieces that a thread has in flight

// W = piece of a row (uint4: 16 bytes at any 4-byte-aligned address, uint32_t, uint8_t); a row's last piece ends where the row
// does, and so may copy some bytes of the one before again.  Consecutive threads copy consecutive pieces; a block
// walks several rows.  d_n (may be NULL): the row count when it is only known on the device; n_loc is then the capacity
// of the launch.
// Short rows are bound by what a thread waits for: ids, then rows.  Both are fetched for kCopies pieces at a time (us, one by
// one, and in words of 4 bytes unless rows are whole 16-byte pieces -> so: 150,000 rows of 200 bytes 37 -> 20.5, their labels
// 8.7 -> 4.6; 125,000 rows of 512 bytes, bound by memory, 24 -> 24).
template <typename W>
__global__ __launch_bounds__(256) void gather_rows_kernel(int64_t n_cap, const int32_t *__restrict__ d_n,
                                                          const int32_t *__restrict__ l2g,
                                                          const char *__restrict__ src, int64_t src_ld,
                                                          int32_t pieces, int32_t last, int32_t rows_per_block,
                                                          char *__restrict__ dst, int64_t dst_ld)
{
    typedef uint32_t Words __attribute__((ext_vector_type(4), aligned(4)));
    using Piece = std::conditional_t<sizeof(W) == 16, Words, W>;
    int64_t n_loc = n_cap;
    if (d_n && *d_n < n_loc) n_loc = *d_n;
    const int64_t row0 = int64_t(blockIdx.x) * rows_per_block;
    if (row0 >= n_loc) return;
    const int32_t rows = n_loc - row0 < rows_per_block ? int32_t(n_loc - row0) : rows_per_block;
    const int32_t block_pieces = rows * pieces;
    for (int32_t t0 = threadIdx.x; t0 < block_pieces; t0 += 256 * kCopies) {
        int32_t row[kCopies], at[kCopies], id[kCopies];
        Piece value[kCopies];
#pragma unroll
        for (int u = 0; u < kCopies; ++u) {   // (a piece past the block's last is that one again)
            const int32_t t = t0 + u * 256 < block_pieces ? t0 + u * 256 : block_pieces - 1;
            row[u] = t / pieces;
            const int32_t offset = (t - row[u] * pieces) * int32_t(sizeof(W));
            at[u] = offset < last ? offset : last;
            id[u] = l2g[row0 + row[u]];
        }
#pragma unroll
        for (int u = 0; u < kCopies; ++u) value[u] = *reinterpret_cast<const Piece *>(src + int64_t(id[u]) * src_ld + at[u]);
#pragma unroll
        for (int u = 0; u < kCopies; ++u)
            if (t0 + u * 256 < block_pieces) *reinterpret_cast<Piece *>(dst + (row0 + row[u]) * dst_ld + at[u]) = value[u];
    }
}

template <typename W>
static int launch_gather(int64_t n_loc, const int32_t *d_n, const int32_t *l2g, const void *src, int64_t src_ld,
                         int64_t row_bytes, void *dst, int64_t dst_ld, hipStream_t s)
{
    const int64_t pieces = ceil_div(row_bytes, int64_t(sizeof(W)));
    // what its threads have in flight per block, less where that leaves the chip without eight blocks per compute unit
    int64_t block_pieces = ceil_div(n_loc * pieces, int64_t(256 * 8));
    block_pieces = block_pieces < 256 ? 256 : block_pieces > 256 * kCopies ? 256 * kCopies : block_pieces;
    int64_t rows_per_block = pieces < block_pieces ? block_pieces / pieces : 1;
    constexpr int64_t kMostBlocks = (int64_t(1) << 24) - 1;   // (a launch has fewer than 2^32 threads)
    if (ceil_div(n_loc, rows_per_block) > kMostBlocks) rows_per_block = ceil_div(n_loc, kMostBlocks);
    TMA_TIMED(sizeof(W) == 16 ? "gather_rows_w16" : (sizeof(W) == 4 ? "gather_rows_w4" : "gather_rows_w1"), s);
    hipLaunchKernelGGL(gather_rows_kernel<W>, dim3(unsigned(ceil_div(n_loc, rows_per_block))), dim3(256), 0, s, n_loc,
                       d_n, l2g, static_cast<const char *>(src), src_ld, int32_t(pieces), int32_t(row_bytes - int64_t(sizeof(W))),
                       int32_t(rows_per_block), static_cast<char *>(dst), dst_ld);
    return TMA_OK;
}

static int gather_rows(const char *fn, int64_t n_loc, const int32_t *d_n, const int32_t *l2g, const void *src,
                       int64_t src_ld_bytes, int64_t row_bytes, void *dst, int64_t dst_ld_bytes, tma_stream_t stream)
{
    TMA_REQUIRE(n_loc >= 0 && row_bytes >= 0, TMA_ERR_INVALID_ARG, "%s: negative size", fn);
    if (n_loc == 0 || row_bytes == 0) return TMA_OK;
    TMA_REQUIRE(l2g && src && dst, TMA_ERR_INVALID_ARG, "%s: NULL argument", fn);
    TMA_REQUIRE(src_ld_bytes >= row_bytes && dst_ld_bytes >= row_bytes, TMA_ERR_BAD_SHAPE, "%s: pitch < row_bytes", fn);
    hipStream_t s = as_stream(stream);
    auto mult = [&](int64_t a) {
        return row_bytes % a == 0 && src_ld_bytes % a == 0 && dst_ld_bytes % a == 0 && aligned(src, size_t(a)) &&
               aligned(dst, size_t(a));
    };
    if (row_bytes / (mult(16) ? 16 : mult(4) ? 4 : 1) > (1 << 24)) return fail(TMA_ERR_BAD_SHAPE, "tma_gather_rows: rows longer than 2^24 words");
    int rc;
    if (mult(4) && row_bytes >= 16) rc = launch_gather<uint4>(n_loc, d_n, l2g, src, src_ld_bytes, row_bytes, dst, dst_ld_bytes, s);
    else if (mult(4)) rc = launch_gather<uint32_t>(n_loc, d_n, l2g, src, src_ld_bytes, row_bytes, dst, dst_ld_bytes, s);
    else rc = launch_gather<uint8_t>(n_loc, d_n, l2g, src, src_ld_bytes, row_bytes, dst, dst_ld_bytes, s);
    if (rc) return rc;
    return check_launch(fn);
}

}  // namespace tma

extern "C" int tma_gather_rows(int64_t n_loc, const int32_t *l2g, const void *src, int64_t src_ld_bytes,
                               int64_t row_bytes, void *dst, int64_t dst_ld_bytes, tma_stream_t stream)
{
    return tma::gather_rows("tma_gather_rows", n_loc, nullptr, l2g, src, src_ld_bytes, row_bytes, dst, dst_ld_bytes, stream);
}

extern "C" int tma_gather_rows_dev(int64_t cap_rows, const int32_t *d_n_rows, const int32_t *l2g, const void *src,
                                   int64_t src_ld_bytes, int64_t row_bytes, void *dst, int64_t dst_ld_bytes,
                                   tma_stream_t stream)
{
    const char *fn = "tma_gather_rows_dev";
    TMA_REQUIRE(d_n_rows, TMA_ERR_INVALID_ARG, "%s: d_n_rows is NULL", fn);
    return tma::gather_rows(fn, cap_rows, d_n_rows, l2g, src, src_ld_bytes, row_bytes, dst, dst_ld_bytes, stream);
}
