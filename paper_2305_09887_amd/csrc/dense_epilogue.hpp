// What becomes of a single-operand product (after gemm_core.hpp).
#pragma once

namespace tma {

template <typename T, bool kRowScale>
struct DenseEpilogue {  // out = act(acc + b)  or  row_scale[row] * acc
    static constexpr bool kColAux = true, kRowAux = kRowScale;
    T *out;
    int64_t ld;
    const float *bias;       // may be NULL
    const float *row_scale;  // read only with kRowScale
    bool relu;
    int Fo;                  // columns from here on are stored as zeros
    __device__ __forceinline__ float col_aux(int col) const { return bias ? bias[col] : 0.0f; }
    __device__ __forceinline__ float row_aux(int64_t row) const { return kRowScale ? row_scale[row] : 0.0f; }
    __device__ __forceinline__ const float *col_at(int col) const { return bias ? bias + col : kZeros; }
    __device__ __forceinline__ const float *row_at(int64_t row) const { return row_scale + row; }
    __device__ __forceinline__ bool padding(int col) const { return col >= Fo; }
    __device__ __forceinline__ float value(float v, float caux, float raux, int) const
    {
        v += caux;
        if (kRowScale) v *= raux;
        if (relu) v = v > 0.0f ? v : 0.0f;
        return v;
    }
    __device__ __forceinline__ void store(int64_t row, int col, float v, int) const { narrow1(out + row * ld + col, v); }
    static constexpr bool kPairs = sizeof(T) == 2;
    __device__ __forceinline__ bool pairs_ok() const { return ld % 2 == 0 && word_aligned(out); }
    __device__ __forceinline__ T *at(int64_t row, int col) const { return out + row * ld + col; }
};

}  // namespace tma
