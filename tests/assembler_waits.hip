// What test_assembler_waits.py reads the assembly of: kernels whose operands are fetched in assembler, those with a mask on the way to the matrix units, one
// whose results have row and column inputs, one of fp32; and a kernel in which a fetch by hand stands between two of the compiler's into one place.
#include "gemm_core.hpp"
#include "dense_epilogue.hpp"
#include "gemm_bf16_async.hpp"

namespace tma {
KernelTimer::KernelTimer(const char *, hipStream_t) {}
KernelTimer::~KernelTimer() {}

template __global__ void gemm_bf16_weight_kernel<256, 2, 3, true>(AsyncCols16, AsyncCols16, const uint16_t *, int64_t, int, int, int, int64_t, float *, float *);
template __global__ void gemm_bf16_weight_kernel<128, 1, 4, true>(AsyncCols16, AsyncCols16, const uint16_t *, int64_t, int, int, int, int64_t, float *, float *);
template __global__ void gemm_bf16_async_kernel<256, 256, 4, 2, 3, true, false, DenseEpilogue<uint16_t, true>>(AsyncRows16, const uint16_t *, AsyncRows16,
                                                                                                              DenseEpilogue<uint16_t, true>, int64_t, int, int, int64_t);
template __global__ void gemm_f32_async_kernel<64, 64, 2, 2, 3, 4, AsyncWeights<true>, HalvesEpilogue<float>>(AsyncRows, AsyncWeights<true>, HalvesEpilogue<float>,
                                                                                                             int64_t, int, int, int64_t);

typedef __attribute__((address_space(1))) const void global_void;
typedef __attribute__((address_space(3))) void shared_void;
__global__ void two_ways(const float *p, float *q)
{
    __shared__ float a[64], b[64];
    __builtin_amdgcn_global_load_lds((global_void *)(p + threadIdx.x), (shared_void *)a, 4, 0, 0);
    lds_fetch<1>(lds_address(b), p + 64 + threadIdx.x);
    __builtin_amdgcn_global_load_lds((global_void *)(p + 128 + threadIdx.x), (shared_void *)a, 4, 0, 0);
    wait_and_meet<0>();
    q[threadIdx.x] = a[threadIdx.x] + b[threadIdx.x];
}
}  // namespace tma
