// dk_mma.h -- 16 x 16 x 4 matrix products of FP64 and FP32 operands.
#pragma once
#include <hip/hip_runtime.h>

namespace dk {

// row(i, q): the row of the result in register i of lane group q (lane / 16); its column is lane % 16
template <typename Real> struct Mma;
template <> struct Mma<double> {
    typedef double Acc __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ Acc mul(double a, double b, Acc c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
    static constexpr __host__ __device__ int row(int i, int q) { return 4 * i + q; }
};
template <> struct Mma<float> {
    typedef float Acc __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ Acc mul(float a, float b, Acc c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
    static constexpr __host__ __device__ int row(int i, int q) { return 4 * q + i; }
};

}  // namespace dk
