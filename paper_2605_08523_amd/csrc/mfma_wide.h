// The 16 x 16 x 4 MFMAs of the FP32 and FP64 kernels and their lane layouts.
#pragma once

#include <hip/hip_runtime.h>

namespace fe {
namespace wide {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef double doublex4 __attribute__((ext_vector_type(4)));

template <typename T>
struct Mfma;

// v_mfma_f32_16x16x4f32: lane l supplies A[l % 16][l / 16] and B[l / 16][l % 16];
// acc[i] of lane l holds D[4 (l / 16) + i][l % 16].
template <>
struct Mfma<float> {
    using vec = floatx4;
    __device__ static vec mma(float a, float b, vec c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    __device__ static int crow(int lane, int i) { return 4 * (lane >> 4) + i; }
};

// v_mfma_f64_16x16x4f64: the same operands; acc[i] of lane l holds D[4 i + l / 16][l % 16].
template <>
struct Mfma<double> {
    using vec = doublex4;
    __device__ static vec mma(double a, double b, vec c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    __device__ static int crow(int lane, int i) { return 4 * i + (lane >> 4); }
};

}  // namespace wide
}  // namespace fe
