// The 16x16x4 matrix-core instruction of either precision (lane layouts: see the
// matrix-core form in ppq_hpsi.hip).
#pragma once
#include "ppq_internal.hpp"

namespace ppq {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef double doublex4 __attribute__((ext_vector_type(4)));

template <class R>
struct Mma;
template <>
struct Mma<float> {
    using V4 = floatx4;
    __device__ static V4 op(float a, float b, V4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
    // row of the accumulator's element r in lane group kr, and the digit fed
    // by lane group k at step kb: the same map, so a lane holds outputs at
    // exactly the digits it feeds
    __device__ static int row(int k, int r) { return 4 * k + r; }
};
template <>
struct Mma<double> {
    using V4 = doublex4;
    __device__ static V4 op(double a, double b, V4 c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
    __device__ static int row(int k, int r) { return k + 4 * r; }
};

}  // namespace
}  // namespace ppq
