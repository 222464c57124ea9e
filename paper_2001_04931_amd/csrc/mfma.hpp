// What the kernels on the 16x16x4 matrix instructions share (gfx950): the
// instruction and its state layout per dtype (described in rollout_linear.hpp),
// and the barrier of their LDS exchanges.
#pragma once
#include <hip/hip_runtime.h>

namespace empc {

// s_waitcnt operand for gfx9: vmcnt = 0, expcnt and lgkmcnt left at their
// maxima (no wait)
constexpr int VMCNT0 = 0x0F70;

template <typename T>
struct Mfma;
template <>
struct Mfma<float> {
    typedef float v4 __attribute__((ext_vector_type(4)));
    __device__ static inline v4 op(float a, float b, v4 c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    // state held by register v of lane group g, and the state whose row the
    // A operand of lane c (output row c) carries
    __device__ static constexpr int row(int g, int v) { return g + 4 * v; }
    __device__ static constexpr int mstate(int c) { return (c >> 2) + 4 * (c & 3); }
};
template <>
struct Mfma<double> {
    typedef double v4 __attribute__((ext_vector_type(4)));
    __device__ static inline v4 op(double a, double b, v4 c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    __device__ static constexpr int row(int g, int v) { return g + 4 * v; }
    __device__ static constexpr int mstate(int c) { return c; }
};

__device__ inline void lds_barrier() {
    // orders LDS accesses only: outstanding global loads (knot prefetches)
    // are not waited for
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

}  // namespace empc
