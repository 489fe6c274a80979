// Shared by the policy kernels with 16 trajectories per workgroup (policy16.hip) and the rollout with one workgroup per trajectory
// (rollout.hip): order of the units inside a block of 16, packed weights, small device functions.
#pragma once

#include "bagel_internal.h"

namespace {

// unit within a block of 16 that row 4 g + r of a tile (lane group g's register r) stands for
__host__ __device__ constexpr int unit16(int g, int r) { return ((g & 1) << 2 | g >> 1) + ((r & 1) << 1 | (r & 2) << 2); }
// instructions a contraction over the first n <= 16 units of a block needs
__host__ __device__ constexpr int steps16(int n) { return n <= 2 ? 1 : (n <= 8 ? 2 : (n <= 10 ? 3 : 4)); }
// blocks of 16 per slice of a contraction over k inputs for `rows` outputs (the split of policy.hip over its eight waves)
__host__ __device__ inline int slice_blocks(int rows, int k)
{
    const int nrt = (rows + 31) / 32, k32 = (k + 31) / 32;
    int ks = 8 / nrt;
    if (ks > k32) ks = k32;
    return 2 * ((k32 + ks - 1) / ks);
}

typedef float f4v __attribute__((ext_vector_type(4)));

// Offsets inside the packed weights, in floats (see pack_theta16_kernel)
struct pack16 {
    int nl, TT, nsi, nsa;                    // nsi, nsa: instructions for a contraction over the inputs / actions
    int fs, bs;                              // blocks per slice of the middle layer, forward and backward
    __host__ __device__ int mid_size() const { return nl == 3 ? TT * TT * 256 : 0; }
    __host__ __device__ int f_first() const { return 0; }
    __host__ __device__ int f_mid() const { return f_first() + TT * nsi * 64; }
    __host__ __device__ int f_last() const { return f_mid() + mid_size(); }
    __host__ __device__ int bias(int l) const { return f_last() + TT * 256 + l * TT * 16; }
    __host__ __device__ int b_top() const { return bias(2) + 16; }
    __host__ __device__ int b_mid() const { return b_top() + TT * nsa * 64; }
    __host__ __device__ int b_first() const { return b_mid() + mid_size(); }
    __host__ __device__ int total() const { return b_first() + TT * 256; }
};

inline pack16 make_pack(const bagel_ctx *c)
{
    const int TT = c->p16 == 1 ? 4 : (c->p16 == 2 ? 8 : 16);
    return pack16{c->n_layers, TT, steps16(c->d_in), steps16(c->dm.d_a), slice_blocks(c->width[2], c->width[1]),
                  slice_blocks(c->width[1], c->width[2])};
}

// tanh in float32, 1 - 2 / (e^{2z} + 1): see policy.hip
__device__ __forceinline__ float tanh_fast(float z)
{
    const float t = __builtin_amdgcn_exp2f(z * 2.8853900817779268f);
    return fmaf(-2.0f, __builtin_amdgcn_rcpf(t + 1.0f), 1.0f);
}

__device__ __forceinline__ f4v mfma16(float a, float b, f4v acc) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, acc, 0, 0, 0); }

// 4-byte read that the optimiser keeps where it is written (see policy.hip)
__device__ __forceinline__ float load_pinned(const float *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT); }
__device__ __forceinline__ double load_pinned(const double *p)
{
    const unsigned long long v = __hip_atomic_load(reinterpret_cast<const unsigned long long *>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
    return __longlong_as_double((long long)v);
}

}  // namespace
