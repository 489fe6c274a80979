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

constexpr int PL = 16;                       // trajectories per workgroup
constexpr int HS = 20;                       // LDS row length of the policy input and the action adjoint

template <int NW, int NT>
struct shape16 {
    static constexpr int TT = NW * NT;       // row tiles of a hidden layer
    static constexpr int ROWS = 4 * NW;      // thread rows of 16 trajectories
    static constexpr int AS = 16 * TT + 4;   // LDS row length of the activations: rows start 4 banks apart
};

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

// theta -> the register contents of the lanes.  "tile t" = units 16 t .. of the layer that is produced, lane = 16 g + i
// with i = 4 gi + ri, u = unit16(gi, ri):
//   wide contraction   [t][kb][lane][s] = W(16 t + u, 16 kb + unit16(g, s))
//   narrow contraction [t][s][lane]     = W(16 t + u, unit16(g, s))
// with W(row, k) the layer's matrix (forward) or its transpose (backward), zero outside it.  Also the biases, padded.
struct pack16_args {
    pack16 p;
    int width[4], w_off[3], b_off[3];
    float *dst;
};
__device__ __forceinline__ void pack_theta16(const pack16_args &a, const float *__restrict__ theta, int idx)
{
    const pack16 &p = a.p;
    if (idx >= p.total()) return;
    const int (&width)[4] = a.width;
    const int wo0 = a.w_off[0], wo1 = a.w_off[1], bo0 = a.b_off[0], bo1 = a.b_off[1];
    const int last = p.nl - 1;
    const int w_last = last == 2 ? a.w_off[2] : wo1, b_last = last == 2 ? a.b_off[2] : bo1;
    const int n_last = width[last + 1], h_last = width[last];              // actions, units of the last hidden layer
    float v = 0.0f;
    auto wide = [&](int e, int &row, int &k, int kbs) {
        const int s = e & 3, lane = (e >> 2) & 63, blk = e >> 8;
        row = 16 * (blk / kbs) + unit16(lane >> 2 & 3, lane & 3);
        k = 16 * (blk % kbs) + unit16(lane >> 4, s);
    };
    auto narrow = [&](int e, int &row, int &k, int ns) {
        const int lane = e & 63, blk = e >> 6;
        row = 16 * (blk / ns) + unit16(lane >> 2 & 3, lane & 3);
        k = unit16(lane >> 4, blk % ns);
    };
    int r, k;
    if (idx < p.f_mid()) {
        narrow(idx - p.f_first(), r, k, p.nsi);
        if (r < width[1] && k < width[0]) v = theta[wo0 + r * width[0] + k];
    } else if (idx < p.f_last()) {
        wide(idx - p.f_mid(), r, k, p.TT);
        if (r < width[2] && k < width[1]) v = theta[wo1 + r * width[1] + k];
    } else if (idx < p.bias(0)) {
        wide(idx - p.f_last(), r, k, p.TT);
        if (r < n_last && k < h_last) v = theta[w_last + r * h_last + k];
    } else if (idx < p.b_top()) {
        const int e = idx - p.bias(0), l = e / (16 * p.TT), q = e - l * 16 * p.TT;
        const int u = (q & ~15) + unit16(q >> 2 & 3, q & 3);               // in the order of a lane's registers
        if (l == 2) v = q < n_last ? theta[b_last + q] : 0.0f;             // the action's bias in the third place, plain
        else if (l < last && u < width[l + 1]) v = theta[(l == 0 ? bo0 : bo1) + u];
    } else if (idx < p.b_mid()) {
        narrow(idx - p.b_top(), r, k, p.nsa);
        if (r < h_last && k < n_last) v = theta[w_last + k * h_last + r];
    } else if (idx < p.b_first()) {
        wide(idx - p.b_mid(), r, k, p.TT);
        if (r < width[1] && k < width[2]) v = theta[wo1 + k * width[1] + r];
    } else {
        wide(idx - p.b_first(), r, k, p.TT);
        if (r < width[0] && k < width[1]) v = theta[wo0 + k * width[0] + r];
    }
    a.dst[idx] = v;
}

inline pack16_args make_pack_args(const bagel_ctx *c)
{
    pack16_args a = {make_pack(c), {}, {}, {}, c->wpack16};
    for (int i = 0; i < 4; ++i) a.width[i] = c->width[i];
    for (int l = 0; l < 3; ++l) {
        a.w_off[l] = c->w_off[l];
        a.b_off[l] = c->b_off[l];
    }
    return a;
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

// (p[0] + .. + p[7]) + (p[8] + p[9] + ...): the order in which step_tail_kernel adds n group sums
template <class P>
__device__ __forceinline__ double sum_groups16(P p, int n, size_t stride)
{
    double s = 0.0, rest = 0.0;
    for (int c0 = 0; c0 < n; c0 += 8) {
        double v[8], t = 0.0;
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = c0 + u < n ? p[(size_t)(c0 + u) * stride] : 0.0;
        if (c0 > 0) t = rest;
#pragma unroll
        for (int u = 0; u < 8; ++u) t += v[u];
        if (c0 > 0) rest = t;
        else s = t;
    }
    return n > 8 ? s + rest : s;
}

// The ten wait states that the results of v_mfma_f32_16x16x4 want before anything but a matrix instruction reads them.  The compiler
// places them by itself, but counts wrongly where a result is used behind a branch and again where the branch joins: it takes the
// longer way round for both.  With two tiles the end of a slice below compiled into that: the last rows of the second tile were
// read four or five wait states after the instruction, and a backward sweep built that way gave other gradients from run to
// run.  tests/test_matrix_wait_states.py follows every path of the compiled kernels.  (No cost: 256-256, B = 1024, N = 2048
// 46.2 us per step with and without.)
__device__ __forceinline__ void matrix_results_ready(f4v &a, f4v &b) { asm volatile("s_nop 7\n\ts_nop 1" : "+v"(a), "+v"(b)); }

// One contraction over the blocks of a wide layer for the wave's NT tiles: w[t][kb] the weights, act the operands, n inputs,
// sl blocks per slice; slices are added up in order
template <int NT, int TT, int AS>
__device__ __forceinline__ void contract_wide(f4v (&z)[NT], const f4v (&w)[NT][TT], const float *act, int lane, int n, int sl)
{
    const float *x0 = act + (lane & 15) * AS + 4 * (lane >> 4);
    f4v acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) z[t] = acc[t] = f4v{0.0f, 0.0f, 0.0f, 0.0f};
    bool first = true;
    int left = sl;
#pragma unroll
    for (int kb = 0; kb < TT; ++kb)
        if (16 * kb < n) {
            const f4v x = *reinterpret_cast<const f4v *>(x0 + 16 * kb);
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int t = 0; t < NT; ++t) acc[t] = mfma16(w[t][kb][s], x[s], acc[t]);
            if constexpr (NT == 2) matrix_results_ready(acc[0], acc[1]);
            if (--left == 0 || 16 * (kb + 1) >= n) {                       // end of a slice (wave-uniform)
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    z[t] = first ? acc[t] : z[t] + acc[t];
                    acc[t] = f4v{0.0f, 0.0f, 0.0f, 0.0f};
                }
                first = false;
                left = sl;
            }
        }
}

// Slice `wave` (two blocks) of a contraction with one row tile: operands from act
template <int TT, int AS>
__device__ __forceinline__ f4v contract_slice(const f4v (&w)[2], const float *act, int wave, int lane)
{
    const float *x0 = act + (lane & 15) * AS + 4 * (lane >> 4) + 32 * wave;
    f4v acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const f4v x = *reinterpret_cast<const f4v *>(x0 + 16 * e);
#pragma unroll
        for (int s = 0; s < 4; ++s) acc = mfma16(w[e][s], x[s], acc);
    }
    return acc;
}

}  // namespace
