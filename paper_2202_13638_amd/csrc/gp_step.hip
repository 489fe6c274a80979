// One evaluation of every function sample at the current GP inputs:
//   f_sm(x) = phi_m(x)^T w_sm + k_m(x, X)^T v_sm      and, optionally, d f_sm / d x.
// This is the dominant kernel of a rollout step (Algorithm 1, the sampled transition).
//
// Mapping.  Lane = trajectory.  A wave holds 64 consecutive trajectories and one work unit:
// either CK training points or CL random features of one GP output m.  The operands that
// all trajectories share (scaled training inputs, frequencies) are read through
// wave-uniform addresses, so they travel through the scalar cache into SGPRs and feed the
// vector FMAs as scalar operands; the per-sample streams v and w are read as one float4
// (four consecutive points / features) per lane, coalesced across lanes.  The four waves
// of a workgroup take four consecutive units of the same output and kind for the same 64
// trajectories and add their sums through LDS in wave order; the workgroup writes one
// partial sum [1+D][B] per group of four units, and a later kernel adds the groups up in
// a fixed order, so results do not depend on scheduling.
//
// Arithmetic.  The kernel row is evaluated in float64: with noise variance far below the
// signal variance the representer weights v are large with alternating signs, the sum
// cancels by many orders of magnitude, and float32 rounding of each exp() alone would
// exceed the error budget of a rollout.  gfx950 issues float64 FMAs at the same rate as
// unpacked float32 FMAs, so this costs registers, not throughput.  In float64 the squared
// distance can be expanded, which turns  -1/2 |x - X_n|^2_Lambda  into one dot product
// against pre-scaled inputs plus two precomputed terms:
//   log2 k_mn(x) = q_m(x) + c_mn + sum_d x_d * Xs_mnd,
//   Xs_mnd = log2(e)/l_md^2 * X_nd,  c_mn = log2(alpha_m^2) - 1/2 sum_d Xs_mnd X_nd,
//   q_m(x) = -1/2 sum_d log2(e)/l_md^2 x_d^2.
// exp2 is evaluated in software (there is no float64 exp instruction): a polynomial form for any
// argument (exp2_poly), and a table form for the normal range that reads the split of the exponent
// straight off the bits of a sum (see gp_step_kernel).
// Jacobian: d k_mn / d x_d = ln2 * k_mn * (Xs_mnd - log2(e)/l_md^2 x_d); the kernel
// accumulates G_d = sum_n v_n k_n Xs_mnd and u = sum_n v_n k_n, the reduction finishes it.
//
// The random-feature phase is accumulated in float64 in revolutions, reduced exactly to
// [0, 1) and only then rounded to float32 for the hardware sin / cos (which take revolutions).
#include <stdlib.h>

#include <type_traits>

#include "bagel_internal.h"
#include "sample_math.h"

namespace {

#ifndef BAGEL_MIN_WAVES
#define BAGEL_MIN_WAVES(D) ((D) <= 8 ? 8 : ((D) <= 11 ? 5 : 4))
#endif
// Launches without the table form have at most four waves per SIMD.  The loops in pairs need more than the 128 registers of
// four from D = 6 on: held to them, D = 6 kept three in scratch memory (N = 512, L = 512, 100 trajectories: 8.8 us a launch,
// 8.5 with three waves; N = 2200, L = 1024, 200 trajectories: 11.8 and 11.6)
#define BAGEL_MIN_WAVES_SMALL(D) ((D) <= 5 ? 4 : 3)
#ifndef BAGEL_SAME_ROWS
#define BAGEL_SAME_ROWS 0      // timing experiment only: every work unit reads the first unit's rows
#endif

typedef float v4f __attribute__((ext_vector_type(4)));
typedef float f4v __attribute__((ext_vector_type(4)));

// The per-sample streams (v and w) are read through buffer loads: a wave-uniform descriptor of the
// work unit's rows, a wave-uniform row offset that the scalar unit advances, and a constant 32-bit
// byte offset per lane (the lane's sample).  The load instruction adds the three itself, so the loop
// spends no vector instruction on addresses.  Non-temporal: each float4 is read once per launch.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t stream_descriptor(const float4 *rows, size_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float4 *>(rows), 0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ v4f stream_load(__amdgpu_buffer_rsrc_t desc, unsigned lane_off, unsigned row_off)
{
    return __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(desc, lane_off, row_off, 2));
}

// End of a workgroup: waves 1-3 hand their sums (value u, Jacobian sums G) to wave 0 through LDS slots
// 0-2, wave 0 adds them in wave order and writes the group's partial sum.  in_lds: every wave, wave 0
// included (slot 3), has already stored its sums (the feature units of a Jacobian launch).  VALUE: with the value sum.
template <int D, bool JAC, int RC, bool VALUE = true>
__device__ __forceinline__ void combine_waves(double (*red)[RC][64], int wave, int lane, bool live, double *out, int B,
                                              bool in_lds, double u, double (&G)[D])
{
    if (wave > 0 && !in_lds) {
        red[wave - 1][0][lane] = u;
        if (JAC) {
#pragma unroll
            for (int d = 0; d < D; ++d) red[wave - 1][1 + d][lane] = G[d];
        }
    }
    __syncthreads();
    if (wave == 0) {
        if (in_lds) {
            if (VALUE) u = red[3][0][lane];
#pragma unroll
            for (int d = 0; d < D; ++d) G[d] = red[3][1 + d][lane];
        }
#pragma unroll
        for (int w = 0; w < 3; ++w) {
            if (VALUE) u += red[w][0][lane];
            if (JAC) {
#pragma unroll
                for (int d = 0; d < D; ++d) G[d] += red[w][1 + d][lane];
            }
        }
        if (live) {
            if (VALUE) out[0] = u;
            if (JAC) {
#pragma unroll
                for (int d = 0; d < D; ++d) out[(size_t)(1 + d) * B] = G[d];
            }
        }
    }
}

// ---- Jacobian sums of one step, added up --------------------------------------------------------
// J[m][d] = -amp_m (2 pi) sum_g Gr_g[d] + ln2 (sum_g Gk_g[d] - log2(e)/l_md^2 x_d sum_g u_g)   (groups in order)
// for the 64 trajectories of one tile, from the partial sums `part` of a sample evaluation at x; the
// result goes to a slot of the Jacobian tape, jdst[M][D][B] (float32).  Nothing on the critical path of
// a rollout needs J, so this runs as M extra rows of workgroups (one per output) inside the NEXT step's
// sample evaluation (or, after the last step, as a launch of its own).  256 threads: the four waves
// share the D entries of the output.  SPLIT: four entries to a workgroup, one a wave, ceil(D / 4) rows per output: in a small launch
// with many training points and few outputs a wave's trips to memory, one for every W groups of an entry (about 0.8 us each), are
// longer than the evaluation beside them.  us a step of a gradient call, unsplit and split: M = 2, D = 5, N = 3212, L = 4149,
// B = 96 23.2 -> 19.5, M = 3, D = 5, N = 6177, L = 439, B = 32 20.5 -> 17.0; 31 problems with D = 5 .. 8 and N >= 2048 1.07 times as fast.
struct jac_sums {
    const double *part;      // [groups][1+D][B]
    const double *x;         // [D][B] inputs the sums were evaluated at
    const double *A, *amp;   // [M][D], [M]
    float *jdst;             // [M][D][B]
};
// Several steps of a rollout at once: B inputs are those of B / trajectories steps, x is [D][x_stride], and the Jacobians go to
// [step][M][D][trajectories].  (An argument type of its own: with these two in every launch
// a call of bagel_sample_eval_static, N = 512, B = 256, took 18.53 us instead of 18.45.)
struct jac_sums_of_steps : jac_sums {
    int trajectories;
    size_t x_stride;
};
template <bool STEPS>
using jac_sums_arg = std::conditional_t<STEPS, jac_sums_of_steps, jac_sums>;

// W: loads in flight per sum (4 inside the large launches, which hide the trips and have few registers; 8 elsewhere)
template <int W, bool STEPS, bool SPLIT = false>
__device__ __forceinline__ void jacobian_tile(const jac_sums_arg<STEPS> &j, int tile, int row, int B, int D, int M, int ngk, int ngl)
{
    constexpr double LN2 = 0.69314718055994530942, TWO_PI = 6.28318530717958647693;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int b = tile * 64 + lane;
    if (b >= B) return;
    // (the same division signed and unsigned: with the other one D = 5 and D = 8 reserve scratch memory that no instruction uses)
    const int parts = SPLIT ? (D + 3) / 4 : 1, m = D == 8 ? row / parts : (int)((unsigned)row / (unsigned)parts), part = row - m * parts;
    int T = B;
    size_t x_stride = B, at = b;
    if constexpr (STEPS) {
        T = j.trajectories;
        x_stride = j.x_stride;
        at = (size_t)(b / T) * M * D * T + b % T;
    }
    const size_t stride = (size_t)(1 + D) * B;
    const double *pk = j.part + (size_t)(m * ngk) * stride + b;
    const double *pr = j.part + (size_t)(M * ngk + m * ngl) * stride + b;
    double u[1];
    if (W < 8) bagel_sums_in_order<1, W>({pk}, {ngk}, stride, u);      // (fewer registers: the value sum on its own first)
    for (int d = 4 * part + wave; d < D; d += SPLIT ? BAGEL_MAX_D : 4) {
        const double *const p[3] = {pk + (size_t)(1 + d) * B, pr + (size_t)(1 + d) * B, pk};
        const int n[3] = {ngk, ngl, ngk};
        const double xd = j.x[(size_t)d * x_stride + b];
        double s[3];
        if (W < 8) {
            double one[1];
            bagel_sums_in_order<1, W>({p[0]}, {ngk}, stride, one);
            s[0] = one[0];
            bagel_sums_in_order<1, W>({p[1]}, {ngl}, stride, one);
            s[1] = one[0];
            s[2] = u[0];
        } else {
            bagel_sums_in_order<3, W>(p, n, stride, s);
        }
        j.jdst[(size_t)(m * D + d) * T + at] = (float)(-j.amp[m] * TWO_PI * s[1] + LN2 * (s[0] - j.A[m * D + d] * xd * s[2]));
    }
}

constexpr bool split_jacobian(int D, bool jac, bool near, bool steps) { return D > 4 && jac && !near && !steps; }

template <bool STEPS>
__global__ __launch_bounds__(BAGEL_BLOCK) void jac_reduce_kernel(jac_sums_arg<STEPS> j, int B, int D, int M, int ngk, int ngl)
{
    jacobian_tile<8, STEPS>(j, blockIdx.x, blockIdx.y, B, D, M, ngk, ngl);
}

// ---- the loops of small launches ------------------------------------------------------------------
// A launch without the table form has at most four waves per SIMD, often one, and nothing else hides what a point
// waits for: its chain of dependent float64 operations (8 cycles each, where independent ones issue every 5),
// the trip of its operand row through the scalar cache, the stream.  So points (features) are worked on in pairs,
// rows are requested a pair ahead, the stream four float4 ahead (into the registers just used: CK and CL are
// multiples of 16).  Every sum keeps the order of the
// point-by-point loops.  A launch at N = 2200, L = 1024, 100 trajectories, D = 3 takes 9.1 -> 7.8 us, at N = 512, L = 1024, 256
// trajectories, D = 5 6.4 -> 5.9 us.  For D > 8 two pairs of rows do not fit the scalar registers: those stay with
// the point-by-point loops.
//
// What a wave then still waits for is the order of its loads.  Scalar loads return in any order, so a wait for one is a wait for
// all: the rows of this pair are waited for (rows_arrived) before those of the next are requested, not after.  Vector loads
// return in order, so the matrix-core operands, which hit in cache, come after the stream's float4 requested before them:
// they are requested three float4 ahead, behind a request that has had as long.  Us a launch, before -> now, evaluations alone in a loop: M = 4,
// D = 5, N = L = 2048, B = 1024 18.6 -> 17.6 (its 67 MB of streams alone take 11.5), M = 6, D = 8, N = 1533, L = 901, B = 777 21.6 -> 20.1; 56 shapes of
// D = 2 .. 8, values alone and with the Jacobian, 1.06 on average, least at N = L = 2048, B = 1024 (values at D = 2 5.1 -> 5.3 and D = 4 8.4 -> 8.6,
// D = 7 25.0 -> 25.6).  Between two ends of step of a rollout: the first of these 17.7 -> 17.3, M = 3, N = 1533, L = 901, B = 777 10.0 -> 9.3.
__device__ __forceinline__ void rows_arrived()
{
    __builtin_amdgcn_s_waitcnt(0xc07f);        // lgkmcnt(0) alone
    __builtin_amdgcn_sched_barrier(0);
}

template <int D>
__device__ __forceinline__ void load_row(double (&r)[D + 1], const double *__restrict__ src)
{
#pragma unroll
    for (int d = 0; d <= D; ++d) r[d] = src[d];
}

// n_iter float4 of training points (a multiple of 4) with rows from Xr and the stream vdesc: see the general loop
template <int D, bool JAC>
__device__ __forceinline__ void kernel_row_pairs(const double *__restrict__ Xr, __amdgpu_buffer_rsrc_t vdesc, unsigned voff,
                                                 unsigned vstep, int n_iter, const double (&xs)[D], double qs, double &u, double (&G)[D])
{
    exp2_coefficients ec;
    asm volatile("" : "+s"(ec.c7), "+v"(ec.c6));
    const int last = n_iter - 1;
    auto pair = [&](const double (&r0)[D + 1], const double (&r1)[D + 1], double (&n0)[D + 1], double (&n1)[D + 1],
                    const double *__restrict__ next, float v0, float v1) {
        rows_arrived();
        load_row<D>(n0, next);
        load_row<D>(n1, next + (D + 1));
        __builtin_amdgcn_sched_barrier(0);
        double t0 = qs + r0[D], t1 = qs + r1[D];
#pragma unroll
        for (int d = 0; d < D; ++d) {
            t0 = fma(xs[d], r0[d], t0);
            t1 = fma(xs[d], r1[d], t1);
        }
        double k0, k1;
        exp2_poly2(t0, t1, ec, k0, k1);
        const double vk0 = (double)v0 * k0, vk1 = (double)v1 * k1;
        u += vk0;
        u += vk1;
        if (JAC) {
#pragma unroll
            for (int d = 0; d < D; ++d) G[d] = fma(vk0, r0[d], G[d]);
#pragma unroll
            for (int d = 0; d < D; ++d) G[d] = fma(vk1, r1[d], G[d]);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    v4f vb[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) vb[i] = stream_load(vdesc, voff, (unsigned)i * vstep);
    double a0[D + 1], a1[D + 1], b0[D + 1], b1[D + 1];
    load_row<D>(a0, Xr);
    load_row<D>(a1, Xr + (D + 1));
    for (int n4 = 0; n4 < n_iter; n4 += 4) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const double *__restrict__ r = Xr + (size_t)((n4 + i) * 4) * (D + 1);
            pair(a0, a1, b0, b1, r + 2 * (D + 1), vb[i].x, vb[i].y);
            pair(b0, b1, a0, a1, n4 + i < last ? r + 4 * (D + 1) : Xr, vb[i].z, vb[i].w);
            vb[i] = stream_load(vdesc, voff, (unsigned)(n4 + 4 + i < last ? n4 + 4 + i : last) * vstep);
        }
    }
}

// A feature unit adds up its features in float32, in one chain per sum, and the units' sums are added up in float64.  The error of a
// chain grows as the square root of its length, so where units are longer for speed alone (bagel_ctx::feature_chains) a chain ends, and its
// sum goes to float64, every 32 features.  (Error of f and its Jacobian against 64 bits, D = 8, L = 4096, units of 128: 2.4e-7 and 2.3e-7 in
// one chain a unit, 1.4e-7 and 1.5e-7 in chains of 32, as with units of 32; a step of a gradient call, M = 4, D = 5, N = 1024, B = 1500 44.9 and
// 45.7 us, 50.6 with units of 32.  CHAINS instances of the kernel, so that the launches without them keep their code.)
constexpr int CHAIN = 32 / 4;                // float4

// n_iter float4 of random features (a multiple of 4): see the feature loops of the kernel.  Without VALUE the Jacobian sums
// alone: the steps of a rollout by rollout.hip have their values, and the cosines are a sixth of the work (100 steps, B = 256,
// N = 512, L = 1024, D = 5: 133.9 us a launch without, 139.6 with them).
template <int D, bool JAC, bool VALUE, bool CHAINS, class F>
__device__ __forceinline__ void feature_pairs(const double *__restrict__ Or, __amdgpu_buffer_rsrc_t wdesc, unsigned woff, unsigned wstep,
                                              __amdgpu_buffer_rsrc_t odesc, unsigned ooff, unsigned ostep, int n_iter,
                                              const double (&x)[D], float &p, f4v (&acc)[(D + 3) / 4], F end_chain)
{
    constexpr int NQ = (D + 3) / 4;
    const int last = n_iter - 1;
    auto pair = [&](const double (&r0)[D + 1], const double (&r1)[D + 1], double (&n0)[D + 1], double (&n1)[D + 1],
                    const double *__restrict__ next, float w0, float w1, const v4f (&bq)[NQ], int j) {
        rows_arrived();
        load_row<D>(n0, next);
        load_row<D>(n1, next + (D + 1));
        __builtin_amdgcn_sched_barrier(0);
        double z0 = x[0] * r0[0], z1 = x[0] * r1[0];
#pragma unroll
        for (int d = 1; d < D; ++d) {
            z0 = fma(x[d], r0[d], z0);
            z1 = fma(x[d], r1[d], z1);
        }
        z0 += r0[D];
        z1 += r1[D];
        const float y0 = (float)__builtin_amdgcn_fract(z0), y1 = (float)__builtin_amdgcn_fract(z1);
        if (VALUE) {
            p = fmaf(w0, __builtin_amdgcn_cosf(y0), p);
            p = fmaf(w1, __builtin_amdgcn_cosf(y1), p);
        }
        if (JAC) {
            const float s0 = w0 * __builtin_amdgcn_sinf(y0), s1 = w1 * __builtin_amdgcn_sinf(y1);
#pragma unroll
            for (int qd = 0; qd < NQ; ++qd) acc[qd] = __builtin_amdgcn_mfma_f32_4x4x1f32(s0, bq[qd][j], acc[qd], 0, 0, 0);
#pragma unroll
            for (int qd = 0; qd < NQ; ++qd) acc[qd] = __builtin_amdgcn_mfma_f32_4x4x1f32(s1, bq[qd][j + 1], acc[qd], 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    v4f wb[4], bq[4][NQ];
    auto operands = [&](v4f (&b)[NQ], int l4) {
        if (JAC) {
#pragma unroll
            for (int qd = 0; qd < NQ; ++qd)
                b[qd] = __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(odesc, ooff + 16u * qd, (unsigned)l4 * ostep, 0));
        }
    };
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        wb[i] = stream_load(wdesc, woff, (unsigned)i * wstep);
        if (i < 3) operands(bq[i], i);
    }
    double a0[D + 1], a1[D + 1], b0[D + 1], b1[D + 1];
    load_row<D>(a0, Or);
    load_row<D>(a1, Or + (D + 1));
    for (int l4 = 0; l4 < n_iter; l4 += 4) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const double *__restrict__ r = Or + (size_t)((l4 + i) * 4) * (D + 1);
            operands(bq[(i + 3) & 3], l4 + i + 3 < last ? l4 + i + 3 : last);
            pair(a0, a1, b0, b1, r + 2 * (D + 1), wb[i].x, wb[i].y, bq[i], 0);
            pair(b0, b1, a0, a1, l4 + i < last ? r + 4 * (D + 1) : Or, wb[i].z, wb[i].w, bq[i], 2);
            wb[i] = stream_load(wdesc, woff, (unsigned)(l4 + 4 + i < last ? l4 + 4 + i : last) * wstep);
        }
        if (CHAINS && (l4 + 4) % CHAIN == 0 && l4 + 4 < n_iter) end_chain();
    }
}

// NEAR adds the fast form of the kernel-row loop for the normal case that data and trajectory are
// within about 19 length scales of the origin; the loop above is then the fallback of a wave that
// holds a trajectory further out, or of a model with training points further out (near_ok == 0).
// With  q = -1/2 sum_d a_d x_d^2  taken out of the exponent (the sums are multiplied by 2^q at the end),
//   t'_n = c_n + sum_d x_d Xs_nd   lies in [-770, 270]   for |q|, |c_n| <= 250 and |log2 alpha^2| <= 20,
// and the near table holds c_n + 6144 in place of c_n: 6144 = 1.5 * 2^12 puts the sum s = t'_n + 6144 into
// [2^12, 2^13), where one unit in the last place is 2^-40, so the bits of s ARE the split of t'_n:
//   high word bits 19..8 = 2048 + floor(t'), bits 7..0 = the next eight bits i (t' in units of 1/256),
//   low word = the remaining fraction g in units of 2^-40 (t' rounded to 2^-41: relative error 3e-13 of k).
// Then 2^t' = 2^floor(t') * 2^(i/256) * 2^g: the middle factor comes from a 256-entry table in LDS,
// indexed by the low byte of the high word; 2^g is a degree-3 polynomial in the low word converted to
// float64 (coefficients pre-scaled by 2^-40k; relative error 7e-14 on [0, 2^-8)); and the power of two is
// applied by adding the high word of s, shifted left by 12, to the high word of the table entry: the
// shift drops the exponent of s and leaves (2048 + floor t') << 20 | i << 12, so the table stores
// 2^(i/256) with i << 12 subtracted from its high word and its sign bit set (adding 2048 << 20 clears
// it again).  No exponent can wrap for t' in the range above.  Per training point: 9 instructions for s,
// 7 for k (address, conversion, 3 polynomial steps, exponent add, product), 2 for v k, 9 to accumulate
// = 27, against 32 of the general loop.
// The table form needs many workgroups per compute unit to pay: its LDS read shares a wait counter
// with the scalar loads of the shared operands, so every look-up also waits for the operand rows
// requested ahead; small launches take the general loop only.
template <int D, bool JAC, bool NEAR, bool STEPS, bool CHAINS>
__global__ __launch_bounds__(BAGEL_BLOCK) __attribute__((amdgpu_waves_per_eu(NEAR ? BAGEL_MIN_WAVES(D) : BAGEL_MIN_WAVES_SMALL(D), 8))) void gp_step_kernel(
    const double *__restrict__ Xs, const double *__restrict__ Xn, const double *__restrict__ Os,
    const float4 *__restrict__ Of, const double *__restrict__ A, const float4 *__restrict__ v4,
    const float4 *__restrict__ w4,
    const double *__restrict__ xbuf, double *__restrict__ part, const double *__restrict__ exp_tab,
    const int *__restrict__ near_ok, int B, int S, int per_sample, int Np, int Lp, int CK, int CL, int nck, int ncl,
    int M, jac_sums_arg<STEPS> prev)
{
    // Rows of workgroups past the work units: the previous step's Jacobian sums (see jacobian_tile).
    // (Placed first in the grid instead, they made the launch slower: 571 vs 556 us.)
    constexpr bool SPLIT = split_jacobian(D, JAC, NEAR, STEPS);
    if ((int)blockIdx.y >= M * (((nck + 3) >> 2) + ((ncl + 3) >> 2))) {
        jacobian_tile<NEAR ? 4 : 8, false, SPLIT>(prev, blockIdx.x, (int)blockIdx.y - M * (((nck + 3) >> 2) + ((ncl + 3) >> 2)), B, D, M,
                      (nck + 3) >> 2, (ncl + 3) >> 2);
        return;
    }
    // Sums handed from wave to wave at the end.  Slot 3 is used only by the feature units of a
    // Jacobian launch; the kernel-row units keep the table of the table form there.
    constexpr int RC = 1 + D > 4 ? 1 + D : 4;      // rows per slot: at least the 256 entries of the exp2 table
    __shared__ double red[4][RC][64];
    double *tab = &red[3][0][0];
    constexpr int NQ = (D + 3) / 4;                // matrix instructions per feature: four Jacobian columns each
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int b_raw = blockIdx.x * 64 + lane;
    const bool live = b_raw < B;
    const int b = live ? b_raw : B - 1;
    int trajectory = b;
    size_t x_stride = B;
    if constexpr (STEPS) {
        trajectory = b % prev.trajectories;
        x_stride = prev.x_stride;
    }
    const int sidx = trajectory / per_sample;
    const int group = blockIdx.y;                  // four consecutive units of one output and kind
    const int ngk = (nck + 3) >> 2, ngl = (ncl + 3) >> 2;

    double x[D];
#pragma unroll
    for (int d = 0; d < D; ++d) x[d] = xbuf[d * x_stride + b];

    double *out = part + (size_t)group * (1 + D) * B + b;

    if (group < M * ngk) {
        double u = 0.0;                            // this wave's sums: value, then the D Jacobian sums
        double G[D];
#pragma unroll
        for (int d = 0; d < D; ++d) G[d] = 0.0;
        // ---------------- kernel-row unit: CK training points of output m ----------------
        const int m = group / ngk, c = 4 * (group - m * ngk) + wave;
        const int n_iter = c < nck ? CK / 4 : 0;   // a wave past the last chunk adds nothing
        if (NEAR) {
            static_assert(BAGEL_BLOCK == 256, "one table entry per thread");
            tab[threadIdx.x] = exp_tab[threadIdx.x];
            __syncthreads();
        }
        double q = 0.0;
#pragma unroll
        for (int d = 0; d < D; ++d) q = fma(-0.5 * A[m * D + d] * x[d], x[d], q);
        const size_t row0 = BAGEL_SAME_ROWS ? 0 : ((size_t)m * Np + (size_t)c * CK) * (D + 1);
        // the stream of this unit for this lane's sample: uniform base address plus a 32-bit lane offset
        const unsigned vstep = (unsigned)S * (unsigned)sizeof(float4);       // one row: four points of every sample
        const float4 *vrows = v4 + ((size_t)m * (Np / 4) + (size_t)c * (CK / 4)) * S;
        const unsigned voff = (unsigned)sidx * (unsigned)sizeof(float4);
        bool wave_near = false;
        if (NEAR) wave_near = near_ok[0] != 0 && !__any(!(q >= -250.0));
        // (Each of the two loops builds the stream's descriptor for itself, from a base pointer the
        // compiler cannot identify with the other loop's: one shared descriptor would live across both
        // loops, and the scalar-register pressure of the general loop would then spill it inside the
        // table loop too - eleven extra vector instructions per eight points.)
        if (NEAR && wave_near) {
            const float4 *vrows_t = vrows;
            asm volatile("" : "+s"(vrows_t));
            const __amdgpu_buffer_rsrc_t vdesc = stream_descriptor(vrows_t, (size_t)(CK / 4) * vstep);
            const double *__restrict__ Xr = Xn + row0;
            const int last = n_iter - 1;
            // leading polynomial coefficients pinned to register classes: the first Horner step is then a
            // single three-operand FMA (an FMA takes at most one scalar operand)
            double ca = 0x1.c726cfe5bfc26p-125, cb = 0x1.ebfbd4e173a43p-83;
            asm volatile("" : "+s"(ca), "+v"(cb));
            {
                // One training point with its row in rc; the next point's row is requested into rn right at
                // the start, so that its trip through the scalar cache overlaps this point's arithmetic and
                // table look-up instead of preceding the next point's.
                auto one_point = [&](const double (&rc)[D + 1], double (&rn)[D + 1], const double *__restrict__ next,
                                     float vf) {
#pragma unroll
                    for (int d = 0; d <= D; ++d) rn[d] = next[d];
                    __builtin_amdgcn_sched_barrier(0);
                    double t = x[0] * rc[0];
#pragma unroll
                    for (int d = 1; d < D; ++d) t = fma(x[d], rc[d], t);
                    const double s = t + rc[D];
                    const int hs = __double2hiint(s);
                    const double T = tab[hs & 255];
                    const double g = (double)(unsigned)__double2loint(s);
                    double p = fma(ca, g, cb);
                    p = fma(p, g, 0x1.62e42fefcb0c8p-41);
                    p = fma(p, g, 1.0);
                    const double sc = __hiloint2double(__double2hiint(T) + (hs << 12), __double2loint(T));
                    const double vk = (double)vf * (sc * p);
                    u += vk;
                    if (JAC) {
#pragma unroll
                        for (int d = 0; d < D; ++d) G[d] = fma(vk, rc[d], G[d]);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                };
                double ra[D + 1], rb[D + 1];
#pragma unroll
                for (int d = 0; d <= D; ++d) ra[d] = Xr[d];
                // rows follow each other in memory; the request past the unit's last row reads the first
                // row of the next unit or, after the very last one, stays inside the table (see below)
                auto four_points = [&](const v4f vv, int n4) {
                    const double *__restrict__ r = Xr + (size_t)(n4 * 4) * (D + 1);
                    one_point(ra, rb, r + 1 * (D + 1), vv.x);
                    one_point(rb, ra, r + 2 * (D + 1), vv.y);
                    one_point(ra, rb, r + 3 * (D + 1), vv.z);
                    one_point(rb, ra, n4 < last ? r + 4 * (D + 1) : Xr, vv.w);
                };
                // The stream is requested one float4 ahead, alternating between two register sets (a request
                // past the end repeats the last row): HBM latency under load is several times a wave's own
                // work on four points, and the loop was idle waiting for it.
                // (CK is a multiple of 16: the loop body handles two float4 without a branch, which keeps
                // the compiler from moving a request down to its use.)
                v4f va = stream_load(vdesc, voff, 0u);
                for (int n4 = 0; n4 < n_iter; n4 += 2) {
                    const v4f vb = stream_load(vdesc, voff, (unsigned)(n4 + 1) * vstep);
                    four_points(va, n4);
                    va = stream_load(vdesc, voff, (unsigned)(n4 + 2 < last ? n4 + 2 : last) * vstep);
                    four_points(vb, n4 + 1);
                }
            }
            // 2^q (q in [-250, 0]) by the loop's own table form: it needs no constants beyond the loop's,
            // whereas the polynomial form's seven would be kept in scalar registers across the loop
            // (shared with the general loop below) and push the loop's operands out into spill lanes
            const double sq = q + 6144.0;
            const int hq = __double2hiint(sq);
            const double Tq = tab[hq & 255];
            const double gq = (double)(unsigned)__double2loint(sq);
            double pq = fma(ca, gq, cb);
            pq = fma(pq, gq, 0x1.62e42fefcb0c8p-41);
            pq = fma(pq, gq, 1.0);
            const double eq = pq * __hiloint2double(__double2hiint(Tq) + (hq << 12), __double2loint(Tq));
            u *= eq;
            if (JAC) {
#pragma unroll
                for (int d = 0; d < D; ++d) G[d] *= eq;
            }
        } else {
            // A trajectory further out than about 400 length scales (q < -2^17) is that far from every
            // training point that is kept (model set-up turns rows with c_n < -2^17 into padding), and its
            // kernel row is zero: it gets a constant exponent of -3000.
            const float4 *vrows_g = vrows;
            asm volatile("" : "+s"(vrows_g));
            const __amdgpu_buffer_rsrc_t vdesc = stream_descriptor(vrows_g, (size_t)(CK / 4) * vstep);
            const bool far = q < -131072.0;
            double xs[D];
#pragma unroll
            for (int d = 0; d < D; ++d) xs[d] = far ? 0.0 : x[d];
            const double qs = far ? -3000.0 : q;
            const double *__restrict__ Xr = Xs + row0;
            if constexpr (!NEAR && D <= 8) {
                if (n_iter > 0) kernel_row_pairs<D, JAC>(Xr, vdesc, voff, vstep, n_iter, xs, qs, u, G);
            } else {
                exp2_coefficients ec;
                asm volatile("" : "+s"(ec.c7), "+v"(ec.c6));
                // same pipeline as the table form: the next point's row is requested while this one is worked
                // on, the stream one float4 ahead
                const int last = n_iter - 1;
                auto one_point = [&](const double (&rc)[D + 1], double (&rn)[D + 1], const double *__restrict__ next,
                                     float vf) {
    #pragma unroll
                    for (int d = 0; d <= D; ++d) rn[d] = next[d];
                    __builtin_amdgcn_sched_barrier(0);
                    double t = qs + rc[D];
    #pragma unroll
                    for (int d = 0; d < D; ++d) t = fma(xs[d], rc[d], t);
                    const double k = exp2_poly(t, ec);
                    const double vk = (double)vf * k;
                    u += vk;
                    if (JAC) {
    #pragma unroll
                        for (int d = 0; d < D; ++d) G[d] = fma(vk, rc[d], G[d]);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                };
                double ra[D + 1], rb[D + 1];
    #pragma unroll
                for (int d = 0; d <= D; ++d) ra[d] = Xr[d];
                auto four_points = [&](const v4f vv, int n4) {
                    const double *__restrict__ r = Xr + (size_t)(n4 * 4) * (D + 1);
                    one_point(ra, rb, r + 1 * (D + 1), vv.x);
                    one_point(rb, ra, r + 2 * (D + 1), vv.y);
                    one_point(ra, rb, r + 3 * (D + 1), vv.z);
                    one_point(rb, ra, n4 < last ? r + 4 * (D + 1) : Xr, vv.w);
                };
                v4f va = stream_load(vdesc, voff, 0u);
                for (int n4 = 0; n4 < n_iter; n4 += 2) {
                    const v4f vb = stream_load(vdesc, voff, (unsigned)(n4 + 1) * vstep);
                    four_points(va, n4);
                    va = stream_load(vdesc, voff, (unsigned)(n4 + 2 < last ? n4 + 2 : last) * vstep);
                    four_points(vb, n4 + 1);
                }
            }
        }
        combine_waves<D, JAC, RC>(red, wave, lane, live, out, B, false, u, G);
    } else {
        // ---------------- random-feature unit: CL features of output m -------------------
        const int gg = group - M * ngk;
        const int m = gg / ngl, c = 4 * (gg - m * ngl) + wave;
        const int n_iter = c < ncl ? CL / 4 : 0;
        const double *__restrict__ Or = Os + (BAGEL_SAME_ROWS ? 0 : ((size_t)m * Lp + (size_t)c * CL) * (D + 1));
        const unsigned wstep = (unsigned)S * (unsigned)sizeof(float4);
        const __amdgpu_buffer_rsrc_t wdesc =
            stream_descriptor(w4 + ((size_t)m * (Lp / 4) + (size_t)c * (CL / 4)) * S, (size_t)(CL / 4) * wstep);
        const unsigned woff = (unsigned)sidx * (unsigned)sizeof(float4);
        float p = 0.0f;
        double p_chains = 0.0;                     // of the chains that have ended (CHAINS)
        if (JAC) {
            // The Jacobian sums of the feature part, G[b][d] = sum_l (w_l sin z_l) omega_ld, tolerate
            // float32 (no cancellation: w has random signs), so they run on the matrix cores as rank-1
            // updates: v_mfma_f32_4x4x1 (16 blocks) multiplies, within every group of four lanes, the A
            // values of the four lanes (here: w sin z of four trajectories) with the B values of the four
            // lanes (here: omega_ld for d = 4 q + lane % 4) and adds the 4 x 4 products to four registers
            // (register i of lane 4 g + j: trajectory 4 g + i, column 4 q + j).  One instruction takes the
            // issue time of two vector FMAs and replaces four of them (and the float64 conversion).
            // Of holds omega / (2 pi) in float32 in the order the B operand needs: per four features and
            // lane class j, NQ float4 (feature 0..3 of column 4 q + j), read through a buffer load whose
            // lane offset is constant; columns >= D are zero.
            const unsigned ostep = 64u * NQ;            // bytes per four features
            const __amdgpu_buffer_rsrc_t odesc = __builtin_amdgcn_make_buffer_rsrc(
                const_cast<float4 *>(Of + ((size_t)m * (Lp / 4) + (size_t)c * (CL / 4)) * 4 * NQ), 0,
                (int)((size_t)(CL / 4) * ostep), 0x00020000);
            const unsigned ooff = (unsigned)(lane & 3) * (16u * NQ);
            f4v acc[NQ];
#pragma unroll
            for (int qd = 0; qd < NQ; ++qd) acc[qd] = f4v{0.0f, 0.0f, 0.0f, 0.0f};
            // the wave's sums so far in float64, where the end of the unit hands them over
            auto add_to_lds = [&](bool first) {
#pragma unroll
                for (int qd = 0; qd < NQ; ++qd) {
                    const int d = 4 * qd + (lane & 3);
                    if (d < D) {
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            double &sum = red[((threadIdx.x >> 6) + 3) & 3][1 + d][(lane & ~3) + i];
                            sum = first ? 0.0 : sum + (double)acc[qd][i];
                        }
                    }
                }
            };
            auto end_chain = [&]() {
                p_chains += (double)p;
                p = 0.0f;
                add_to_lds(false);
#pragma unroll
                for (int qd = 0; qd < NQ; ++qd) acc[qd] = f4v{0.0f, 0.0f, 0.0f, 0.0f};
            };
            if (CHAINS) add_to_lds(true);
            if constexpr (!NEAR && D <= 8) {
                if constexpr (CHAINS) {
                    if (n_iter > 0) feature_pairs<D, true, true, true>(Or, wdesc, woff, wstep, odesc, ooff, ostep, n_iter, x, p, acc, end_chain);
                } else {
                    if (n_iter > 0) feature_pairs<D, true, !STEPS, false>(Or, wdesc, woff, wstep, odesc, ooff, ostep, n_iter, x, p, acc, [] {});
                }
            } else {
                const int last = n_iter - 1;         // CL is a multiple of 16: two float4 per trip, no branch
                auto one_feature = [&](const double (&rc)[D + 1], double (&rn)[D + 1], const double *__restrict__ next,
                                       float wf, const v4f (&bq)[NQ], int j) {
#pragma unroll
                    for (int d = 0; d <= D; ++d) rn[d] = next[d];
                    __builtin_amdgcn_sched_barrier(0);
                    // product first, phase offset last: both are scalar operands, and an FMA takes only one
                    double z = x[0] * rc[0];
#pragma unroll
                    for (int d = 1; d < D; ++d) z = fma(x[d], rc[d], z);
                    z += rc[D];
                    // z is the phase in revolutions; its fractional part is exact in float64 and the
                    // hardware sin / cos take revolutions (absolute error about one float32 ulp)
                    const float y = (float)__builtin_amdgcn_fract(z);
                    const float sn = __builtin_amdgcn_sinf(y);
                    const float cs = __builtin_amdgcn_cosf(y);
                    p = fmaf(wf, cs, p);
                    const float ws = wf * sn;
#pragma unroll
                    for (int qd = 0; qd < NQ; ++qd)
                        acc[qd] = __builtin_amdgcn_mfma_f32_4x4x1f32(ws, bq[qd][j], acc[qd], 0, 0, 0);
                    __builtin_amdgcn_sched_barrier(0);
                };
                double fa[D + 1], fb[D + 1];
#pragma unroll
                for (int d = 0; d <= D; ++d) fa[d] = Or[d];
                // four features whose weights are in ww; `next` receives the stream's float4 of step l4_next,
                // requested after this step's B operands (loads return in order: the wait for the operands,
                // which hit in cache, must not include the stream's trip to HBM)
                auto four_features = [&](const v4f ww, int l4, v4f &next, int l4_next) {
                    v4f bq[NQ];
#pragma unroll
                    for (int qd = 0; qd < NQ; ++qd)
                        bq[qd] = __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(odesc, ooff + 16u * qd, (unsigned)l4 * ostep, 0));
                    __builtin_amdgcn_sched_barrier(0);
                    next = stream_load(wdesc, woff, (unsigned)l4_next * wstep);
                    __builtin_amdgcn_sched_barrier(0);
                    // each feature's row was requested while the previous feature was being worked on (see the
                    // kernel-row loop); the request after the unit's last row stays inside the table
                    const double *__restrict__ r = Or + (size_t)(l4 * 4) * (D + 1);
                    one_feature(fa, fb, r + 1 * (D + 1), ww.x, bq, 0);
                    one_feature(fb, fa, r + 2 * (D + 1), ww.y, bq, 1);
                    one_feature(fa, fb, r + 3 * (D + 1), ww.z, bq, 2);
                    one_feature(fb, fa, l4 < last ? r + 4 * (D + 1) : Or, ww.w, bq, 3);
                };
                // the stream of w one float4 ahead in alternating register sets, as in the kernel-row loop
                v4f wa = stream_load(wdesc, woff, 0u), wb = wa;
                for (int l4 = 0; l4 < n_iter; l4 += 2) {
                    four_features(wa, l4, wb, l4 + 1);
                    four_features(wb, l4 + 1, wa, l4 + 2 < last ? l4 + 2 : last);
                    // (D = 16 without the table form, every eight features: a condition takes scalar registers that the rows leave no room for)
                    if (CHAINS && ((D == 16 && !NEAR) || ((l4 + 2) % CHAIN == 0 && l4 + 2 < n_iter))) end_chain();
                }
            }
            // every wave, wave 0 included, hands its sums over through LDS: that is also the transposition
            // from the accumulator layout (lane = column, register = trajectory) to lane = trajectory
            const int slot = (wave + 3) & 3;
            if (!STEPS) red[slot][0][lane] = CHAINS ? p_chains + (double)p : (double)p;
            if constexpr (CHAINS) {
                add_to_lds(false);
            } else {
#pragma unroll
                for (int qd = 0; qd < NQ; ++qd) {
                    const int d = 4 * qd + (lane & 3);
                    if (d < D) {
#pragma unroll
                        for (int i = 0; i < 4; ++i) red[slot][1 + d][(lane & ~3) + i] = (double)acc[qd][i];
                    }
                }
            }
            double u = 0.0, G[D];
            combine_waves<D, JAC, RC, !STEPS>(red, wave, lane, live, out, B, true, u, G);
        } else {
            auto end_chain = [&]() {
                p_chains += (double)p;
                p = 0.0f;
            };
            if constexpr (!NEAR && D <= 8) {
                f4v none[NQ];
                if (n_iter > 0) feature_pairs<D, false, true, CHAINS>(Or, wdesc, woff, wstep, wdesc, 0u, 0u, n_iter, x, p, none, end_chain);
            } else {
                // value only: the same pipeline without the Jacobian sums
                const int last = n_iter - 1;
                auto one_feature = [&](const double (&rc)[D + 1], double (&rn)[D + 1], const double *__restrict__ next,
                                       float wf) {
#pragma unroll
                    for (int d = 0; d <= D; ++d) rn[d] = next[d];
                    __builtin_amdgcn_sched_barrier(0);
                    double z = x[0] * rc[0];
#pragma unroll
                    for (int d = 1; d < D; ++d) z = fma(x[d], rc[d], z);
                    z += rc[D];
                    const float y = (float)__builtin_amdgcn_fract(z);
                    p = fmaf(wf, __builtin_amdgcn_cosf(y), p);
                    __builtin_amdgcn_sched_barrier(0);
                };
                double fa[D + 1], fb[D + 1];
#pragma unroll
                for (int d = 0; d <= D; ++d) fa[d] = Or[d];
                auto four_features = [&](const v4f ww, int l4) {
                    const double *__restrict__ r = Or + (size_t)(l4 * 4) * (D + 1);
                    one_feature(fa, fb, r + 1 * (D + 1), ww.x);
                    one_feature(fb, fa, r + 2 * (D + 1), ww.y);
                    one_feature(fa, fb, r + 3 * (D + 1), ww.z);
                    one_feature(fb, fa, l4 < last ? r + 4 * (D + 1) : Or, ww.w);
                };
                v4f wa = stream_load(wdesc, woff, 0u);
                for (int l4 = 0; l4 < n_iter; l4 += 2) {
                    const v4f wb = stream_load(wdesc, woff, (unsigned)(l4 + 1) * wstep);
                    four_features(wa, l4);
                    wa = stream_load(wdesc, woff, (unsigned)(l4 + 2 < last ? l4 + 2 : last) * wstep);
                    four_features(wb, l4 + 1);
                    if (CHAINS && (l4 + 2) % CHAIN == 0 && l4 + 2 < n_iter) end_chain();
                }
            }
            double u = CHAINS ? p_chains + (double)p : (double)p, G[D];
            combine_waves<D, JAC, RC>(red, wave, lane, live, out, B, false, u, G);
        }
    }
}

template <int D, bool JAC, bool NEAR, bool CHAINS>
void launch_variant(bagel_ctx *c, float *prev_jac)
{
    dim3 grid((c->dm.B + 63) / 64, c->groups + (prev_jac ? c->M * (split_jacobian(D, JAC, NEAR, false) ? (D + 3) / 4 : 1) : 0));
    const int per_sample = c->dm.B / c->dm.S;
    const jac_sums prev = {c->part_alt, c->xbuf_alt, c->A, c->amp, prev_jac};
    hipLaunchKernelGGL((gp_step_kernel<D, JAC, NEAR, false, CHAINS>), grid, dim3(BAGEL_BLOCK), 0, c->stream, c->Xs, c->Xn, c->Os,
                       reinterpret_cast<const float4 *>(c->Of), c->A, c->v4, c->w4, c->xbuf, c->part, c->exp_tab,
                       c->near_ok, c->dm.B, c->dm.S, per_sample, c->Np, c->Lp, c->CK, c->CL, c->nck, c->ncl, c->M, prev);
}

template <int D, bool JAC>
void launch_variant(bagel_ctx *c, float *prev_jac)
{
    if (c->exp_table) {
        if (c->feature_chains) launch_variant<D, JAC, true, true>(c, prev_jac);
        else launch_variant<D, JAC, true, false>(c, prev_jac);
    } else {
        if (c->feature_chains) launch_variant<D, JAC, false, true>(c, prev_jac);
        else launch_variant<D, JAC, false, false>(c, prev_jac);
    }
}

template <int D>
hipError_t launch_d(bagel_ctx *c, bool jac, float *prev_jac)
{
    if (jac) launch_variant<D, true>(c, prev_jac);
    else launch_variant<D, false>(c, prev_jac);
    return hipGetLastError();
}

// The Jacobians of the steps t0 .. t0 + steps - 1 of a rollout by rollout.hip (the same loops as step by step: the same bits)
template <int D>
hipError_t launch_steps(bagel_ctx *c, int t0, int steps)
{
    const int B = c->dm.B, n = steps * B;
    const jac_sums_of_steps j = {{c->part_all, c->xall + (size_t)t0 * B, c->A, c->amp, c->tape_J + (size_t)t0 * c->M * c->D * B}, B, (size_t)c->dm.H * B};
    hipLaunchKernelGGL((gp_step_kernel<D, true, false, true, false>), dim3((n + 63) / 64, c->groups), dim3(BAGEL_BLOCK), 0, c->stream, c->Xs, c->Xn,
                       c->Os, reinterpret_cast<const float4 *>(c->Of), c->A, c->v4, c->w4, j.x, c->part_all, c->exp_tab, c->near_ok, n,
                       c->dm.S, B / c->dm.S, c->Np, c->Lp, c->CK, c->CL, c->nck, c->ncl, c->M, j);
    hipLaunchKernelGGL(jac_reduce_kernel<true>, dim3((n + 63) / 64, c->M), dim3(BAGEL_BLOCK), 0, c->stream, j, n, D, c->M, (c->nck + 3) / 4,
                       (c->ncl + 3) / 4);
    return hipGetLastError();
}

}  // namespace

int bagel_env_int(const char *name, int dflt)
{
    const char *s = getenv(name);
    if (!s || !*s) return dflt;
    const int v = atoi(s);
    return v > 0 ? v : dflt;
}

// The units of a launch of few workgroups (fewer than 1024: all of them are on the chip at once).  *CK = *CL: the equal units of 32 or 64 that
// stay where the following does not apply.
// Its time is that of the fullest compute unit, or, where a compute unit has one or two workgroups, of the longest unit: a wave
// alone on its SIMD waits for its own chain.  So the pair (CK, CL) is taken whose fullest compute unit, with the workgroups
// dealt out in turn, has the least to do.  Costs are in instructions per lane: 2 D + 18 a point, 1.6 times the D + 9 + 4 ceil(D / 4) of a
// feature (sines and cosines issue slower), 500 a workgroup, 40 a partial sum (the end-of-step kernel adds them up).  Fitted
// to 17 problems timed at up to 87 pairs each (B = 100 .. 4096, N = 512 .. 8000, L = 256 .. 4096, D = 3 .. 8): the pair taken is on
// average 2.8 % of a step from the best one, units of 32 or 64 were 13 % from it.  us a step of a gradient call, before and after:
// M = 4, N = L = 2048, B = 1024 26.6 -> 24.6 (128 and 64 instead of 64 and 64), M = 3, N = 1533, L = 901, B = 777 21.7 -> 18.6 (48, 48),
// M = 5, N = 4000, L = 2000, B = 640 36.6 -> 32.2 (128, 80), M = 4, N = 5000, L = 3000, B = 400 27.7 -> 25.4 (96, 64).
// Where equal units make 1024 workgroups or more they have the table form, which suits launches with much to do for the training points, values
// alone above all, and they are a candidate like the pairs: 8 instructions a point less, no round of workgroups to fill, 4000 to begin
// with.  (D = 3 .. 8, N = 256 .. 6000, L = 256 .. 4096, 746 such problems: the pairs are 1.04 times as fast in gradient calls and 0.98 times in
// forward passes over all of them, but 0.96 and 0.91 times over the 92 that this leaves with equal units, of which 5 and 4 would be more than 2 %
// faster with pairs.  us a step, pair and equal: M = 6, D = 8, N = 437, L = 864, B = 2729 46.1 and 40.2, forward 32.2 and 28.4;
// M = 4, D = 6, N = 1585, L = 398, B = 3342 49.2 and 44.6, 35.4 and 31.7; M = 2, D = 3, N = 3209, L = 323, B = 4078 43.0 and 40.8, 34.8 and 30.5.)
// Past eight inputs the loops do not take points in pairs, and the pairs of sizes pay where equal units make a launch of 321 to 2047
// workgroups (23 problems with D = 9 .. 14: 0.97 to 1.25 times as fast, 1.05 on average), not outside (11 others: 0.86 to 1.01; above, equal
// units make launches of the table form: M = 8, D = 16, N = L = 1024, B = 1024 54.7 us at (32, 32), 58.1 at (128, 64)), and not for 16 inputs,
// whose float32 chains cost what they give (M = 8, N = 468, L = 1747, B = 592 43.2 us at (32, 32), 44.7 at (64, 64)).
static void small_launch_units(int D, int M, int N, int L, int B, int *CK, int *CL)
{
    const int sizes[] = {32, 48, 64, 80, 96, 128, 160, 192, 256};
    const int64_t tiles = (int64_t)M * ((B + 63) / 64), point = 2 * D + 18, feature5 = 8 * (D + 9 + 4 * ((D + 3) / 4));
    int64_t least = INT64_MAX;
    {
        const int64_t gk = ((N + *CK - 1) / *CK + 3) / 4, gl = ((L + *CL - 1) / *CL + 3) / 4, wk = tiles * gk, w = wk + tiles * gl;
        if (D > 8 && (w <= 320 || w >= 2048 || D == 16)) return;
        if (D <= 8 && w >= 1024)
            least = (wk * (*CK * (point - 8) + 100) + (w - wk) * (*CL * feature5 / 5 + 100)) / 256 + 4000 + 40 * M * (gk + gl);
    }
    for (const int ck : sizes)
        for (const int cl : sizes) {
            if (cl > 2 * ck || ck > 4 * cl) continue;
            const int64_t gk = ((N + ck - 1) / ck + 3) / 4, gl = ((L + cl - 1) / cl + 3) / 4, wk = tiles * gk, w = wk + tiles * gl;
            if (w >= 1024) continue;
            const int64_t tk = ck * point, tl = cl * feature5 / 5;
            int64_t fullest = 0;             // the load changes only where a kind's last round ends
            for (const int64_t cu : {(int64_t)0, wk & 255, w & 255}) {
                const int64_t nk = (wk - cu + 255) / 256, n = (w - cu + 255) / 256, load = nk * (tk + 500) + (n - nk) * (tl + 500);
                if (load > fullest) fullest = load;
            }
            const int64_t longest = tk > tl ? tk : tl;
            if (fullest < longest * 14 / 5) fullest = longest * 14 / 5;
            const int64_t cost = fullest + longest / 5 + 40 * M * (gk + gl);
            if (cost < least) {
                least = cost;
                *CK = ck;
                *CL = cl;
            }
        }
}

// Work decomposition of one sample evaluation (sets CK, CL, nck, ncl, Np, Lp, units, groups and the
// exp2 form from dm, D, M); returns a message if the problem cannot be decomposed.  plain: without what the unit sizes of small
// launches and of features were refined by (bagel_sample_eval_static, whose fixed scratch array decides which sizes it takes).
const char *bagel_plan_sample_eval(bagel_ctx *c, bool plain)
{
    // work decomposition of one sample evaluation: power-of-two chunk of training points / features
    const bagel_dims *dims = &c->dm;
    const int B = dims->B, N = dims->N, L = dims->L, M = c->M;
    const int64_t tb = (B + BAGEL_BLOCK - 1) / BAGEL_BLOCK;
    const int64_t items = (int64_t)(N + L) * M * tb;
    const int target = bagel_env_int("BAGEL_TARGET_WGS", 4096);
    int chunk = 1024;
    while (chunk > 32 && items / chunk < target) chunk /= 2;
    // Longer units for the training points when there are plenty of them (fewer partial sums), shorter
    // ones for the features of a large problem: workgroups are dispatched in grid order, training-point
    // units first, so short feature units at the end fill the tail of the launch.  Measured on MI355X:
    // stress 0.650 ms per launch at (CK, CL) = (1024, 512), 0.628 ms at (1024, 256); the large-policy
    // step 140.6 ms at (128, 64), 136.8 ms at (256, 64).  Features in units of 32 pay only where there are few of them: M = 4,
    // N = L = 2048, B = 2048 44.1 us a step at (128, 32), 41.6 at (128, 64), N = L = 1024, B = 4096 46.8 and 43.3, N = 8192, L = 4096,
    // B = 1024 58.4 and 56.4, M = 6, D = 9, N = 1024, L = 1500, B = 2560 64.4 and 60.1, but M = 3, N = 1024, L = 512, B = 8192 47.9 and 48.7.
    const bool small_launch = chunk == 32 && items / chunk < target;
    int ck = N / chunk >= 32 ? 4 * chunk : (N / chunk >= 16 ? 2 * chunk : chunk);
    int chain = (chunk >= 512 && L / chunk >= 8) ? chunk / 2 : chunk;       // longest float32 sum of features
    int cl = chunk == 32 && L >= 1024 && !plain ? 64 : chain;
    if (small_launch) {
        // equal units of 32 or 64 where a rollout may take one workgroup per trajectory (rollout.hip; whether it does depends on more,
        // but results must not), the best pair otherwise
        ck = cl = chain = N / chunk >= 64 ? 64 : 32;
        if (!plain && !bagel_rollout_rows_fit(c, ck)) small_launch_units(c->D, M, N, L, B, &ck, &cl);
    }
    c->CK = bagel_env_int("BAGEL_CK", ck);
    c->CL = bagel_env_int("BAGEL_CL", cl);
    c->feature_chains = c->CL == cl && cl > chain;
    c->CK = (c->CK + 15) & ~15;       // the sample-evaluation loops take two or four float4 (eight or sixteen points) per trip
    c->CL = (c->CL + 15) & ~15;
    c->nck = (N + c->CK - 1) / c->CK;
    c->ncl = (L + c->CL - 1) / c->CL;
    c->Np = c->nck * c->CK;
    c->Lp = c->ncl * c->CL;
    c->units = M * (c->nck + c->ncl);
    c->groups = M * ((c->nck + 3) / 4 + (c->ncl + 3) / 4);
    // The table form of the kernel-row loop (gp_step.hip) pays once the launch has a few workgroups per
    // compute unit; below that its extra set-up per workgroup (the table copy) and the wait counter its
    // LDS read shares with the scalar loads cost more than its five fewer instructions per training point
    // save.  Measured on MI355X, table vs general form, per launch: stress (4608 workgroups) 583 vs 655 us; large policy (3072) 85.1 vs 97.6;
    // M = 4, N = L = 2048, B = 2048 (1536) 34.9 vs 38.9; the same at B = 1400 in units of 64 (1408) 28.3 vs 29.5, at B = 1024 (1024)
    // 22.5 vs 22.0, and in units of 128 and 64 (768) 23.6 vs 21.3; small (192) 9.5 vs 8.5.
    {
        const int64_t wgs = (int64_t)((B + 63) / 64) * c->groups;
        const int tab = bagel_env_int("BAGEL_EXP_TABLE", 0);         // 1: off, 2: on, otherwise by launch size
        c->exp_table = tab == 2 ? true : (tab == 1 ? false : wgs >= 1024);
    }
    if (c->units > 65535 - BAGEL_MAX_STATE) return "too many work units (M * (N + L) / 32 must stay below 65527)";
    return nullptr;
}

hipError_t bagel_launch_gp_step(bagel_ctx *c, bool jac, float *prev_jac)
{
    switch (c->D) {
#define CASE(n) case n: return launch_d<n>(c, jac, prev_jac);
        CASE(2) CASE(3) CASE(4) CASE(5) CASE(6) CASE(7) CASE(8) CASE(9) CASE(10) CASE(11) CASE(12)
        CASE(13) CASE(14) CASE(15) CASE(16)
#undef CASE
    }
    return hipErrorInvalidValue;
}

hipError_t bagel_launch_jac_reduce(bagel_ctx *c, float *jdst)
{
    const jac_sums j = {c->part, c->xbuf, c->A, c->amp, jdst};
    hipLaunchKernelGGL(jac_reduce_kernel<false>, dim3((c->dm.B + 63) / 64, c->M), dim3(BAGEL_BLOCK), 0, c->stream, j, c->dm.B, c->D,
                       c->M, (c->nck + 3) / 4, (c->ncl + 3) / 4);
    return hipGetLastError();
}

hipError_t bagel_launch_gp_steps(bagel_ctx *c)
{
    const int H = c->dm.H;
    for (int t0 = 0; t0 < H; t0 += c->rollout_steps) {
        const int steps = t0 + c->rollout_steps < H ? c->rollout_steps : H - t0;
        hipError_t e = hipErrorInvalidValue;
        switch (c->D) {
#define CASE(n) case n: e = launch_steps<n>(c, t0, steps); break;
            CASE(2) CASE(3) CASE(4) CASE(5) CASE(6) CASE(7) CASE(8)
#undef CASE
        }
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}
