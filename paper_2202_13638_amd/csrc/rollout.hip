// The forward pass of a whole rollout in one launch, one workgroup per trajectory.
//
// With few trajectories a rollout is a chain of latencies: a sample evaluation spread over the chip and an end-of-step
// kernel take two launches, four trips to memory and a hand-over between compute units for every step, whatever little
// there is to compute.  Here a trajectory never leaves its compute unit: 512 threads hold the rows of the model tables and the
// trajectory's weights v and w in registers for the whole horizon (the policy's weights in LDS), and a step is three to five
// barriers.  What bounds it is the float64 arithmetic of one compute unit and what lies between the barriers.  A forward step of a gradient
// call takes 2.4 us at M = 4, N = 512, L = 1024, 64-64, B = 256 (11.7 in two launches), 2.5 at M = 2, N = 2200, L = 1024, 8-8,
// B = 100 (13.2) and 1.2 at M = 2, N = 64, L = 256, 16, B = 16 (8.6), reading the model and the weights 25, 14 and 7 us; the Jacobians afterwards
// take 1.3, 0.4 and 0.3 us a step.
// Of a step of the first of them (about 6000 cycles) the policy and the state take 3000, one wave after the other with one contraction each,
// the terms 2300 (float64 instructions of two waves a SIMD, about 5 cycles each) and their sums 650 (a chain of dependent additions).
// What is off that chain, the tapes, the goals ahead and the cost, belongs to waves that wait anyway.  (2.9, 2.8 and 1.4 us a step while
// addresses were formed anew for every store, 1400 cycles of one wave, and the waits for the rows stood inside the loop.)
//
// Only values are computed here.  The Jacobians feed nothing but the backward pass, so they are computed afterwards for all
// steps at once, where they fill the chip (bagel_launch_gp_steps): the exponentials are computed twice, which is cheaper than
// a chain with D times more sums in it.
//
// Every number is formed in the order of gp_step.hip and policy16.hip, so states and costs have the same bits as a rollout by
// those kernels: terms are computed by whichever thread has the operands and left in LDS, and one thread per work unit adds
// them up in order; four units make a group sum, group sums are added as step_tail16_kernel adds them.
#include <cstddef>
#include <type_traits>

#include "policy16.h"
#include "sample_math.h"

namespace {

constexpr int NT = 512;                      // threads
constexpr int NW = NT / 64;
constexpr int MAX_SUMS = 512;                // group sums in LDS (a multiple of eight for every output and kind)
constexpr int LDS_BYTES = 152 * 1024;        // what the launch may ask for beside the static arrays

// Pairs of an output and a training point or feature go to the waves in chunks of 64, in turn.  A thread keeps the rows of
// this many pairs, 2 (D + 1) + 1 registers each, in about 160 of its 256 registers.
template <int D>
constexpr int chunks_per_wave() { return 160 / (2 * D + 3) < 16 ? 160 / (2 * D + 3) : 16; }

__device__ __forceinline__ double from_lane(double v, int lane)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane), __builtin_amdgcn_readlane(__double2loint(v), lane));
}

template <int CTRL>
__device__ __forceinline__ double dpp_move(double v)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}

// A contraction runs through a block of 16 units as the matrix instructions of policy16.hip do: unit16(g, e) is at place 4 e + g.
// Weights and activations lie in that order here, so that a chain reads four of each at a time.
// Slices of 32 start nine groups apart, on banks of their own.
__host__ __device__ constexpr int act_place(int unit)
{
    return (unit >> 5) * 36 + (unit & 0x18) + ((unit & 2) << 1 | (unit & 1) << 1 | (unit >> 2 & 1));
}

// a chain over one block: weights in steps of STRIDE groups, requested ahead (they do not depend on the layer before; requested after the
// barrier in front of the layer, 112 calls of 100 steps take 1.2 % longer on average)
template <int STRIDE>
__device__ __forceinline__ void load16(f4v (&a)[4], const f4v *w, bool there = true)
{
    if (there) {
#pragma unroll
        for (int i = 0; i < 4; ++i) a[i] = w[i * STRIDE];
    } else {
        // (not used; without a value of any kind here the registers of the step before would be kept)
#pragma unroll
        for (int i = 0; i < 4; ++i) asm volatile("" : "=v"(a[i]));
    }
}
__device__ __forceinline__ float chain16(const f4v (&a)[4], const f4v *x, float acc)
{
    f4v h[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) h[i] = x[i];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc = fmaf(a[i][e], h[i][e], acc);
    __builtin_amdgcn_sched_barrier(0);       // (the operands of the next block in the registers of this one's)
    return acc;
}

// The policy's weights in LDS, in groups of four along a chain, zero past the layers' ends, so that a chain needs no condition.  What a
// zero weight adds changes no bit as long as its operand is finite: activations of units that do not exist stay zero (an infinite goal
// saturates the units there are, and zero times infinity would make the others not a number).
//   hidden layer 1 [4][width], hidden layer 2 [4 blocks][lanes], output layer [2 * 4][32 lanes], biases [3][128] floats.
// A long contraction is cut into slices that are added up in order, as in policy16.hip: at most four for up to 64 units, two for more.
// Hidden layer 2 gives two or four neighbouring lanes to a unit, one a slice (lanes for slices that are not there would read weights as
// the others do, and the layer is bound by reading them), the output layer four to an action.
template <bool WIDE>
struct policy_weights {
    static constexpr int W = WIDE ? 128 : 64, LANES = 256;
    static constexpr int MID = 4 * W, LAST = MID + (WIDE ? 16 : 8) * LANES, BIAS = LAST + 8 * 32;      // in groups of four
    static constexpr int FLOATS = 4 * BIAS + 3 * 128;
};

struct policy_shape {
    int nl, width[4];
    int fs;                                  // blocks per slice of hidden layer 2
};

struct rollout_args {
    int B, S, per_sample, H, M, da, Np, Lp, nck, ncl;
    int GS;                                  // room for the group sums of an output and kind
    int KC, FC;                              // chunks of training points (per output whole ones) and of features
    int d_in, dg, cost_kind, keep;
    int w_off[3], b_off[3];
    int tracked[8];
    float q[8];
    float act_bound, sigma_r;
    float *tape_s, *states_out;              // null: not kept
    float *h[3], *a_slot;                    // activation tapes (keep)
    double *lpt;
    double *xall;                            // [D][H][B], inputs of every step for the Jacobians, null: not kept
    pack16_args pack;                        // for the workgroups past the trajectories
};

__device__ __forceinline__ double shuffle(double v, int lane)
{
    return __hiloint2double(__builtin_amdgcn_ds_bpermute(4 * lane, __double2hiint(v)), __builtin_amdgcn_ds_bpermute(4 * lane, __double2loint(v)));
}

// A wave's own LDS writes are seen by its later reads; this keeps the compiler from moving them
__device__ __forceinline__ void wave_sync() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }

// What a step leaves behind, as floats in one place: a lane that stores one of them to a tape knows its place
struct step_values {
    static constexpr int ACT = 144;          // floats of a layer
    double x[16];                            // inputs of the sample evaluation
    float act[2][ACT];
    float hin[16];                           // policy input
    float a[8];                              // action tape
};
// places in it, in floats (those of x: two a value)
constexpr int AT_ACT = offsetof(step_values, act) / sizeof(float), AT_HIN = offsetof(step_values, hin) / sizeof(float),
              AT_A = offsetof(step_values, a) / sizeof(float);
static_assert(offsetof(step_values, x) == 0 && AT_ACT == 2 * 16 && AT_HIN == AT_ACT + 2 * step_values::ACT && AT_A == AT_HIN + 16 &&
                  sizeof(step_values) == (AT_A + 8) * sizeof(float),
              "no gaps: a value is stored from its place counted in floats");
// the second unit of a lane lies this far behind the first
constexpr int ACT_MORE = act_place(64) - act_place(0);
static_assert(act_place(127) < step_values::ACT && act_place(63 + 64) - act_place(63) == ACT_MORE, "units 64 apart lie equally far apart");

template <int D, int CK, bool WIDE>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(2, 2))) void rollout_kernel(
    rollout_args r, policy_shape p, const float *__restrict__ theta, const double *__restrict__ Xs, const double *__restrict__ Os,
    const double *__restrict__ A, const double *__restrict__ amp, const float *__restrict__ v4, const float *__restrict__ w4,
    const float *__restrict__ s0, const float *__restrict__ goals)
{
    constexpr int E = chunks_per_wave<D>();
    constexpr int RS = CK + 2, CHUNK = 64 / CK * RS;                       // doubles per row and per chunk of terms
    // terms: [KC 64 / CK][CK + 2] doubles of the kernel rows, then [FC 64 / CK][CK + 2] pairs (w, cos) of the features; policy weights
    extern __shared__ __align__(16) double terms[];
    __shared__ __align__(16) double gsum[MAX_SUMS];
    __shared__ double AS[8][D];              // -1/2 A
    __shared__ float goalS[2][16];           // goals of the next step and this one (lane M + j: entry M + j)
    __shared__ __align__(16) step_values sv;
    // Workgroups past the trajectories pack the weights for the backward pass (a launch of its own in front took 4.7 us)
    if ((int)blockIdx.x >= r.B) {
        pack_theta16(r.pack, theta, ((int)blockIdx.x - r.B) * NT + (int)threadIdx.x);
        return;
    }
    int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // workgroups of one chiplet (they go to the eight in turn) take neighbouring trajectories: these share the lines of a tape row
    int b;
    {
        const int n = r.B, x = blockIdx.x & 7, q = n >> 3, rest = n & 7;
        b = x * q + (x < rest ? x : rest) + ((int)blockIdx.x >> 3);
    }
    const int B = r.B, M = r.M, sample = b / r.per_sample;

    // ---- what stays where it is for the whole horizon ---------------------------------------------------------------
    double row[E][D + 1];
    float weight[E];
    // Chunks of points take slots 0, 1, ..., chunks of features E - 1, E - 2, ...: every slot index below is a constant
    const int kchunks = (r.KC - wave + NW - 1) / NW, fchunks = (r.FC - (NW - 1 - wave) + NW - 1) / NW;
    int m_of_chunk = 0;                      // lane i: the output of the wave's chunk i
    {
        const int per_m = r.KC / M;          // chunks per output
        m_of_chunk = min((lane * NW + wave) / per_m, M - 1);
#pragma unroll
        for (int i = 0; i < E; ++i) {
            const int c = i * NW + wave, cf = (E - 1 - i) * NW + (NW - 1 - wave);
            const double *src = Xs;
            const float *wsrc = nullptr;
            if (i < kchunks) {
                const int m = c / per_m, n = min((c - m * per_m) * 64 + lane, r.Np - 1);
                src = Xs + ((size_t)m * r.Np + n) * (D + 1);
                wsrc = v4 + ((size_t)(m * (r.Np / 4) + n / 4) * r.S + sample) * 4 + (n & 3);
            } else if (E - 1 - i < fchunks) {
                const int f = min(cf * 64 + lane, M * r.Lp - 1);
                src = Os + (size_t)f * (D + 1);
                wsrc = w4 + ((size_t)(f / 4) * r.S + sample) * 4 + (f & 3);
            }
#pragma unroll
            for (int d = 0; d <= D; ++d) row[i][d] = src[d];
            weight[i] = wsrc ? *wsrc : 0.0f;
        }
    }
    // policy weights into LDS
    using PW = policy_weights<WIDE>;
    f4v *const w0 = reinterpret_cast<f4v *>(terms + (r.KC + r.FC) * CHUNK), *const w1 = w0 + PW::MID, *const w2 = w0 + PW::LAST;
    float *const biases = reinterpret_cast<float *>(w0 + PW::BIAS);
    // lanes a unit of hidden layer 2, one a slice: two for up to 64 inputs or more than 64 units, otherwise four (four for all but more than 64
    // units: the same calls 1.1 % longer, 3.7 at 64-64)
    const bool two = !WIDE || p.width[1] <= 64 || p.width[2] > 64;
    {
        const int n0 = p.width[0], n1 = p.width[1], n2 = p.width[2], n_last = p.width[p.nl - 1];
        auto load = [&](int l, bool live, int u, int k, int n_in) { return live && k < n_in ? theta[r.w_off[l] + u * n_in + k] : 0.0f; };
        for (int e = tid; e < 4 * PW::W; e += NT) {
            const int u = e % PW::W, c4 = e / PW::W;
            f4v w;
#pragma unroll
            for (int i = 0; i < 4; ++i) w[i] = load(0, u < n1, u, unit16(i, c4), n0);
            w0[e] = w;
        }
        for (int e = tid; p.nl == 3 && e < 4 * p.fs * PW::LANES; e += NT) {
            const int ln = e % PW::LANES, c4 = e / PW::LANES, u = ln >> (two ? 1 : 2), sl = ln & (two ? 1 : 3);
            f4v w;
#pragma unroll
            for (int i = 0; i < 4; ++i) w[i] = load(1, u < n2, u, 16 * (sl * p.fs + (c4 >> 2)) + unit16(i, c4 & 3), n1);
            w1[e] = w;
        }
        if (tid < 8 * 32) {
            const int ln = tid & 31, c4 = tid >> 5;
            f4v w;
#pragma unroll
            for (int i = 0; i < 4; ++i) w[i] = load(p.nl - 1, (ln >> 2) < r.da, ln >> 2, 16 * (2 * (ln & 3) + (c4 >> 2)) + unit16(i, c4 & 3), n_last);
            w2[tid] = w;
        }
        if (tid < 3 * 128) {
            const int l = tid >> 7, u = tid & 127;
            const int n = l == 0 ? n1 : (l == 1 ? n2 : p.width[3]), off = l == 0 ? r.b_off[0] : (l == 1 ? r.b_off[1] : r.b_off[2]);
            biases[tid] = l < p.nl && u < n ? theta[off + u] : 0.0f;
        }
        if (tid < 2 * step_values::ACT) sv.act[tid / step_values::ACT][tid % step_values::ACT] = 0.0f;
        if (tid < MAX_SUMS) gsum[tid] = 0.0;                               // (group sums past an output's last are never written)
        if (tid < M * D) AS[tid / D][tid % D] = -0.5 * A[tid];
    }
    // a layer that only the first wave has a part in needs no barrier after it
    const int lanes1 = p.nl == 3 ? p.width[2] << (two ? 1 : 2) : 0;        // lanes of hidden layer 2
    // blocks of 16 inputs of a slice, at least (with two for all, calls with layers of 8 take 3 % longer, of 64 and more 2 % less)
    const int blocks1 = p.width[1] > 16 ? 2 : 1, blocks2 = p.width[p.nl - 1] > 16 ? 2 : 1;
    const bool barrier0 = p.width[1] > 64 || lanes1 > 64, barrier1 = lanes1 > 64;

    int ml = min(lane, M - 1);
    const double amp_lane = amp[ml];
    const int my_term = (lane / CK) * RS + lane % CK, my_points = wave * CHUNK + my_term, my_features = (r.KC + NW - 1 - wave) * CHUNK + my_term;
    // the work unit this thread adds up: kernel rows first, features from the next whole wave on.  Group sums of output m: the
    // kernel rows' from (2 m) GS, the features' from (2 m + 1) GS on
    int unit_at = 0, unit_to = 0;            // first term; group sum
    bool unit_live;
    const int ngk = (r.nck + 3) >> 2, ngl = (r.ncl + 3) >> 2, fbegin = (4 * M * ngk + 63) & ~63;
    const bool wave_kernel = 64 * wave < fbegin, sum_wave = 64 * wave < fbegin + 4 * M * ngl;
    {
        const int u = wave_kernel ? tid : tid - fbegin, ng = wave_kernel ? ngk : ngl, nc = wave_kernel ? r.nck : r.ncl;
        const int gr = u >> 2, m = gr / ng, g = gr - m * ng, c = 4 * g + (u & 3);
        unit_live = m < M && c < nc;
        if (unit_live) unit_at = wave_kernel ? (m * (r.KC / M * (64 / CK)) + c) * RS : r.KC * CHUNK + (m * nc + c) * RS;
        unit_to = m < M ? (2 * m + (wave_kernel ? 0 : 1)) * r.GS + g : MAX_SUMS - 1;
    }

    // ---- what is kept of a step: one value a lane (two of a layer of more than 64 units), by waves 5 to 7 --------------------
    // keep_at: place in sv (-1: none), keep_to: where it goes in this step, keep_stride: floats from step to step.  (Formed from the
    // arguments in every step instead, addresses and conditions took these waves 1400 cycles, and the others waited.)
    // goal_from: of wave 4 instead, the goals to fetch next; it keeps nothing (keep_at, keep_more), so nothing is ever stored there.  The two
    // share registers on purpose: with a pointer for each a launch took 792 instead of 775 us (B = 100, N = 2200, H = 300), 268 instead of 266 and,
    // saturating, 290 instead of 278 (B = 256, N = 512, H = 100), with the goals' in scalar registers 806, 275 and 297.
    int keep_at = -1, keep_more = 0, keep_stride = 0;
    union {
        float *keep_to = nullptr;
        const float *goal_from;
    } walk;
    const float *const svf = reinterpret_cast<const float *>(&sv);
    {
        auto keep = [&](bool mine, float *base, size_t offset, int stride, int at) {
            if (mine && base) {
                walk.keep_to = base + offset;
                keep_stride = stride;
                keep_at = at;
            }
        };
        const size_t Bz = (size_t)B;
        if (wave == 7) {
            const int j = lane & 15;
            keep(lane < M, r.tape_s, lane * Bz + b, M * B, AT_HIN + lane);
            keep(lane >= 8 && lane < 8 + M, r.states_out, (size_t)b * M + lane - 8, M * B, AT_HIN + lane - 8);
            keep(lane >= 16 && lane < 16 + r.d_in && r.keep, r.h[0], j * Bz + b, r.d_in * B, AT_HIN + j);
            keep(lane >= 32 && lane < 32 + 2 * D, reinterpret_cast<float *>(r.xall), 2 * ((j >> 1) * (size_t)r.H * Bz + b) + (j & 1), 2 * B, j);
            keep(lane >= 48 && lane < 48 + r.da && r.keep, r.a_slot, j * Bz + b, r.da * B, AT_A + j);
        }
        if (wave == 5 || wave == 6) {
            const int l = 6 - wave;          // wave 6: hidden layer 1
            if (l < p.nl - 1 && r.keep) {
                const int n = l == 0 ? p.width[1] : p.width[2];
                keep(lane < n, l == 0 ? r.h[1] : r.h[2], lane * Bz + b, n * B, AT_ACT + step_values::ACT * l + act_place(lane));
                keep_more = n - 64;
            }
        }
    }

    // ---- state: lane m < M of every wave holds s_m, lanes M .. d_in - 1 the goal the policy sees ------------------------
    double s = lane < M ? (double)s0[(size_t)b * M + ml] : 0.0;
    // (zero past d_in).  Wave 4 fetches the goals two steps ahead and hands them to the others.
    const bool goal_lane = lane >= M && lane < r.d_in;
    float goal = goal_lane ? goals[(size_t)b * r.dg + lane - M] : 0.0f, goal_ahead = 0.0f;
    if (wave == 4) {
        walk.goal_from = goals + (size_t)b * r.dg + lane - M;
        keep_stride = B * r.dg;
        if (goal_lane && r.H > 1) goal_ahead = walk.goal_from[(size_t)keep_stride];
        walk.goal_from += 2 * (size_t)keep_stride;
    }
    if (tid < 16) {
        goalS[0][tid] = goal;
        goalS[1][tid] = 0.0f;
    }
    const int H = r.H, dg = r.dg, da = r.da, GS = r.GS;
    const float act_bound = r.act_bound;
    const bool saturating = r.cost_kind == 1;
    // cost of state s against the goals the policy saw before it (against[M + j]: goal j), by wave 4.  Lane j: tracked state j
    const int cost_lane = r.tracked[min(lane, dg - 1)];
    const double cost_q = (double)r.q[min(lane, dg - 1)];
    double cost = 0.0;
    auto add_cost = [&](const float *against) {
        const double dlt = shuffle(s, cost_lane) - (double)against[M + min(lane, dg - 1)], term = cost_q * dlt * dlt;
        double e = 0.0;
        for (int i = 0; i < dg; ++i) e += from_lane(term, i);
        if (saturating) {
            const double sr2 = (double)r.sigma_r * (double)r.sigma_r;
            e = -cost_exp(-e / (2.0 * sr2));
        }
        cost += e;
    };
    exp2_coefficients ec;
    asm volatile("" : "+v"(ec.c6));
    __syncthreads();
    __builtin_amdgcn_s_waitcnt(0x0f70);      // (vmcnt(0): inside the loop the waits for the rows above would be waits for its stores)

    int t = 0;
    for (;;) {
        // What is the same in every step (addresses, conditions, float64 copies of the weights) is formed again in every step: kept
        // from before the loop, as it would be without this, it takes more registers than there are.
        asm volatile("" : "+v"(tid), "+v"(lane), "+v"(ml));
#pragma unroll
        for (int i = 0; i < E; ++i) asm volatile("" : "+v"(weight[i]));
        // ---- policy ----------------------------------------------------------------------------------------------------
        const float hin = lane < M ? (float)s : goal;
        if (64 * wave < p.width[1]) {
            const float bias = biases[tid];
            f4v w[2] = {w0[tid], w0[PW::W + tid]};
            float z = 0.0f;
            auto inputs = [&](int e) {
                float x[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) x[i] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(hin), unit16(i, e)));
#pragma unroll
                for (int i = 0; i < 4; ++i) z = fmaf(w[e & 1][i], x[i], z);
            };
            inputs(0);
            inputs(1);
            if (r.d_in > 8) {
                w[0] = w0[2 * PW::W + tid];
                w[1] = w0[3 * PW::W + tid];
                inputs(2);
                inputs(3);
            }
            sv.act[0][act_place(tid)] = tid < p.width[1] ? tanh_fast(z + bias) : 0.0f;
        }
        if (wave == 7 && lane < 16) sv.hin[lane] = hin;
        if (p.nl == 3) {
            const int u = two ? tid >> 1 : tid >> 2, sl = two ? tid & 1 : tid & 3;
            auto arrive = [&] {              // (each wave at one of the two places below)
                if (barrier0) __syncthreads();
                else wave_sync();
            };
            if (64 * wave >= lanes1) {
                arrive();
            } else {
                f4v wa[4], wb[4];
                load16<PW::LANES>(wa, w1 + tid);
                const float bias = biases[128 + u];
                arrive();
                load16<PW::LANES>(wb, w1 + 4 * PW::LANES + tid, blocks1 > 1);
                // (past the last slice the weights are zero: operands of any place will do, as one that is not a number is in every unit's chain)
                const f4v *x = reinterpret_cast<const f4v *>(sv.act[0]) + (two ? 9 * (p.fs >> 1) * sl : 9 * sl);
                float z = chain16(wa, x, 0.0f);
                if (blocks1 > 1) z = chain16(wb, x + 4, z);
                if (WIDE && p.fs == 4) {
                    load16<PW::LANES>(wa, w1 + 8 * PW::LANES + tid);
                    z = chain16(wa, x + 9, z);
                    load16<PW::LANES>(wb, w1 + 12 * PW::LANES + tid);
                    z = chain16(wb, x + 13, z);
                }
                // slices in order: quad_perm broadcasts
                const int zi = __float_as_int(z);
                if (two) {
                    z += __int_as_float(__builtin_amdgcn_update_dpp(0, zi, 0xf5, 0xf, 0xf, true));
                } else {
                    z += __int_as_float(__builtin_amdgcn_update_dpp(0, zi, 0x55, 0xf, 0xf, true));
                    z += __int_as_float(__builtin_amdgcn_update_dpp(0, zi, 0xaa, 0xf, 0xf, true));
                    z += __int_as_float(__builtin_amdgcn_update_dpp(0, zi, 0xff, 0xf, 0xf, true));
                }
                if (sl == 0 && u < p.width[2]) sv.act[1][act_place(u)] = tanh_fast(z + bias);
            }
        }
        auto arrive = [&] {
            if (p.nl == 3 ? barrier1 : barrier0) __syncthreads();
            else wave_sync();
        };
        if (wave == 0) {                     // actions: lane 4 o + slice
            const int o = (lane & 31) >> 2, sl = lane & 3;
            f4v wa[4], wb[4];
            load16<32>(wa, w2 + (lane & 31));
            const float bias = biases[128 * (p.nl - 1) + o];
            arrive();
            load16<32>(wb, w2 + 128 + (lane & 31), blocks2 > 1);
            const f4v *x = reinterpret_cast<const f4v *>(sv.act[p.nl - 2]) + 9 * sl;
            float z = chain16(wa, x, 0.0f);
            if (blocks2 > 1) z = chain16(wb, x + 4, z);
            const int zi = __float_as_int(z);
            z += __int_as_float(__builtin_amdgcn_update_dpp(0, zi, 0x55, 0xf, 0xf, true));
            if (WIDE) {
                z += __int_as_float(__builtin_amdgcn_update_dpp(0, zi, 0xaa, 0xf, 0xf, true));
                z += __int_as_float(__builtin_amdgcn_update_dpp(0, zi, 0xff, 0xf, 0xf, true));
            }
            z += bias;
            float a = z, out = z;
            if (act_bound > 0.0f) {
                a = tanh_fast(z);
                out = act_bound * a;
            }
            if (lane < 4 * da && sl == 0) {
                sv.x[M + o] = (double)out;
                sv.a[o] = a;
            }
            if (lane < M) sv.x[lane] = s;
        } else {
            arrive();
            if (wave == 4 && t > 0) add_cost(goalS[(t - 1) & 1]);
        }
        double Am[D];
#pragma unroll
        for (int d = 0; d < D; ++d) Am[d] = AS[ml][d];
        __syncthreads();
        const double xl = sv.x[lane & 15];
        double x[D];
#pragma unroll
        for (int d = 0; d < D; ++d) x[d] = from_lane(xl, d);

        // ---- terms of the kernel rows and features ---------------------------------------------------------------------
        double q = 0.0;                      // lane m
#pragma unroll
        for (int d = 0; d < D; ++d) q = fma(Am[d] * x[d], x[d], q);
        const unsigned far = (unsigned)__ballot(q < -131072.0);            // outputs whose kernel row is zero (see gp_step.hip)
        {
            int nk = kchunks, nf = fchunks;
            asm volatile("" : "+s"(nk), "+s"(nf));
            asm volatile("" : "+s"(ec.c7), "+s"(ec.c5), "+s"(ec.c4), "+s"(ec.c3), "+s"(ec.c2), "+s"(ec.c1), "+s"(ec.c0));
            double *kout = terms + my_points, *fout = terms + my_features;
            const double q_of_chunk = shuffle(q, m_of_chunk);              // lane i: of chunk i (looked up chunk by chunk: 1.2 % longer)
            auto exponent = [&](int i) {
                double e = from_lane(q_of_chunk, i) + row[i][D];
#pragma unroll
                for (int d = 0; d < D; ++d) e = fma(x[d], row[i][d], e);
                return e;
            };
            auto point = [&](int i, double e) { kout[i * (NW * CHUNK)] = (double)weight[i] * exp2_poly(e, ec); };
            auto phase = [&](int j) {
                double z = x[0] * row[E - 1 - j][0];
#pragma unroll
                for (int d = 1; d < D; ++d) z = fma(x[d], row[E - 1 - j][d], z);
                return z + row[E - 1 - j][D];
            };
            auto feature = [&](int j, double z) {
                const float y = (float)__builtin_amdgcn_fract(z);
                *reinterpret_cast<float2 *>(fout + j * (NW * CHUNK)) = make_float2(weight[E - 1 - j], __builtin_amdgcn_cosf(y));
            };
            // (nested, so that a wave leaves with one branch after its last chunk)
            auto points = [&](auto self, auto slot) {
                constexpr int i = decltype(slot)::value;
                if constexpr (i < E) {
                    if (i >= nk) return;
                    if (i + 1 < E && i + 1 < nk) {
                        const double e0 = exponent(i), e1 = exponent(i + 1);
                        double k0, k1;
                        exp2_poly2(e0, e1, ec, k0, k1);
                        kout[i * (NW * CHUNK)] = (double)weight[i] * k0;
                        kout[(i + 1) * (NW * CHUNK)] = (double)weight[i + 1] * k1;
                        self(self, std::integral_constant<int, i + 2>{});
                    } else {
                        point(i, exponent(i));
                    }
                }
            };
            auto features = [&](auto self, auto slot) {
                constexpr int j = decltype(slot)::value;
                if constexpr (j < E) {
                    if (j >= nf) return;
                    if (j + 1 < E && j + 1 < nf) {
                        const double z0 = phase(j), z1 = phase(j + 1);
                        feature(j, z0);
                        feature(j + 1, z1);
                        self(self, std::integral_constant<int, j + 2>{});
                    } else {
                        feature(j, phase(j));
                    }
                }
            };
            // The order of points and features decides what the compiler keeps in registers.  100 steps, N = 300, L = 500, B = 128, one layer of 30, features
            // first and last: D = 2 140.1 and 141.1 us, D = 3 149 and 154, D = 4 150.4 and 151.3, D = 5 182 and 171, D = 6 186 and 174, D = 7 224 and 216,
            // D = 8 (N = 250, L = 300) 171 and 160.
            if constexpr (D <= 4) features(features, std::integral_constant<int, 0>{});
            if (__builtin_expect(far == 0, 1)) {
                points(points, std::integral_constant<int, 0>{});
            } else {
                double outside = -3000.0;
                asm volatile("" : "+s"(outside));
#pragma unroll
                for (int i = 0; i < E; ++i)
                    if (i < nk) point(i, far >> __builtin_amdgcn_readlane(m_of_chunk, i) & 1 ? outside + row[i][D] : exponent(i));
            }
            if constexpr (D > 4) features(features, std::integral_constant<int, 0>{});
        }
        __syncthreads();
        // ---- sums of the work units, four of them to a group ---------------------------------------------------------
        if (sum_wave) {
            double sum = 0.0;
            constexpr int N4 = CK / 8;       // batches of four reads, the next one under way while one is added up
            if (wave_kernel) {
                const double2 *t2 = reinterpret_cast<const double2 *>(terms + unit_at);
                double2 a[2][4];
#pragma unroll
                for (int i = 0; i < 4; ++i) a[0][i] = t2[i];
#pragma unroll
                for (int n = 0; n < N4; ++n) {
                    if (n + 1 < N4) {
#pragma unroll
                        for (int i = 0; i < 4; ++i) a[(n + 1) & 1][i] = t2[4 * n + 4 + i];
                    }
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        sum += a[n & 1][i].x;
                        sum += a[n & 1][i].y;
                    }
                }
            } else {
                const f4v *t2 = reinterpret_cast<const f4v *>(terms + unit_at);
                float pf = 0.0f;
                f4v a[2][4];
#pragma unroll
                for (int i = 0; i < 4; ++i) a[0][i] = t2[i];
#pragma unroll
                for (int n = 0; n < N4; ++n) {
                    if (n + 1 < N4) {
#pragma unroll
                        for (int i = 0; i < 4; ++i) a[(n + 1) & 1][i] = t2[4 * n + 4 + i];
                    }
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        pf = fmaf(a[n & 1][i][0], a[n & 1][i][1], pf);
                        pf = fmaf(a[n & 1][i][2], a[n & 1][i][3], pf);
                    }
                }
                sum = (double)pf;
            }
            if (!unit_live) sum = 0.0;
            // quad broadcasts: the four units of the group in order
            double tot = dpp_move<0x00>(sum) + dpp_move<0x55>(sum);
            tot += dpp_move<0xaa>(sum);
            tot += dpp_move<0xff>(sum);
            if ((lane & 3) == 0) gsum[unit_to] = tot;
        }
        // ---- meanwhile, what is kept of this step and the goals ahead (by the last waves, which mostly have no unit) -------------
        if (wave >= 4) {
            if (wave == 4) {
                if (lane < 16) goalS[(t + 1) & 1][lane] = goal_lane ? goal_ahead : 0.0f;
                if (goal_lane && t + 2 < H) goal_ahead = load_pinned(walk.goal_from);
            } else {
                if (keep_at >= 0) *walk.keep_to = svf[keep_at];
                if (WIDE && lane < keep_more) walk.keep_to[64 * (size_t)B] = svf[keep_at + ACT_MORE];
            }
            walk.goal_from += keep_stride;   // (either)
        }
        __syncthreads();
        // ---- state s_{t+1}: lanes 2 m add up the kernel rows of output m, lanes 2 m + 1 its features (8 sums, then the rest: see
        // step_tail16_kernel) ------------------------------------------------------------------------------------------
        float goal_next;
        {
            goal_next = goalS[(t + 1) & 1][lane & 15];
            const double2 *g2 = reinterpret_cast<const double2 *>(gsum + min(lane, 2 * M - 1) * GS);
            double tot = 0.0, rest = 0.0;
            for (int c0 = 0; c0 < GS; c0 += 8) {
                double2 a[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) a[i] = g2[c0 / 2 + i];
                double v = c0 > 0 ? rest : 0.0;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    v += a[i].x;
                    v += a[i].y;
                }
                if (c0 > 0) rest = v;
                else tot = v;
            }
            if ((lane & 1 ? ngl : ngk) > 8) tot = tot + rest;
            const double k = shuffle(tot, 2 * ml), e = shuffle(tot, 2 * ml + 1);
            s += amp_lane * e + k;
        }
        goal = lane < 16 ? goal_next : 0.0f;
        if (++t == H) break;
    }
    if (wave == 7 && lane < M) {
        const float f = (float)s;
        if (r.tape_s) (r.tape_s + (size_t)t * M * B)[lane * B + b] = f;
        if (r.states_out) (r.states_out + (size_t)t * M * B)[b * M + lane] = f;
    }
    if (wave == 4) {
        add_cost(goalS[(t - 1) & 1]);
        if (lane == 0) r.lpt[b] = cost;
    }
}

#define ROLLOUT_INPUTS(X) X(2) X(3) X(4) X(5) X(6) X(7) X(8)

int point_chunks(int M, int Np) { return M * ((Np + 63) / 64); }
int feature_chunks(int M, int Lp) { return (M * Lp + 63) / 64; }
int point_chunks(const bagel_ctx *c) { return point_chunks(c->M, c->Np); }
int feature_chunks(const bagel_ctx *c) { return feature_chunks(c->M, c->Lp); }

policy_shape shape(const bagel_ctx *c)
{
    policy_shape p = {};
    p.nl = c->n_layers;
    for (int i = 0; i < 4; ++i) p.width[i] = c->width[i];
    p.fs = p.nl == 3 ? slice_blocks(p.width[2], p.width[1]) : 0;
    return p;
}

size_t lds_bytes(const bagel_ctx *c)
{
    return sizeof(double) * (size_t)(point_chunks(c) + feature_chunks(c)) * (64 / c->CK) * (c->CK + 2) + sizeof(float) * (c->p16 == 2 ? policy_weights<true>::FLOATS : policy_weights<false>::FLOATS);
}

int sums_room(int nck, int ncl) { return ((nck > ncl ? nck : ncl) + 31) / 32 * 8; }
int sums_room(const bagel_ctx *c) { return sums_room(c->nck, c->ncl); }

template <int D>
bool chunks_fit(int points, int features)
{
    for (int w = 0; w < NW; ++w)
        if ((points - w + NW - 1) / NW + (features - (NW - 1 - w) + NW - 1) / NW > chunks_per_wave<D>()) return false;
    return true;
}

// the trips of a compute unit's registers and sums suffice for units of CK points and CK features
bool rows_fit(const bagel_ctx *c, int CK)
{
    const int M = c->M, nck = (c->dm.N + CK - 1) / CK, ncl = (c->dm.L + CK - 1) / CK, ngk = (nck + 3) / 4, ngl = (ncl + 3) / 4;
    if (((4 * M * ngk + 63) & ~63) + 4 * M * ngl > NT) return false;       // one work unit a thread
    if (2 * M * sums_room(nck, ncl) >= MAX_SUMS) return false;
    switch (c->D) {
#define FITS(d) case d: return chunks_fit<d>(point_chunks(M, nck * CK), feature_chunks(M, ncl * CK));
        ROLLOUT_INPUTS(FITS)
#undef FITS
    }
    return false;
}

constexpr int MOST_TRAJECTORIES = 768;       // of a rollout with one workgroup each (see bagel_plan_rollout)

template <int D, int CK, bool WIDE>
hipError_t raise_lds(size_t lds)
{
    return hipFuncSetAttribute(reinterpret_cast<const void *>(rollout_kernel<D, CK, WIDE>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
}

template <int D, int CK, bool WIDE>
hipError_t launch(bagel_ctx *c, const rollout_args &r, const float *theta, const float *s0, const float *goals)
{
    hipLaunchKernelGGL((rollout_kernel<D, CK, WIDE>), dim3(c->dm.B + (r.pack.dst ? (r.pack.p.total() + NT - 1) / NT : 0)), dim3(NT), lds_bytes(c), c->stream, r, shape(c), theta, c->Xs, c->Os,
                       c->A, c->amp, reinterpret_cast<const float *>(c->v4), reinterpret_cast<const float *>(c->w4), s0, goals);
    return hipGetLastError();
}

// the instance f<D, CK, WIDE> for the context
#define FOR_CONTEXT(c, f, ...) \
    ((c)->CK == 32 ? ((c)->p16 == 2 ? f<D, 32, true>(__VA_ARGS__) : f<D, 32, false>(__VA_ARGS__)) \
                   : ((c)->p16 == 2 ? f<D, 64, true>(__VA_ARGS__) : f<D, 64, false>(__VA_ARGS__)))
template <int D>
hipError_t raise_lds(const bagel_ctx *c) { return FOR_CONTEXT(c, raise_lds, LDS_BYTES); }
template <int D>
hipError_t launch(bagel_ctx *c, const rollout_args &r, const float *theta, const float *s0, const float *goals)
{
    return FOR_CONTEXT(c, launch, c, r, theta, s0, goals);
}

}  // namespace

// Whether rollouts take one workgroup per trajectory: where the rows of all points and features fit the registers of a compute
// unit (about 8000 pairs of an output and a point or feature at D = 3, 6000 at D = 5, 4000 at D = 8), the policy is one of up to 128
// units (its weights lie in LDS) and three rounds of workgroups do (one workgroup per compute unit at a time).  Measured on
// MI355X, 60 steps, a gradient call / a forward pass in us, step by step -> here: M = 2, N = 2200, L = 1024, 64-64 at B = 100
// 959 -> 382 / 766 -> 198, B = 512 937 -> 681 / 729 -> 391, B = 768 1046 -> 947 / 773 -> 586, B = 1024 1085 -> 1203 / 868 -> 778;
// M = 4, N = 512, L = 1024, 128-128 at B = 256 972 -> 508 / 711 -> 193, B = 640 1101 -> 1046 / 720 -> 558, B = 1024 1206 -> 1374 /
// 768 -> 742; M = 6, d_a = 2, N = L = 256, 8-8 at B = 16 766 -> 272 / 640 -> 139, B = 768 912 -> 751 / 671 -> 415.
// A round begins with reading the model and the weights into a compute unit, which a few steps do not pay for: five steps for every round
// after the first.  Eight models, calls step by step / here, gradient and forward: one round, H = 1 0.95 .. 1.22 and 1.00 .. 1.46; two
// rounds, H = 1 0.71 .. 1.06 and 0.62 .. 1.08, H = 2 0.84 .. 1.28 and 0.86 .. 1.80, H = 4 1.00 .. 1.53 and 1.16 .. 2.17; three rounds, H = 4
// 0.81 .. 1.25 and 0.87 .. 1.59, H = 8 0.91 .. 1.50 and 1.07 .. 1.87, H = 11 0.97 .. 1.56 and 1.16 .. 2.10.
bool bagel_rollout_rows_fit(const bagel_ctx *c, int units)
{
    return (c->dm.B <= MOST_TRAJECTORIES || bagel_env_int("BAGEL_ROLLOUT", 0) == 2) && rows_fit(c, units);
}

void bagel_plan_rollout(bagel_ctx *c)
{
    c->rollout = false;
    if (c->exp_table || !(c->p16 == 1 || c->p16 == 2)) return;
    if (c->CK != c->CL || (c->CK != 32 && c->CK != 64) || c->feature_chains) return;
    if (!rows_fit(c, c->CK) || lds_bytes(c) > LDS_BYTES) return;
    const int want = bagel_env_int("BAGEL_ROLLOUT", 0);                    // 1: never, 2: wherever it fits, otherwise by size
    c->rollout = want == 2 || (want != 1 && c->dm.B <= MOST_TRAJECTORIES && c->dm.H >= 5 * ((c->dm.B - 1) / 256));
}

hipError_t bagel_raise_rollout_lds(bagel_ctx *c)
{
    switch (c->D) {
#define RAISE(d) case d: return raise_lds<d>(c);
        ROLLOUT_INPUTS(RAISE)
#undef RAISE
    }
    return hipErrorInvalidValue;
}

hipError_t bagel_launch_rollout(bagel_ctx *c, const float *theta, const float *s0, const float *goals, float *states_out, bool tape, bool acts)
{
    rollout_args r = {};
    r.B = c->dm.B; r.S = c->dm.S; r.per_sample = c->dm.B / c->dm.S; r.H = c->dm.H; r.M = c->M; r.da = c->dm.d_a;
    r.Np = c->Np; r.Lp = c->Lp; r.nck = c->nck; r.ncl = c->ncl; r.GS = sums_room(c);
    r.KC = point_chunks(c); r.FC = feature_chunks(c);
    r.d_in = c->d_in; r.dg = c->dm.d_g; r.cost_kind = c->dm.cost_kind; r.keep = acts ? 1 : 0;
    for (int l = 0; l < 3; ++l) { r.w_off[l] = c->w_off[l]; r.b_off[l] = c->b_off[l]; }
    for (int j = 0; j < 8; ++j) { r.tracked[j] = c->dm.tracked[j]; r.q[j] = c->dm.q[j]; }
    r.act_bound = c->dm.act_bound; r.sigma_r = c->dm.sigma_r;
    r.tape_s = tape ? c->tape_s : nullptr;
    r.states_out = states_out;
    for (int l = 0; l < 3; ++l) r.h[l] = l < c->n_layers ? c->tape_h[l] : nullptr;
    r.a_slot = c->tape_a;
    r.lpt = c->lpt;
    r.xall = tape ? c->xall : nullptr;
    if (tape) r.pack = make_pack_args(c);
    switch (c->D) {
#define LAUNCH(d) case d: return launch<d>(c, r, theta, s0, goals);
        ROLLOUT_INPUTS(LAUNCH)
#undef LAUNCH
    }
    return hipErrorInvalidValue;
}
