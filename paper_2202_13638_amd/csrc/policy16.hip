// The policy network, the end of a rollout step around it and the backward sweep, 16 trajectories per workgroup.
//
// Same mathematics as policy.hip, for the sizes at which a step is a chain of latencies: narrow policies at any
// batch, wide ones while the batch leaves compute units idle with 32 trajectories per workgroup (the rule is in
// bagel_plan_policy).  What bounds these kernels is not the matrix work (a 64 x 64 layer for 16 trajectories is 512
// cycles of a wave) but what lies between: launches, trips to memory, barriers, exchanges through LDS.  So:
//   - v_mfma_f32_16x16x4_f32 (D[16x16] += A[16x4] B[4x16]; lane l = 16 g + j feeds A[l % 16][g] and B[g][j], register
//     r holds D[4 g + r][j]): rows = units, columns = trajectories.  Wave w owns the NT row tiles w NT .. of every
//     hidden layer, all weights it needs are in its registers for the whole launch.
//   - Every sum is formed in the order of policy.hip, so results agree with it bit for bit (a matrix instruction is a
//     chain of fused multiply-adds over its contraction index, and 16x16x4 continues a chain where 32x32x2 takes
//     two instructions).  There, a chain runs through eight inputs as 0 4 1 5 2 6 3 7 and a long contraction is cut
//     into slices that are added up afterwards (slice_blocks).  Hence the order of units inside a block of 16: row
//     i = 4 g + r of a tile is unit unit16(g, r), and instruction s of a block contracts, in lane group g, unit16(g, s).
//     A lane's four results of a tile are then its operands of the next contraction over those 16 units, in the order
//     they are needed: one 16-byte LDS write and reads of [trajectory][tile][4 g + r].
//   - The output layer (forward) and the input layer (backward) have one row tile: wave w takes slice w of them.
// Instances: 4 waves of one tile (hidden widths <= 64), 8 of one (<= 128), 8 of two (<= 256; not the backward sweep).
#include "policy16.h"
#include "sample_math.h"

namespace {

struct policy16_args {
    int B, nl, ds, da;
    int width[4];
    float act_bound;
    const float *pack;                       // packed weights of this pass
    float *h[3];                             // slot 0 of the tapes of the layer inputs
    float *a_slot;                           // slot 0: [d_a][B]
    int keep;                                // 0: nobody reads the tapes of this step (forward pass alone, checkpointing)
};

// The trajectories of a workgroup.  Workgroups go to the eight chiplets in turn; a line of a tape row holds two tiles of
// 16 trajectories, so neighbouring tiles are given to workgroups of one chiplet: its L2 then sees whole lines.  With this
// and without activations that nobody reads (policy16_args::keep), forward passes at 256-256, B = 4096 took 57.7 instead of 68.4
// us per step; gradient calls at 64-64, B = 2048, 53.3 instead of 54.2.
// The number of tiles comes from B, which the end of a step has fetched for other reasons, not from the grid's size.  The sweep is compiled
// differently with either (10 to 18 more scalar registers spilled in four instances) and takes the same time: 61 steps at B = 777, from B and from the grid,
// <4, 1, 2, 2, false> 142.9 and 143.4 us, <4, 1, 6, 2, true> 145.5 and 146.5, <8, 1, 6, 2, true> 164.7 and 162.3, <8, 1, 8, 2, false> 169.3 and 170.9.
__device__ __forceinline__ int first_trajectory(int B)
{
    const int n = (B + PL - 1) / PL, x = blockIdx.x & 7, q = n >> 3, r = n & 7;
    return (x * q + min(x, r) + ((int)blockIdx.x >> 3)) * PL;
}

__global__ __launch_bounds__(256) void pack_theta16_kernel(pack16_args a, const float *__restrict__ theta)
{
    pack_theta16(a, theta, blockIdx.x * 256 + threadIdx.x);
}

// The weights of the forward pass a wave multiplies with
template <int NW, int NT>
struct forward_weights {
    float first[NT][4];                      // narrow contraction over the policy input, at most 16 wide
    f4v mid[NT][NW * NT], last[2], bias0[NT], bias1[NT];      // last: the two blocks of slice `wave`
};

// those of the narrow layers and the biases, and the middle layer
template <int NW, int NT>
__device__ __forceinline__ void load_narrow(forward_weights<NW, NT> &f, const float *pack, const pack16 &p, int wave, int lane)
{
    constexpr int TT = NW * NT;
    // (a scalar base and the lane, unsigned: the load adds them itself)
    const unsigned ul = lane, g = ul >> 4;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int tile = wave * NT + t;
#pragma unroll
        for (int s = 0; s < 4; ++s) f.first[t][s] = (pack + p.f_first() + (tile * p.nsi + min(s, p.nsi - 1)) * 64)[ul];
        f.bias0[t] = reinterpret_cast<const f4v *>(pack + p.bias(0) + 16 * tile)[g];
        f.bias1[t] = reinterpret_cast<const f4v *>(pack + p.bias(1) + 16 * tile)[g];
    }
#pragma unroll
    for (int e = 0; e < 2; ++e) f.last[e] = reinterpret_cast<const f4v *>(pack + p.f_last() + min(2 * wave + e, TT - 1) * 256)[ul];
}
template <int NW, int NT>
__device__ __forceinline__ void load_middle(forward_weights<NW, NT> &f, const float *pack, const pack16 &p, int wave, int lane)
{
    constexpr int TT = NW * NT;
    const unsigned ul = lane;
    if (p.nl == 3) {
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int kb = 0; kb < TT; ++kb) f.mid[t][kb] = reinterpret_cast<const f4v *>(pack + p.f_mid() + ((wave * NT + t) * TT + kb) * 256)[ul];
    }
}

// pi_theta for the 16 trajectories of a workgroup, input in h0 ([trajectory][HS], published by a barrier): hidden activations
// to slot `slot` of their tapes, the slices of the action's contraction to red ([slice][action][PL]; the caller's barrier
// publishes them).  act: two buffers.
template <int NW, int NT>
__device__ __forceinline__ void policy16_layers(const policy16_args &a, const pack16 &p, const forward_weights<NW, NT> &f, size_t slot,
                                                int wave, int lane, int b, bool live, const float *h0, float (*act)[PL * shape16<NW, NT>::AS],
                                                float *red)
{
    constexpr int TT = NW * NT, AS = shape16<NW, NT>::AS;
    const int j = lane & 15, g = lane >> 4;
    const bool keep = live && a.keep;
    f4v h[NT];
    float in[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) in[s] = h0[j * HS + unit16(0, s) + ((g & 1) << 2 | g >> 1)];   // zero past the input
    auto epilogue = [&](int l, const f4v (&bias)[NT], float *out) {
        const int n = a.width[l + 1];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int u0 = 16 * (wave * NT + t) + ((g & 1) << 2 | g >> 1);
            float *dst = a.h[l + 1] + (slot * n + u0) * a.B + b;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int u = u0 + unit16(0, r);
                h[t][r] = u < n ? tanh_fast(h[t][r] + bias[t][r]) : 0.0f;
                if (keep && u < n) dst[(size_t)unit16(0, r) * a.B] = h[t][r];
            }
            *reinterpret_cast<f4v *>(out + j * AS + 16 * (wave * NT + t) + 4 * g) = h[t];
        }
        __syncthreads();
    };
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        h[t] = f4v{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int s = 0; s < 4; ++s)
            if (s < p.nsi) h[t] = mfma16(f.first[t][s], in[s], h[t]);
    }
    epilogue(0, f.bias0, act[0]);
    if (p.nl == 3) {
        contract_wide<NT, TT, AS>(h, f.mid, act[0], lane, a.width[1], p.fs);
        epilogue(1, f.bias1, act[1]);
    }
    const int n_last = a.width[p.nl - 1];
    if (32 * wave < n_last) {
        const f4v o = contract_slice<TT, AS>(f.last, act[p.nl - 2], wave, lane);
        const int o0 = (g & 1) << 2 | g >> 1;                               // actions o0 and o0 + 2, at most 8
#pragma unroll
        for (int r = 0; r < 2; ++r) red[(wave * 8 + o0 + 2 * r) * PL + j] = o[r];
    }
}

// The action of thread (output o, trajectory): slices in order, bias, bound; to the tape and, if x, to the GP input
__device__ __forceinline__ void finish_action(const policy16_args &a, const pack16 &p, size_t slot, int o, int bl, int b, bool live,
                                              const float *red, float bias, double *x)
{
    const int slices = (a.width[p.nl - 1] + 31) / 32;
    float z = red[o * PL + bl];
    for (int w = 1; w < slices; ++w) z += red[(w * 8 + o) * PL + bl];
    z += bias;
    float v = z, out = z;
    if (a.act_bound > 0.0f) {
        v = tanh_fast(z);
        out = a.act_bound * v;
    }
    if (live) {
        if (a.keep) a.a_slot[(slot * a.da + o) * a.B + b] = v;
        if (x) x[(size_t)(a.ds + o) * a.B + b] = (double)out;
    }
}

// ---- end of step t and policy of step t + 1 ------------------------------------------------------------------------
// As step_tail_kernel of policy.hip.  s0 != null: the start of a rollout instead (state from s0, no sums, no cost).
struct tail16_args {
    int D, M, dg, ngk, ngl, ncomp;
    int cost_kind, do_policy, direct;
    float sigma_r;
    int tracked[8];
    float q[8];
    const double *amp, *part, *x_cur;
    double *x_next, *lpt;
    float *tape_s_next, *states_out_next;
    const float *goals_t, *goals_next, *s0;
    float *jdst;
    size_t slot;                             // tape slot of the policy's activations
};

constexpr int TAIL_GROUPS = 128;             // value sums of a trajectory that are staged in LDS

// The value of the lane 16 further on, in the even rows of 16 lanes
__device__ __forceinline__ double next_row(double v)
{
    unsigned a = __double2loint(v), b = __double2hiint(v);
    const auto lo = __builtin_amdgcn_permlane16_swap(a, a, false, false), hi = __builtin_amdgcn_permlane16_swap(b, b, false, false);
    return __hiloint2double((int)hi[1], (int)lo[1]);
}

enum tail_mode { TAIL_SUMS, TAIL_DIRECT, TAIL_START };                     // part: groups' sums, final values; s0 instead

// What a step waits for is trips to memory one after the other, so everything is requested before anything waits: the arguments
// (they come from memory as well, and the compiler would fetch each where it is first used, a trip of 300 to 700 cycles a time), what is
// summed, the weights, those of the narrow layers first.  No load stands in a branch of its own: where paths join, the compiler waits for what
// one of them has requested.  What is kept of the state, and the cost, come last, beside the action.  (us a launch, before and now: 64-64,
// B = 1024 6.0 and 4.9, 100-37, B = 777 6.9 and 6.1, 256-256, B = 4096 14.7 and 13.9, of which the matrix instructions take 3.4.  Of that: without the
// arguments at once calls of 40 steps take 1.2 % longer, 1.7 with up to 64 units and 0.4 with 256, with the tapes before the policy 0.7 %.  Half of a
// middle layer of 256 units requested only during the first layer gave nothing: 14.2 and 14.1 us at B = 4096, 13.7 and 13.0 at B = 1024.)
template <int NW, int NT, int MODE>
__global__ __launch_bounds__(64 * NW) void step_tail16_kernel(tail16_args r, policy16_args a, pack16 p)
{
    using S = shape16<NW, NT>;
    __shared__ __align__(16) float act[2][PL * S::AS], h0[PL * HS], red[NW * 8 * PL];
    __shared__ double fS[TAIL_GROUPS][PL], sS[8][PL];
    asm volatile("" ::"s"(r.x_cur), "s"(r.part), "s"(r.amp), "s"(r.goals_t), "s"(r.goals_next), "s"(r.lpt), "s"(r.x_next), "s"(r.tape_s_next),
                 "s"(r.states_out_next), "s"(a.pack), "s"(a.h[0]), "s"(a.h[1]), "s"(a.h[2]), "s"(r.slot), "s"(r.D), "s"(r.M), "s"(r.dg), "s"(r.ngk),
                 "s"(r.ngl), "s"(r.do_policy), "s"(a.B), "s"(a.ds), "s"(a.width[0]), "s"(a.keep), "s"(p.nl), "s"(p.nsi), "s"(p.fs));
    asm volatile("" ::"s"(a.width[1]), "s"(a.width[2]), "s"(a.width[3]), "s"(a.da), "s"(a.act_bound), "s"(a.a_slot), "s"(r.cost_kind));
    p.TT = NW * NT;                          // (not an argument to wait for)
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int bl = tid & (PL - 1), row = tid >> 4;
    const int b0 = first_trajectory(a.B);
    const bool live = b0 + bl < a.B;         // (trajectory bl is also lane % 16: the same for the matrix phases)
    const int b = live ? b0 + bl : a.B - 1;
    const int B = a.B, ds = a.ds, d_in = a.width[0];

    // Thread row 2 m has state m and its kernel rows' sums, row 2 m + 1 its features' sums and goal m.
    const int m = row >> 1, ms = min(m, ds - 1);
    const bool even = (row & 1) == 0;
    double x_in;
    if constexpr (MODE == TAIL_START) x_in = (double)load_pinned(r.s0 + (size_t)b * ds + ms);
    else x_in = load_pinned(r.x_cur + (size_t)ms * B + b);
    const float *const goals = MODE == TAIL_START || r.goals_next ? r.goals_next : r.goals_t;      // (after the last step any will do)
    const float g_in = load_pinned(goals + (size_t)b * r.dg + min(m, r.dg - 1));
    const double amp_in = MODE == TAIL_SUMS ? load_pinned(r.amp + ms) : 0.0;
    // The groups' value sums are fetched by all threads, a few each, and added up from LDS in the order of policy.hip (the
    // first eight, then the rest); more than fit there are added up by one thread row per sum.
    const size_t stride = (size_t)(1 + r.D) * B;
    const int groups = r.M * (r.ngk + r.ngl);
    const bool staged = groups <= TAIL_GROUPS;
    constexpr int PER = TAIL_GROUPS / S::ROWS;
    double v[PER];
    if constexpr (MODE == TAIL_SUMS) {
        if (staged) {
#pragma unroll
            for (int u = 0; u < PER; ++u)
                if (u * S::ROWS < groups) v[u] = load_pinned(r.part + (size_t)min(row + u * S::ROWS, groups - 1) * stride + b);
        }
    }
    const bool cost_row = MODE != TAIL_START && row == S::ROWS - 1;
    float gt_in[8];
    double lp_in = 0.0;
    if (MODE != TAIL_START && wave == NW - 1) {
#pragma unroll
        for (int j = 0; j < 8; ++j) gt_in[j] = load_pinned(r.goals_t + (size_t)b * r.dg + min(j, r.dg - 1));
        lp_in = load_pinned(r.lpt + b);
    }
    forward_weights<NW, NT> f;
    float bias_in = 0.0f;
    if (r.do_policy) {
        load_narrow(f, a.pack, p, wave, lane);
        bias_in = a.pack[p.bias(2) + min(row, 7)];
        load_middle(f, a.pack, p, wave, lane);
    }
    if constexpr (MODE == TAIL_DIRECT) {
        for (int qi = row; qi < r.M * r.ncomp; qi += S::ROWS) {
            const int mq = qi / r.ncomp, comp = qi - mq * r.ncomp;
            const double val = r.part[(size_t)mq * stride + (size_t)comp * B + b];
            if (comp == 0) fS[mq][bl] = val;
            else if (live) r.jdst[(size_t)(mq * r.D + comp - 1) * B + b] = (float)val;
        }
    }
    if constexpr (MODE == TAIL_SUMS) {
        if (staged) {
#pragma unroll
            for (int u = 0; u < PER; ++u)
                if (u * S::ROWS < groups) fS[min(row + u * S::ROWS, TAIL_GROUPS - 1)][bl] = v[u];
        }
    }
    if constexpr (MODE != TAIL_START) __syncthreads();
    if (row < 16) {
        double s = x_in;
        if constexpr (MODE == TAIL_DIRECT) s += fS[ms][bl];
        if constexpr (MODE == TAIL_SUMS) {
            double sum = 0.0;
            if (m < ds) {
                const int n = even ? r.ngk : r.ngl, first = even ? m * r.ngk : r.M * r.ngk + m * r.ngl;
                sum = staged ? sum_groups16(&fS[first][bl], n, PL) : sum_groups16(r.part + (size_t)first * stride + b, n, stride);
            }
            s += amp_in * next_row(sum) + sum;
        }
        const float hin = even ? (float)s : g_in;
        if (even && m < ds) sS[m][bl] = s;
        if (m < (even ? ds : r.dg)) h0[bl * HS + (even ? m : ds + m)] = hin;
        if (row >= d_in) h0[bl * HS + row] = 0.0f;
    }
    if (MODE == TAIL_START && row == 0 && live) r.lpt[b] = 0.0;
    __syncthreads();
    if (r.do_policy) {
        policy16_layers<NW, NT>(a, p, f, r.slot, wave, lane, b, live, h0, act, red);
        __syncthreads();
        if (row < a.da) finish_action(a, p, r.slot, row, bl, b, live, red, bias_in, r.x_next);
    }
    // what is kept of the state and the policy's input, and the cost, by the waves that have no action to finish
    if (row >= 4 && live)
        for (int i = row - 4; i < d_in; i += S::ROWS - 4) {
            const float hin = h0[bl * HS + i];
            if (r.do_policy && a.keep) a.h[0][(r.slot * d_in + i) * B + b] = hin;
            if (i < ds) {
                r.x_next[(size_t)i * B + b] = sS[i][bl];
                if (r.tape_s_next) r.tape_s_next[(size_t)i * B + b] = hin;
                if (r.states_out_next) r.states_out_next[(size_t)b * ds + i] = hin;
            }
        }
    if (cost_row && live) {
        double e = 0.0;
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (j < r.dg) {
                const double dlt = sS[r.tracked[j]][bl] - (double)gt_in[j];
                e += (double)r.q[j] * dlt * dlt;
            }
        if (r.cost_kind == 1) {
            const double sr2 = (double)r.sigma_r * (double)r.sigma_r;
            e = -cost_exp(-e / (2.0 * sr2));
        }
        r.lpt[b] = lp_in + e;
    }
}

// ---- activation tape of the steps t0 .. t0 + n_slots - 1 rebuilt from the kept states (see policy_replay_kernel) --------
struct replay16_args {
    const float *tape_s, *goals;
    int t0, dg, n_slots, per;                // per: steps per workgroup
};

template <int NW, int NT>
__global__ __launch_bounds__(64 * NW) void policy_replay16_kernel(replay16_args r, policy16_args a, pack16 p)
{
    using S = shape16<NW, NT>;
    __shared__ __align__(16) float act[2][PL * S::AS], h0[PL * HS], red[NW * 8 * PL];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int bl = tid & (PL - 1), row = tid >> 4;
    const int b0 = first_trajectory(a.B);
    const bool live = b0 + bl < a.B;
    const int b = live ? b0 + bl : a.B - 1;
    const int B = a.B, ds = a.ds, d_in = a.width[0];
    forward_weights<NW, NT> f;
    load_narrow(f, a.pack, p, wave, lane);
    load_middle(f, a.pack, p, wave, lane);
    const float bias = a.pack[p.bias(2) + min(row, 7)];
    const int s_end = min(r.n_slots, (int)(blockIdx.y + 1) * r.per);
    auto input = [&](int sl) {
        const size_t t = (size_t)(r.t0 + sl);
        if (row < ds) return load_pinned(r.tape_s + (t * ds + row) * B + b);
        if (row < d_in) return load_pinned(r.goals + (t * B + b) * r.dg + (row - ds));
        return 0.0f;
    };
    float in = input(blockIdx.y * r.per);
    for (int sl = blockIdx.y * r.per; sl < s_end; ++sl) {
        if (row < 16) h0[bl * HS + row] = in;
        if (live && row < d_in) a.h[0][((size_t)sl * d_in + row) * B + b] = in;
        __syncthreads();
        if (sl + 1 < s_end) in = input(sl + 1);
        policy16_layers<NW, NT>(a, p, f, sl, wave, lane, b, live, h0, act, red);
        __syncthreads();
        if (row < a.da) finish_action(a, p, sl, row, bl, b, live, red, bias, nullptr);
    }
}

// ---- backward sweep -----------------------------------------------------------------------------------------------------
// As backward_sweep_kernel of policy.hip: the steps t_hi-1 .. t_lo of 16 trajectories per workgroup.  What a step reads from
// the tapes is requested two steps ahead, into the registers that held the values of the step just done with them
// (two sets, the loop body handles two steps), so that no value is copied and nothing waits for a load it does not need.
// For widths up to 128.  Above, the 128 registers of middle weights leave too few for two steps of tape values (an instance
// kept 400 bytes a lane in scratch memory); the sweep of policy.hip, in registers, serves those policies.
struct sweep16_args {
    int B, nl, ds, da, dg, D, M, H, t_hi, t_lo;
    int width[4];
    float act_bound, sigma_r;
    int cost_kind;
    int tracked[8];
    float q[8];
    const float *pack;
    const float *tape_h[3];
    float *tape_d[3];
    const float *tape_a, *tape_J, *tape_s, *goals;
    double *lam;
    float *grad_s0;
};

// MM, DG: at least M and d_g (rounded up to 2, 3, 4, 6 or 8, 2 or 8); ALL: M = MM
template <int NT, int MM, int DG>
struct sweep16_tape {
    float J[MM], th;                         // rows d < D: J[m][d]; actions: tanh output of the bounded action
    float sv[DG], gv[DG];                    // tracked states of s_{t-1} and the goals they are compared with
    f4v top[NT], mid[NT];                    // tanh outputs of the wave's units
};

// lam + (1/B) d cost / d s_i
template <int DG>
__device__ __forceinline__ double add_cost_gradient16(const sweep16_args &a, double lam, int i, const float (&sv)[DG], const float (&gv)[DG])
{
    double r[DG], e = 0.0;
#pragma unroll
    for (int j = 0; j < DG; ++j) {
        r[j] = j < a.dg ? (double)sv[j] - (double)gv[j] : 0.0;
        e += (double)a.q[j] * r[j] * r[j];                                 // (q is zero past d_g: adds +0.0)
    }
    double factor = 2.0;
    if (a.cost_kind == 1) {
        const double sr2 = (double)a.sigma_r * (double)a.sigma_r;
        factor = exp(-e / (2.0 * sr2)) / sr2;
    }
    factor /= (double)a.B;
#pragma unroll
    for (int j = 0; j < DG; ++j)
        if (j < a.dg && a.tracked[j] == i) lam += factor * (double)a.q[j] * r[j];
    return lam;
}

template <int NW, int NT, int MM, int DG, bool ALL>
__global__ __launch_bounds__(64 * NW) void backward_sweep16_kernel(sweep16_args a, pack16 p)
{
    using S = shape16<NW, NT>;
    constexpr int TT = S::TT, AS = S::AS;
    __shared__ __align__(16) float act[2][PL * AS], dS[PL * HS], red[NW * PL * HS];
    __shared__ double lamS[8][PL];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int j = lane & 15, g = lane >> 4, ug = (g & 1) << 2 | g >> 1;       // unit16(g, r) = ug + unit16(0, r)
    const int bl = tid & (PL - 1), row = tid >> 4;
    const int b0 = first_trajectory(a.B);
    const bool live = b0 + bl < a.B;
    const int b = live ? b0 + bl : a.B - 1;
    const int last = a.nl - 1;
    const size_t B = a.B;
    const int n_top = a.width[last];

    // weights: top layer (contraction over the actions), middle, input layer (the wave's slice)
    float w_top[NT][2];
    f4v w_mid[NT][TT], w_first[2];           // w_first: the two blocks of slice `wave`
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int tile = wave * NT + t;
#pragma unroll
        for (int s = 0; s < 2; ++s) w_top[t][s] = a.pack[p.b_top() + (tile * p.nsa + min(s, p.nsa - 1)) * 64 + lane];
        if (a.nl == 3) {
#pragma unroll
            for (int kb = 0; kb < TT; ++kb) w_mid[t][kb] = reinterpret_cast<const f4v *>(a.pack + p.b_mid())[(tile * TT + kb) * 64 + lane];
        }
    }
#pragma unroll
    for (int e = 0; e < 2; ++e) w_first[e] = reinterpret_cast<const f4v *>(a.pack + p.b_first())[min(2 * wave + e, TT - 1) * 64 + lane];
    // rows and units past the end are clamped duplicates nobody uses
    const int rowc = min(row, a.D - 1), ra = min(max(rowc - a.ds, 0), a.da - 1);
    auto request_front = [&](int t, sweep16_tape<NT, MM, DG> &s) {          // what the first phase of step t - 1 reads
        const size_t slot = (size_t)(t - 1 - a.t_lo);
        const float *Jt = a.tape_J + slot * a.M * a.D * B + (size_t)rowc * B + b;
#pragma unroll
        for (int m = 0; m < MM; ++m) s.J[m] = load_pinned(Jt + (size_t)min(m, a.M - 1) * a.D * B);
        s.th = load_pinned(a.tape_a + (slot * a.da + ra) * B + b);
    };
    auto request_units = [&](int t, f4v (&h)[NT], int l) {
        const size_t slot = (size_t)(t - 1 - a.t_lo);
        const int n = a.width[l];
        const float *hl = a.tape_h[l] + slot * n * B + b;
#pragma unroll
        for (int k = 0; k < NT; ++k)
#pragma unroll
            for (int r = 0; r < 4; ++r) h[k][r] = load_pinned(hl + (size_t)min(16 * (wave * NT + k) + ug + unit16(0, r), n - 1) * B);
    };
    auto request_cost = [&](int t, sweep16_tape<NT, MM, DG> &s) {           // data of the state s_{t-1}, for t - 1 >= 1
        const int tc = t - 1 >= 1 ? t : 2;
        const float *st = a.tape_s + (size_t)min(tc - 1, a.H) * a.ds * B + b;
        const float *gt = a.goals + ((size_t)min(tc - 2, a.H - 1) * B + b) * a.dg;
#pragma unroll
        for (int k = 0; k < DG; ++k) {
            const int kc = min(k, a.dg - 1);
            s.sv[k] = load_pinned(st + (size_t)a.tracked[kc] * B);
            s.gv[k] = load_pinned(gt + kc);
        }
    };
    sweep16_tape<NT, MM, DG> set[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const int t = max(a.t_hi - e, a.t_lo + 1);
        request_front(t, set[e]);
        request_units(t, set[e].top, last);
        if (a.nl == 3) request_units(t, set[e].mid, 1);
        request_cost(t, set[e]);
    }

    // adjoint of the state of thread (row < d_s, trajectory): in its register, and in LDS for the contraction with J
    double lam = 0.0, us = 0.0;
    if (row < a.ds) {
        if (a.t_hi == a.H) {
            float sv[DG], gv[DG];
#pragma unroll
            for (int k = 0; k < DG; ++k) {
                const int kc = min(k, a.dg - 1);
                sv[k] = a.tape_s[((size_t)a.H * a.ds + a.tracked[kc]) * B + b];
                gv[k] = a.goals[((size_t)(a.H - 1) * B + b) * a.dg + kc];
            }
            lam = add_cost_gradient16<DG>(a, 0.0, row, sv, gv);
        } else {
            lam = a.lam[(size_t)row * B + b];
        }
        lamS[row][bl] = lam;
    } else if (row < 8) {
        lamS[row][bl] = 0.0;                 // outputs past M add nothing to u
    }
    for (int e = tid; e < PL * HS; e += 64 * NW) dS[e] = 0.0f;
    __syncthreads();

    auto step = [&](int t, sweep16_tape<NT, MM, DG> &s) {
        const size_t slot = (size_t)(t - 1 - a.t_lo);
        const int tn = max(t - 2, a.t_lo + 1);                             // the step this register set is requested for next
        // u = J^T lam: rows d < d_s stay with their thread, the action rows go through the bound to the policy backward
        if (row < a.D) {
            double u = 0.0;
#pragma unroll
            for (int m = 0; m < MM; ++m) {
                float Jm = s.J[m];
                // past M: a duplicate, which may be infinite.  (Instances without this where M = MM: it made a gradient call at
                // 64-64, M = 4, B = 256 take 1387 us instead of 1376, and calls with M = 2, B = 20, N = 858 2796 instead of 2768,
                // or 2707 with a register set of two.)
                if (!ALL) Jm = __int_as_float(__float_as_int(Jm) & ((m - a.M) >> 31));
                u += (double)Jm * lamS[m][bl];
            }
            if (row < a.ds) {
                us = u;
            } else {
                if (a.act_bound > 0.0f) u *= (double)a.act_bound * (1.0 - (double)s.th * (double)s.th);
                const float d = (float)u;
                dS[bl * HS + row - a.ds] = d;
                if (live) a.tape_d[last][(slot * a.da + row - a.ds) * B + b] = d;
            }
        }
        request_front(tn, s);
        __syncthreads();
        f4v dl[NT];
        auto derivative = [&](const f4v (&h)[NT], int l, float *out) {     // delta_l = (W^T delta) (1 - h^2), to its tape and LDS
            const int n = a.width[l];
#pragma unroll
            for (int k = 0; k < NT; ++k) {
                const int u0 = 16 * (wave * NT + k) + ug;
                float *dst = a.tape_d[l - 1] + (slot * n + u0) * B + b;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int u = u0 + unit16(0, r);
                    dl[k][r] *= 1.0f - h[k][r] * h[k][r];
                    if (u >= n) dl[k][r] = 0.0f;
                    else if (live) dst[(size_t)unit16(0, r) * B] = dl[k][r];
                }
                *reinterpret_cast<f4v *>(out + j * AS + 16 * (wave * NT + k) + 4 * g) = dl[k];
            }
            __syncthreads();
        };
        float din[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) din[e] = dS[j * HS + ug + unit16(0, e)];
#pragma unroll
        for (int k = 0; k < NT; ++k) {
            dl[k] = f4v{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int e = 0; e < 2; ++e)
                if (e < p.nsa) dl[k] = mfma16(w_top[k][e], din[e], dl[k]);
        }
        derivative(s.top, last, act[0]);
        request_units(tn, s.top, last);
        if (a.nl == 3) {
            contract_wide<NT, TT, AS>(dl, w_mid, act[0], lane, n_top, p.bs);
            derivative(s.mid, 1, act[1]);
            request_units(tn, s.mid, 1);
        }
        // adjoint of the policy input: one row tile, wave w takes slice w
        if (32 * wave < a.width[1]) {
            const f4v o = contract_slice<TT, AS>(w_first, act[a.nl - 2], wave, lane);
#pragma unroll
            for (int r = 0; r < 4; ++r) red[(wave * PL + j) * HS + ug + unit16(0, r)] = o[r];
        }
        __syncthreads();
        if (row < a.ds) {
            float dh = red[bl * HS + row];
            for (int w = 1; 32 * w < a.width[1]; ++w) dh += red[(w * PL + bl) * HS + row];
            lam = lam + us + (double)dh;
            if (t - 1 >= 1) lam = add_cost_gradient16<DG>(a, lam, row, s.sv, s.gv);
            lamS[row][bl] = lam;
        }
        request_cost(tn, s);
        __syncthreads();
    };
    int t = a.t_hi;
    for (; t - 1 > a.t_lo; t -= 2) {
        step(t, set[0]);
        step(t - 1, set[1]);
    }
    if (t > a.t_lo) step(t, set[0]);
    if (row < a.ds && live) {
        a.lam[(size_t)row * B + b] = lam;
        if (a.t_lo == 0 && a.grad_s0) a.grad_s0[(size_t)b * a.ds + row] = (float)lam;
    }
}

policy16_args make_policy(const bagel_ctx *c, bool keep)
{
    policy16_args a;
    a.keep = keep ? 1 : 0;
    a.B = c->dm.B; a.nl = c->n_layers; a.ds = c->dm.d_s; a.da = c->dm.d_a;
    for (int i = 0; i < 4; ++i) a.width[i] = c->width[i];
    a.act_bound = c->dm.act_bound;
    a.pack = c->wpack16;
    for (int l = 0; l < 3; ++l) a.h[l] = l < c->n_layers ? c->tape_h[l] : nullptr;
    a.a_slot = c->tape_a;
    return a;
}

template <int NW, int NT>
void launch_tail(bagel_ctx *c, const tail16_args &r, bool keep)
{
    const dim3 grid((c->dm.B + PL - 1) / PL), block(64 * NW);
    const policy16_args a = make_policy(c, keep);
    const pack16 p = make_pack(c);
    if (r.s0) hipLaunchKernelGGL((step_tail16_kernel<NW, NT, TAIL_START>), grid, block, 0, c->stream, r, a, p);
    else if (r.direct) hipLaunchKernelGGL((step_tail16_kernel<NW, NT, TAIL_DIRECT>), grid, block, 0, c->stream, r, a, p);
    else hipLaunchKernelGGL((step_tail16_kernel<NW, NT, TAIL_SUMS>), grid, block, 0, c->stream, r, a, p);
}

hipError_t launch_tail(bagel_ctx *c, const tail16_args &r, bool keep)
{
    if (c->p16 == 1) launch_tail<4, 1>(c, r, keep);
    else if (c->p16 == 2) launch_tail<8, 1>(c, r, keep);
    else launch_tail<8, 2>(c, r, keep);
    return hipGetLastError();
}

template <int NW, int NT>
void launch_sweep(bagel_ctx *c, const sweep16_args &a)
{
    const dim3 grid((c->dm.B + PL - 1) / PL), block(64 * NW);
    const pack16 p = make_pack(c);
#define SWEEP(mm, dgm, all) hipLaunchKernelGGL((backward_sweep16_kernel<NW, NT, mm, dgm, all>), grid, block, 0, c->stream, a, p)
    if (a.dg > 2) {
        if (a.M == 8) SWEEP(8, 8, true);
        else SWEEP(8, 8, false);
        return;
    }
    switch (a.M) {
    case 1: SWEEP(2, 2, false); break;
    case 2: SWEEP(2, 2, true); break;
    case 3: SWEEP(3, 2, true); break;
    case 4: SWEEP(4, 2, true); break;
    case 5: SWEEP(6, 2, false); break;
    case 6: SWEEP(6, 2, true); break;
    case 7: SWEEP(8, 2, false); break;
    default: SWEEP(8, 2, true); break;
    }
#undef SWEEP
}

}  // namespace

// Which policy kernels the context uses: 0 those of policy.hip, 1 .. 3 the instances here (3: not the backward sweep).
// Measured per step of a gradient call, policy.hip / here (N = 2048, L = 1024 unless said): hidden 64-64 at B = 256 (N = 512)
// 22.4 / 13.5 us, B = 2048 46.5 / 37.6, B = 8192 109 / 100, B = 32768 406 / 377, B = 65536 (16 to a sample) 678 / 614; one layer of
// 16 at B = 8192 100 / 96, B = 65536 630 / 583; 128-128 (N = 4096, L = 2048) at B = 4096 113 / 102, at B = 8192
// 188 / 183; 256-256 at B = 1024 55.6 / 48.0, B = 2048 67.1 / 61.0 (checkpointed 71.5 / 66.9), B = 4096 (N = 4096) 131.7 /
// 128.4 (checkpointed, 500 steps 127.1 / 123.2), forward pass with 16 trajectories per sample there 64.0 / 57.7.  Wider policies on
// larger batches fill the chip with 32 trajectories per workgroup, and fetching the weights twice as often costs what the
// shorter chain gives: N = 2048, B = 6144 256-256 118.0 / 120.4, 192-192 108.7 / 112.6, checkpointed 126.2 / 127.3 and 116.9 / 119.9,
// B = 8192 checkpointed 157.0 / 160.1, 128-128 127.3 / 116.3.  Above 2048 trajectories, checkpointed, 130 policies with one layer of 129 to 256
// units (H = 40): a second layer of up to 64 behind it 0.90 .. 0.99 times as fast as policy.hip (0.97 on average; 254-25 0.91, 139-50
// 0.99), of 65 to 128 1.00 on average, the narrow layer first 1.01 .. 1.10, two wide ones 1.02 .. 1.11, one layer 1.04 .. 1.15; not checkpointed,
// up to 64 behind it, 0.97 .. 1.02.  So the second layer sets the limit when checkpointed; both kernels give the same bits.
void bagel_plan_policy(bagel_ctx *c)
{
    int w = 0;
    for (int l = 1; l < c->n_layers; ++l) w = c->width[l] > w ? c->width[l] : w;
    c->p16 = w <= 64 ? 1 : (w <= 128 ? 2 : 3);
    const bool narrow_second = c->n_layers == 3 && c->width[2] <= 64;
    const int most = c->p16 == 3 ? (narrow_second && c->T_tape < c->dm.H ? 2048 : 4096) : 8192;
    const int tile = bagel_env_int("BAGEL_POLICY_TILE", 0);                // 16 or 32: always that one, otherwise by size
    if (tile == 32 || (tile != 16 && c->p16 != 1 && c->dm.B > most)) c->p16 = 0;
    c->pack16_floats = c->p16 ? make_pack(c).total() : 0;
}

hipError_t bagel_launch_pack_theta16(bagel_ctx *c, const float *theta)
{
    const pack16_args a = make_pack_args(c);
    hipLaunchKernelGGL(pack_theta16_kernel, dim3((a.p.total() + 255) / 256), dim3(256), 0, c->stream, a, theta);
    return hipGetLastError();
}

hipError_t bagel_launch_start16(bagel_ctx *c, const float *s0, const float *goals, float *states_out, bool tape, bool acts)
{
    tail16_args r = {};
    r.D = c->D; r.M = c->M; r.dg = c->dm.d_g;
    r.do_policy = 1;
    r.x_next = c->xbuf; r.lpt = c->lpt;
    r.tape_s_next = tape ? c->tape_s : nullptr;
    r.states_out_next = states_out;
    r.goals_next = goals; r.s0 = s0;
    return launch_tail(c, r, acts);
}

hipError_t bagel_launch_step_tail16(bagel_ctx *c, int t, int slot, int next_slot, bool jac, bool acts, bool write_tape_s,
                                    const float *goals, float *states_out, bool direct)
{
    const size_t B = c->dm.B;
    const bool has_next = t + 1 < c->dm.H && next_slot >= 0;
    tail16_args r = {};
    r.D = c->D; r.M = c->M; r.dg = c->dm.d_g;
    r.ngk = (c->nck + 3) / 4; r.ngl = (c->ncl + 3) / 4;
    r.ncomp = jac ? 1 + c->D : 1;
    r.cost_kind = c->dm.cost_kind; r.do_policy = has_next ? 1 : 0; r.direct = direct ? 1 : 0;
    r.sigma_r = c->dm.sigma_r;
    for (int j = 0; j < 8; ++j) { r.tracked[j] = c->dm.tracked[j]; r.q[j] = c->dm.q[j]; }
    r.amp = c->amp; r.part = c->part; r.lpt = c->lpt;
    r.x_cur = c->xbuf; r.x_next = c->xbuf_alt;
    r.tape_s_next = write_tape_s ? c->tape_s + (size_t)(t + 1) * c->dm.d_s * B : nullptr;
    r.states_out_next = states_out ? states_out + (size_t)(t + 1) * B * c->dm.d_s : nullptr;
    r.goals_t = goals + (size_t)t * B * c->dm.d_g;
    r.goals_next = has_next ? goals + (size_t)(t + 1) * B * c->dm.d_g : nullptr;
    r.jdst = (jac && direct) ? c->tape_J + (size_t)slot * c->M * c->D * B : nullptr;
    r.slot = has_next ? (size_t)next_slot : 0;
    return launch_tail(c, r, acts);
}

hipError_t bagel_launch_policy_replay16(bagel_ctx *c, int t0, int t1, const float *goals)
{
    replay16_args r;
    r.tape_s = c->tape_s; r.goals = goals; r.t0 = t0; r.dg = c->dm.d_g; r.n_slots = t1 - t0; r.per = 5;
    const dim3 grid((c->dm.B + PL - 1) / PL, (t1 - t0 + r.per - 1) / r.per);
    const policy16_args a = make_policy(c, true);
    const pack16 p = make_pack(c);
    if (c->p16 == 1) hipLaunchKernelGGL((policy_replay16_kernel<4, 1>), grid, dim3(256), 0, c->stream, r, a, p);
    else if (c->p16 == 2) hipLaunchKernelGGL((policy_replay16_kernel<8, 1>), grid, dim3(512), 0, c->stream, r, a, p);
    else hipLaunchKernelGGL((policy_replay16_kernel<8, 2>), grid, dim3(512), 0, c->stream, r, a, p);
    return hipGetLastError();
}

hipError_t bagel_launch_backward_sweep16(bagel_ctx *c, int t_lo, int t_hi, const float *goals, float *grad_s0)
{
    sweep16_args a;
    a.B = c->dm.B; a.nl = c->n_layers; a.ds = c->dm.d_s; a.da = c->dm.d_a; a.dg = c->dm.d_g; a.D = c->D; a.M = c->M;
    a.H = c->dm.H; a.t_hi = t_hi; a.t_lo = t_lo;
    for (int i = 0; i < 4; ++i) a.width[i] = c->width[i];
    for (int l = 0; l < 3; ++l) {
        a.tape_h[l] = l < c->n_layers ? c->tape_h[l] : nullptr;
        a.tape_d[l] = l < c->n_layers ? c->tape_d[l] : nullptr;
    }
    a.act_bound = c->dm.act_bound; a.cost_kind = c->dm.cost_kind; a.sigma_r = c->dm.sigma_r;
    // what dims.q holds past d_g is the caller's and may be anything.  (Left out by the host: with a branch in the kernel for
    // every component a gradient call at 64-64, B = 256 took 1387 us instead of 1376.)
    for (int j = 0; j < 8; ++j) { a.tracked[j] = c->dm.tracked[j]; a.q[j] = j < c->dm.d_g ? c->dm.q[j] : 0.0f; }
    a.pack = c->wpack16;
    // the Jacobian tape spans the whole horizon when the activation tape is kept per segment
    const bool per_segment = c->T_tape < c->dm.H;
    a.tape_a = c->tape_a; a.tape_s = c->tape_s;
    a.tape_J = c->tape_J + (per_segment ? (size_t)t_lo * c->M * c->D * c->dm.B : 0);
    a.goals = goals; a.lam = c->lam; a.grad_s0 = grad_s0;
    if (c->p16 == 1) launch_sweep<4, 1>(c, a);
    else launch_sweep<8, 1>(c, a);
    return hipGetLastError();
}
