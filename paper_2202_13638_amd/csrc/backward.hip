// The backward pass with its steps side by side.
//
// Of a backward sweep only the adjoint of the state is a chain from step to step, and that chain is linear.  With
// Pi_o = d (action o) / d (state), a policy's backward pass for a unit adjoint of one action, a step is
//   lam_i <- lam_i + sum_m C_im lam_m + (cost gradient)_i,      C_im = J_mi + sum_o Pi_oi J_m,(d_s + o),
// and everything else, the policy's layers above all, does not depend on lam (C) or only on the lam of its own step (the adjoints
// that the weight gradients are made of): it is done for all steps and trajectories at once, where it fills the chip.
//   policy_layers_kernel<.., false>  C and the cost gradients of every (step, trajectory)
//   adjoint_chain_kernel             lam through the steps, 16 lanes to a trajectory
//   policy_layers_kernel<.., true>   adjoints of the actions and hidden layers of every (step, trajectory), to their tapes
// A sweep by policy16.hip has the layers inside its chain, 1.3 to 2.2 us a step; here a step of the chain is a few products, and the
// rest is d_a + 1 passes through the layers at the rate of the matrix units.  64-64, M = 4, B = 256, 100 steps: the sweep 207 us; here
// 16.6 + 15.0 + 11.3; 8-8, M = 2, B = 100, 300 steps: 443; 15.9 + 29.6 + 7.3; 64-64, M = 4, B = 1024, 200 steps: 418; 82 + 26 + 66.
#include "policy16.h"

namespace {

struct layers_args {
    int B, nl, ds, da, dg, H, t_lo, columns, tiles;          // columns: steps x trajectories
    int M, D;
    int width[4];
    float act_bound, sigma_r;
    int cost_kind;
    int tracked[8];
    float q[8];
    const float *pack;
    const float *tape_h[3];
    float *tape_d[3];
    const float *tape_s, *tape_a, *tape_J, *goals;           // tape_J: slot 0 = step t_lo
    double *steps;                           // [step][B][d_s][d_s + 1]: C, then the cost gradient of the state the step starts from
    const double *lam;                       // [step][B][d_s]: the adjoint of the state the step ends in
};

// (1/B) d cost / d s_i for the state s (component k at s[k B]) and goal
__device__ __forceinline__ double cost_gradient(const float *s, size_t B, const float *goal, int i, int dg, const int (&tracked)[8],
                                                const float (&q)[8], int kind, float sigma_r)
{
    double e = 0.0, own = 0.0;
    for (int j = 0; j < dg; ++j) {
        const double r = (double)s[tracked[j] * B] - (double)goal[j];
        e += (double)q[j] * r * r;
        if (tracked[j] == i) own += (double)q[j] * r;
    }
    double factor = 2.0;
    if (kind == 1) {
        const double sr2 = (double)sigma_r * (double)sigma_r;
        factor = exp(-e / (2.0 * sr2)) / sr2;
    }
    return factor / (double)B * own;
}

// 16 columns, a column = a step of a trajectory, per tile; a workgroup takes tiles in turn with the weights in registers, as in
// backward_sweep16_kernel.  ADJOINT: from the state's adjoints to the adjoints of the actions and hidden layers, to their tapes.
// Otherwise from a unit adjoint of each action to Pi, from there to C, and the cost gradients.
template <int NW, bool ADJOINT>
__global__ __launch_bounds__(64 * NW) void policy_layers_kernel(layers_args a, pack16 p)
{
    using S = shape16<NW, 1>;
    constexpr int TT = S::TT, AS = S::AS;
    __shared__ __align__(16) float act[2][PL * AS], red[ADJOINT ? PL * HS : NW * PL * HS];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int j = lane & 15, g = lane >> 4, ug = (g & 1) << 2 | g >> 1;       // unit16(g, r) = ug + unit16(0, r)
    const int last = a.nl - 1;
    const size_t B = a.B;

    float w_top[2];
    f4v w_mid[1][TT], w_first[2];            // w_first: the two blocks of slice `wave`
#pragma unroll
    for (int s = 0; s < 2; ++s) w_top[s] = a.pack[p.b_top() + (wave * p.nsa + min(s, p.nsa - 1)) * 64 + lane];
    if (a.nl == 3) {
#pragma unroll
        for (int kb = 0; kb < TT; ++kb) w_mid[0][kb] = reinterpret_cast<const f4v *>(a.pack + p.b_mid())[(wave * TT + kb) * 64 + lane];
    }
    if (!ADJOINT) {
#pragma unroll
        for (int e = 0; e < 2; ++e) w_first[e] = reinterpret_cast<const f4v *>(a.pack + p.b_first())[min(2 * wave + e, TT - 1) * 64 + lane];
    }
    // tanh outputs of the wave's units of layer l for the lane's column
    auto units = [&](f4v &h, int l, int step, int b) {
        const int n = a.width[l];
        const float *hl = a.tape_h[l] + (size_t)step * n * B + b;
#pragma unroll
        for (int r = 0; r < 4; ++r) h[r] = load_pinned(hl + (size_t)min(16 * wave + ug + unit16(0, r), n - 1) * B);
    };
    auto column = [&](int tile, int &step, int &b) {
        const int i = min(tile * PL + j, a.columns - 1);
        step = i / a.B;
        b = i - step * a.B;
    };
    int step, b;
    column(blockIdx.x, step, b);
    f4v top, mid = {0.0f, 0.0f, 0.0f, 0.0f};
    units(top, last, step, b);
    if (a.nl == 3) units(mid, 1, step, b);
    for (int tile = blockIdx.x; tile < a.tiles; tile += gridDim.x) {
        const bool live = tile * PL + j < a.columns;
        const f4v h_top = top, h_mid = mid;
        const int step_now = step, b_now = b;
        column(min(tile + (int)gridDim.x, a.tiles - 1), step, b);           // the next tile's values are requested early
        units(top, last, step, b);
        if (a.nl == 3) units(mid, 1, step, b);
        f4v dl[1];
        auto derivative = [&](const f4v &h, int l, float *out) {            // delta_l = (W^T delta) (1 - h^2), to LDS (and its tape)
            const int n = a.width[l], u0 = 16 * wave + ug;
            float *dst = ADJOINT ? a.tape_d[l - 1] + ((size_t)step_now * n + u0) * B + b_now : nullptr;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int u = u0 + unit16(0, r);
                dl[0][r] *= 1.0f - h[r] * h[r];
                if (u >= n) dl[0][r] = 0.0f;
                else if (ADJOINT && live) dst[(size_t)unit16(0, r) * B] = dl[0][r];
            }
            if (!ADJOINT || l > 1) *reinterpret_cast<f4v *>(out + j * AS + 16 * wave + 4 * g) = dl[0];
        };
        const int row = tid >> 4;                                          // (column: tid % 16 = j)
        const float *J = a.tape_J + (size_t)step_now * a.M * a.D * B + b_now;
        // d action o / d (its layer's output): the bound's derivative
        auto slope = [&](int o) {
            if (a.act_bound <= 0.0f) return 1.0;
            const double th = (double)a.tape_a[((size_t)step_now * a.da + o) * B + b_now];
            return (double)a.act_bound * (1.0 - th * th);
        };
        if constexpr (ADJOINT) {
            if (row < a.da) {
                double u = 0.0;
                const double *lam = a.lam + ((size_t)step_now * B + b_now) * a.M;
                for (int m = 0; m < a.M; ++m) u += (double)J[(size_t)(m * a.D + a.ds + row) * B] * lam[m];
                const float d = (float)(u * slope(row));
                red[j * HS + row] = d;
                if (live) a.tape_d[last][((size_t)step_now * a.da + row) * B + b_now] = d;
            }
            __syncthreads();
            dl[0] = f4v{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int e = 0; e < 2; ++e)
                if (e < p.nsa) {
                    const int u = ug + unit16(0, e);
                    const float d = red[j * HS + u];
                    dl[0] = mfma16(w_top[e], u < a.da ? d : 0.0f, dl[0]);
                }
            derivative(h_top, last, act[0]);
            __syncthreads();
            if (a.nl == 3) {
                contract_wide<1, TT, AS>(dl, w_mid, act[0], lane, a.width[last], p.bs);
                derivative(h_mid, 1, act[1]);
            }
            // (act[0] is written again after the next tile's first barrier)
        } else {
            double C[8], cost = 0.0;
            const bool mine = row < a.ds;
            const int k = a.t_lo + step_now;                               // the step's first state
            if (mine) {
#pragma unroll
                for (int m = 0; m < 8; ++m) C[m] = (double)J[(size_t)(min(m, a.M - 1) * a.D + row) * B];
                if (k > 0)
                    cost = cost_gradient(a.tape_s + (size_t)k * a.ds * B + b_now, B, a.goals + ((size_t)(k - 1) * B + b_now) * a.dg, row, a.dg,
                                         a.tracked, a.q, a.cost_kind, a.sigma_r);
            }
            for (int o = 0; o < a.da; ++o) {
                dl[0] = f4v{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int e = 0; e < 2; ++e)
                    if (e < p.nsa) dl[0] = mfma16(w_top[e], ug + unit16(0, e) == o ? 1.0f : 0.0f, dl[0]);
                derivative(h_top, last, act[0]);
                __syncthreads();
                if (a.nl == 3) {
                    contract_wide<1, TT, AS>(dl, w_mid, act[0], lane, a.width[last], p.bs);
                    derivative(h_mid, 1, act[1]);
                    __syncthreads();
                }
                // adjoint of the policy input: one row tile, wave w takes slice w
                if (32 * wave < a.width[1]) {
                    const f4v z = contract_slice<TT, AS>(w_first, act[a.nl - 2], wave, lane);
#pragma unroll
                    for (int r = 0; r < 4; ++r) red[(wave * PL + j) * HS + ug + unit16(0, r)] = z[r];
                }
                __syncthreads();
                if (mine) {
                    float dh = red[j * HS + row];
                    for (int w = 1; 32 * w < a.width[1]; ++w) dh += red[(w * PL + j) * HS + row];
                    const double pi = (double)dh * slope(o);
#pragma unroll
                    for (int m = 0; m < 8; ++m) C[m] = fma(pi, (double)J[(size_t)(min(m, a.M - 1) * a.D + a.ds + o) * B], C[m]);
                }
                // (red is written again after at least one more barrier)
            }
            if (mine && live) {
                double *dst = a.steps + (((size_t)step_now * B + b_now) * a.M + row) * (a.M + 1);
#pragma unroll
                for (int m = 0; m < 8; ++m)
                    if (m < a.M) dst[m] = C[m];
                dst[a.M] = cost;
            }
        }
    }
}

constexpr int CHAIN_AHEAD = BAGEL_CHAIN_AHEAD;

struct chain_args {
    int B, dg, H, t_hi, t_lo;
    float sigma_r;
    int cost_kind;
    int tracked[8];
    float q[8];
    const double *steps;                     // [step][B][M][M + 1], CHAIN_AHEAD steps of anything in front
    const float *tape_s, *goals;
    double *lam_steps;                       // [step][B][M]
    double *lam;
    float *grad_s0;
};

// f(n, value of lane n of the row of 16 lanes) for n < N
template <int N, class F>
__device__ __forceinline__ void for_lanes(double v, F f)
{
    if constexpr (N > 0) {
        for_lanes<N - 1>(v, f);
        const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), 0x150 + N - 1, 0xf, 0xf, true);      // row_newbcast
        const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), 0x150 + N - 1, 0xf, 0xf, true);
        f(N - 1, __hiloint2double(hi, lo));
    }
}

// 16 lanes to a trajectory, the first M of them at work: lane i holds lam_i.  What bounds it is the trip to memory, so a step's
// row of C is requested DEPTH steps ahead: as far as the counter of outstanding requests goes.
template <int M>
__global__ __launch_bounds__(256) void adjoint_chain_kernel(chain_args a)
{
    constexpr int REQUESTS = M / 2 + 2, DEPTH = 56 / REQUESTS < CHAIN_AHEAD ? 56 / REQUESTS : CHAIN_AHEAD;
    const int i = threadIdx.x & 15, b = blockIdx.x * 16 + (threadIdx.x >> 4);
    if (i >= M || b >= a.B) return;
    const size_t B = a.B, stride = B * M * (M + 1);
    struct values {
        double r[M + 1];
    } v[DEPTH];
    const double *next = a.steps + ((size_t)(a.t_hi - 1 - a.t_lo) * B + b) * (M * (M + 1)) + i * (M + 1);
    auto request = [&](values &s) {          // one step after the other (CHAIN_AHEAD steps lie in front of the first)
#pragma unroll
        for (int m = 0; m <= M; ++m) s.r[m] = next[m];
        next -= stride;
    };
    double *out = a.lam_steps + ((size_t)(a.t_hi - 1 - a.t_lo) * B + b) * M + i;
    double lam = a.t_hi == a.H ? cost_gradient(a.tape_s + (size_t)a.H * M * B + b, B, a.goals + ((size_t)(a.H - 1) * B + b) * a.dg, i, a.dg, a.tracked,
                                               a.q, a.cost_kind, a.sigma_r)
                               : a.lam[(size_t)i * B + b];
#pragma unroll
    for (int k = 0; k < DEPTH; ++k) {
        request(v[k]);
        __builtin_amdgcn_sched_barrier(0);
    }
    auto step = [&](const values &s) {
        *out = lam;
        out -= B * M;
        double even = lam + s.r[M], odd = 0.0;
        for_lanes<M>(lam, [&](int m, double l) {
            if (m & 1) odd = fma(s.r[m], l, odd);
            else even = fma(s.r[m], l, even);
        });
        lam = even + odd;
    };
    int t = a.t_hi;
    for (; t - DEPTH >= a.t_lo; t -= DEPTH) {
#pragma unroll
        for (int k = 0; k < DEPTH; ++k) {
            step(v[k]);
            request(v[k]);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
#pragma unroll
    for (int k = 0; k < DEPTH; ++k)
        if (t - k > a.t_lo) step(v[k]);
    a.lam[(size_t)i * B + b] = lam;
    if (a.t_lo == 0 && a.grad_s0) a.grad_s0[(size_t)b * M + i] = (float)lam;
}

template <int NW, bool ADJOINT>
void launch_layers(bagel_ctx *c, const layers_args &a)
{
    // four workgroups of four waves, two of eight, to a compute unit
    const int most = 256 * (NW == 4 ? 4 : 2);
    hipLaunchKernelGGL((policy_layers_kernel<NW, ADJOINT>), dim3(a.tiles < most ? a.tiles : most), dim3(64 * NW), 0, c->stream, a, make_pack(c));
}

}  // namespace

// Whether the backward pass takes its steps side by side: where a sweep leaves the chip idle (it has 16 trajectories per workgroup and
// the layers inside the chain of steps) and there are steps enough for two launches more and, when checkpointing, for what the
// second stream no longer hides.  Measured on MI355X, sweep / here, calls with a small model (N = L = 64), in us:
//   M = 6, d_a = 2, 64-64, 64 steps: B = 16 305 / 189, 256 345 / 239, 768 688 / 617, 1024 905 / 848, 2048 1028 / 1036, 4096 1270 / 1452;
//   128-128: B = 256 447 / 309, 768 856 / 806, 1024 1092 / 1090, 2048 1354 / 1491;   M = 4, d_a = 1, 128-128: B = 1024 1036 / 972;
//   M = 6, d_a = 2, 64-64, B = 256: 16 steps 114 / 93, 8 steps 77 / 72, 4 steps 54 / 57;
//   64 steps in segments of 32 408 / 311, of 16 443 / 370, of 8 520 / 501; one layer of 64: of 16 335 / 313, of 8 406 / 409
//   (segments shorter than 16 steps are put together, see bagel_create).
// With two actions, which are two passes through the layers, the line lies where 128-128 no longer gains; narrower policies still do at 1024.
void bagel_plan_backward(bagel_ctx *c)
{
    const int want = bagel_env_int("BAGEL_BACKWARD", 0);                   // 1: sweep, 2: steps side by side, otherwise by size
    c->backward_parallel = false;
    if (!(c->p16 == 1 || c->p16 == 2) || c->dm.d_a > 2 || (int64_t)c->dm.H * c->dm.B > (1 << 30)) return;
    // (not by the checkpoint interval: gradients with and without checkpointing have the same bits)
    c->backward_parallel = want == 2 || (want != 1 && bagel_env_int("BAGEL_POLICY_TILE", 0) == 0 && c->dm.H >= 12 &&
                                         c->dm.B <= (c->dm.d_a == 1 ? 1024 : 768));
}

// The steps t_hi - 1 .. t_lo, at most backward_steps of them, of a segment that begins with the step t_seg
static hipError_t launch_steps(bagel_ctx *c, int t_seg, int t_lo, int t_hi, const float *goals, float *grad_s0)
{
    const size_t slot = (size_t)(t_lo - t_seg) * c->dm.B;
    double *const steps = c->adjoint_steps + (size_t)CHAIN_AHEAD * c->dm.B * c->M * (c->M + 1);
    layers_args a = {};
    a.B = c->dm.B; a.nl = c->n_layers; a.ds = c->dm.d_s; a.da = c->dm.d_a; a.dg = c->dm.d_g; a.H = c->dm.H; a.t_lo = t_lo;
    a.columns = (t_hi - t_lo) * c->dm.B;
    a.tiles = (a.columns + PL - 1) / PL;
    for (int i = 0; i < 4; ++i) a.width[i] = c->width[i];
    a.sigma_r = c->dm.sigma_r; a.cost_kind = c->dm.cost_kind;
    for (int l = 0; l < 3; ++l) {
        a.tape_h[l] = l < c->n_layers ? c->tape_h[l] + slot * c->width[l] : nullptr;
        a.tape_d[l] = l < c->n_layers ? c->tape_d[l] + slot * c->width[l + 1] : nullptr;
    }
    a.M = c->M; a.D = c->D; a.act_bound = c->dm.act_bound;
    a.pack = c->wpack16;
    a.tape_s = c->tape_s; a.tape_a = c->tape_a + slot * c->dm.d_a; a.goals = goals; a.steps = steps; a.lam = c->lam_steps;
    a.tape_J = c->tape_J + (size_t)t_lo * c->M * c->D * c->dm.B;           // (spans the whole horizon)
    chain_args k = {};
    for (int j = 0; j < 8; ++j) {
        a.tracked[j] = k.tracked[j] = c->dm.tracked[j];
        a.q[j] = k.q[j] = c->dm.q[j];
    }
    if (c->p16 == 1) launch_layers<4, false>(c, a);
    else launch_layers<8, false>(c, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;

    k.B = c->dm.B; k.dg = c->dm.d_g; k.H = c->dm.H; k.t_hi = t_hi; k.t_lo = t_lo;
    k.sigma_r = c->dm.sigma_r; k.cost_kind = c->dm.cost_kind;
    k.steps = steps; k.tape_s = c->tape_s; k.goals = goals;
    k.lam_steps = c->lam_steps; k.lam = c->lam; k.grad_s0 = grad_s0;
    const dim3 grid((c->dm.B + 15) / 16), block(256);
    switch (c->M) {
#define CHAIN(m) case m: hipLaunchKernelGGL(adjoint_chain_kernel<m>, grid, block, 0, c->stream, k); break;
        CHAIN(1) CHAIN(2) CHAIN(3) CHAIN(4) CHAIN(5) CHAIN(6) CHAIN(7) CHAIN(8)
#undef CHAIN
    default: return hipErrorInvalidValue;
    }
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (c->p16 == 1) launch_layers<4, true>(c, a);
    else launch_layers<8, true>(c, a);
    return hipGetLastError();
}

hipError_t bagel_launch_backward_parallel(bagel_ctx *c, int t_lo, int t_hi, const float *goals, float *grad_s0)
{
    for (int hi = t_hi; hi > t_lo; hi -= c->backward_steps) {
        const int lo = hi - c->backward_steps > t_lo ? hi - c->backward_steps : t_lo;
        const hipError_t e = launch_steps(c, t_lo, lo, hi, goals, grad_s0);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}
