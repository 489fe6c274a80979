// Re-layout of the model and of the per-sample streams into the form the step kernel reads.
//   Xs[m][n][0..D-1] = log2(e)/l_md^2 * X_nd,   Xs[m][n][D] = log2(alpha_m^2) - 1/2 sum_d Xs_mnd X_nd
//   Xn[m][n] = the same row with 6144 added to its last entry (rows of the step kernel's table form);
//   near_ok = 0 if a training point or a signal variance lies outside the range of that form
//   Os[m][l][0..D-1] = omega_mld / (2 pi),      Os[m][l][D] = phase_ml / (2 pi)   (revolutions)
//   Of[m][l/4][j][q][l%4] = (float) omega_ml,4q+j / (2 pi), zero for columns >= D: the same frequencies in the
//                           order of the matrix-core operand of the feature Jacobian (see gp_step.hip)
//   v4[m][n/4][s] = v[s][m][4(n/4) .. +3],      w4[m][l/4][s] likewise
// Rows past N (or L) are padding: they evaluate to a kernel value of zero (or a feature of one)
// and carry a zero weight, so they add nothing.  Everything is computed in float64 from the
// float32 inputs (eq. (4) hyper-parameters; random-feature frequencies and phases).
#include "bagel_internal.h"

namespace {

constexpr double LOG2E = 1.4426950408889634074;
constexpr double INV_TWO_PI = 0.15915494309189533577;

__global__ void set_flag_kernel(int *flag, int value) { flag[0] = value; }

struct model_args {
    const float *X, *ell, *sf2, *omega, *phase;
    double *Xs, *Xn, *Os, *A, *amp;
    float *Of;
    int *near_ok;
    int M, N, L, Np, Lp;
};

// Row i of the training points' tables of output m.  Every input is requested before the first is used: D is a template
// parameter for that (with a loop over a run-time D each column waited for its own loads, and so do the other parts below).
template <int D>
__device__ __forceinline__ void build_point_row(const model_args &t, int m, int i)
{
    const int N = t.N, Np = t.Np;
    if (i >= Np) return;
    double ell[D], a[D], xv[D];
    const double sf2 = (double)t.sf2[m];
#pragma unroll
    for (int d = 0; d < D; ++d) {
        ell[d] = (double)t.ell[m * D + d];
        xv[d] = (double)t.X[(size_t)(i < N ? i : N - 1) * D + d];
    }
    double row[D + 1], rown[D + 1];
    double c = log2(sf2);
#pragma unroll
    for (int d = 0; d < D; ++d) {
        a[d] = LOG2E / (ell[d] * ell[d]);
        rown[d] = row[d] = a[d] * xv[d];
        c -= 0.5 * a[d] * xv[d] * xv[d];
    }
    row[D] = c;
    rown[D] = c + 6144.0;
    // the table form needs |c_n| <= 250 and |log2 alpha^2| <= 20 (negated tests: NaN fails them)
    if (t.Xn && i < N) {
        const double la = log2(sf2);
        if (!(c >= -250.0) || !(la >= -20.0 && la <= 20.0)) t.near_ok[0] = 0;
    }
    const bool padding = i >= N;
    if (padding || c < -131072.0) {                  // c: outside the step kernel's range (see gp_step.hip), k = 0
#pragma unroll
        for (int d = 0; d < D; ++d) row[d] = 0.0;
        row[D] = -2000.0;
    }
    if (padding) {                                   // padding row of the table form: k = 1, weight 0
#pragma unroll
        for (int d = 0; d < D; ++d) rown[d] = 0.0;
        rown[D] = 6144.0;
    }
    double *__restrict__ to = t.Xs + ((size_t)m * Np + i) * (D + 1);
#pragma unroll
    for (int d = 0; d <= D; ++d) to[d] = row[d];
    if (t.Xn) {
        double *__restrict__ ton = t.Xn + ((size_t)m * Np + i) * (D + 1);
#pragma unroll
        for (int d = 0; d <= D; ++d) ton[d] = rown[d];
    }
    if (i == 0) {
#pragma unroll
        for (int d = 0; d < D; ++d) t.A[m * D + d] = a[d];
        t.amp[m] = sqrt(2.0 * sf2 / (double)t.L);
    }
}

// Row i of the features' tables of output m
template <int D>
__device__ __forceinline__ void build_feature_row(const model_args &t, int m, int i)
{
    constexpr int NQ = (D + 3) / 4;
    const int L = t.L, Lp = t.Lp;
    if (i >= Lp) return;
    const size_t from = (size_t)m * L + (i < L ? i : L - 1);
    float in[D + 1];
#pragma unroll
    for (int d = 0; d < D; ++d) in[d] = t.omega[from * D + d];
    in[D] = t.phase[from];
    double row[D + 1];
#pragma unroll
    for (int d = 0; d <= D; ++d) row[d] = i < L ? INV_TWO_PI * (double)in[d] : 0.0;
    double *__restrict__ to = t.Os + ((size_t)m * Lp + i) * (D + 1);
#pragma unroll
    for (int d = 0; d <= D; ++d) to[d] = row[d];
    float *__restrict__ tof = t.Of + ((size_t)m * (Lp / 4) + (i >> 2)) * 16 * NQ + (i & 3);
#pragma unroll
    for (int col = 0; col < 4 * NQ; ++col) tof[((col & 3) * NQ + (col >> 2)) * 4] = col < D ? (float)row[col < D ? col : 0] : 0.0f;
}

// One 64 x 64 block of a stream, src[S][M][n] -> dst[M][np/4][S] (float4 of four consecutive n, zero past n), through LDS so
// that both sides are contiguous: sample s0 + r, entries q0 ..
__device__ __forceinline__ void pack_block(const float *__restrict__ src, float4 *__restrict__ dst, int S, int M, int n, int np4, int m,
                                           int s0, int q0, float (*t)[65])
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    // a wave's 16 rows all requested before the first is waited for
    float in[16];
    const int col = min(q0 + lane, n - 1);
#pragma unroll
    for (int e = 0; e < 16; ++e) in[e] = src[((size_t)min(s0 + wave + 4 * e, S - 1) * M + m) * n + col];
#pragma unroll
    for (int e = 0; e < 16; ++e) t[wave + 4 * e][lane] = q0 + lane < n ? in[e] : 0.0f;
    __syncthreads();
#pragma unroll
    for (int q = wave; q < 16; q += 4)
        if (q0 / 4 + q < np4 && s0 + lane < S)
            dst[((size_t)m * np4 + q0 / 4 + q) * S + s0 + lane] =
                make_float4(t[lane][4 * q], t[lane][4 * q + 1], t[lane][4 * q + 2], t[lane][4 * q + 3]);
}

// What one call installs: blocks of the training points' and the features' rows, of the two streams and of the inputs, one after
// the other in the grid
struct install_args {
    model_args t;
    const float *v, *w, *x;
    float4 *v4, *w4;
    double *xbuf;
    int S, B;
    int point_blocks, feature_blocks, v_blocks, w_blocks;      // first four parts of the grid; the rest are inputs
};

// Bound: one trip to memory, little work (see build_point_row).  N = 512, L = 1024, 256 trajectories: 5.3 us, 8.2 before.
template <int D>
__global__ __launch_bounds__(256) void install_kernel(install_args a)
{
    __shared__ float t[64][65];
    int blk = blockIdx.x;
    const int M = a.t.M, sb = (a.S + 63) / 64;
    if (blk < a.point_blocks) {
        const int per = a.point_blocks / M;
        build_point_row<D>(a.t, blk / per, (blk % per) * 256 + threadIdx.x);
        return;
    }
    blk -= a.point_blocks;
    if (blk < a.feature_blocks) {
        const int per = a.feature_blocks / M;
        build_feature_row<D>(a.t, blk / per, (blk % per) * 256 + threadIdx.x);
        return;
    }
    blk -= a.feature_blocks;
    if (blk < a.v_blocks + a.w_blocks) {
        const bool is_v = blk < a.v_blocks;
        if (!is_v) blk -= a.v_blocks;
        const int n = is_v ? a.t.N : a.t.L, np4 = (is_v ? a.t.Np : a.t.Lp) / 4, qb = (np4 + 15) / 16;
        const int s = blk % sb, q = (blk / sb) % qb, m = blk / (sb * qb);
        pack_block(is_v ? a.v : a.w, is_v ? a.v4 : a.w4, a.S, M, n, np4, m, 64 * s, 64 * q, t);
        return;
    }
    blk -= a.v_blocks + a.w_blocks;
    const int b = blk * 256 + threadIdx.x;
    if (b < a.B) {
        float x[D];
#pragma unroll
        for (int d = 0; d < D; ++d) x[d] = a.x[(size_t)b * D + d];
#pragma unroll
        for (int d = 0; d < D; ++d) a.xbuf[(size_t)d * a.B + b] = (double)x[d];
    }
}

template <int D>
void launch_install(const install_args &a, int d, unsigned blocks, hipStream_t stream)
{
    if (d == D) hipLaunchKernelGGL(install_kernel<D>, dim3(blocks), dim3(256), 0, stream, a);
    else if constexpr (D < BAGEL_MAX_D) launch_install<D + 1>(a, d, blocks, stream);
}

}  // namespace

hipError_t bagel_launch_install(bagel_ctx *c, const float *X, const float *ell, const float *sf2, const float *omega,
                                const float *phase, const float *w, const float *v, const float *x)
{
    // near_ok starts at 1 and is cleared by any row outside the table form's range (contexts without the
    // table form have no Xn)
    if (c->Xn) hipLaunchKernelGGL(set_flag_kernel, dim3(1), dim3(1), 0, c->stream, c->near_ok, 1);
    install_args a;
    a.t = model_args{X, ell, sf2, omega, phase, c->Xs, c->Xn, c->Os, c->A, c->amp, c->Of, c->near_ok, c->M, c->dm.N, c->dm.L, c->Np,
                     c->Lp};
    a.v = v; a.w = w; a.x = x;
    a.v4 = c->v4; a.w4 = c->w4; a.xbuf = c->xbuf;
    a.S = c->dm.S; a.B = c->dm.B;
    const int64_t sb = (c->dm.S + 63) / 64;
    const int64_t pb = (int64_t)c->M * ((c->Np + 255) / 256), fb = omega ? (int64_t)c->M * ((c->Lp + 255) / 256) : 0;
    const int64_t vb = v ? c->M * sb * ((c->Np / 4 + 15) / 16) : 0, wb = w ? c->M * sb * ((c->Lp / 4 + 15) / 16) : 0;
    const int64_t xb = x ? (c->dm.B + 255) / 256 : 0;
    if (pb + fb + vb + wb + xb > 0x7fffffff) return hipErrorInvalidValue;
    a.point_blocks = (int)pb; a.feature_blocks = (int)fb; a.v_blocks = (int)vb; a.w_blocks = (int)wb;
    launch_install<2>(a, c->D, (unsigned)(pb + fb + vb + wb + xb), c->stream);
    return hipGetLastError();
}
