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
    int M, N, L, D, Np, Lp;
};

// rows i of the tables of output m
__device__ __forceinline__ void build_rows(const model_args &t, int m, int i)
{
    const float *__restrict__ X = t.X, *__restrict__ ell = t.ell, *__restrict__ sf2 = t.sf2, *__restrict__ omega = t.omega,
                *__restrict__ phase = t.phase;
    double *__restrict__ Xs = t.Xs, *__restrict__ Xn = t.Xn, *__restrict__ Os = t.Os, *__restrict__ A = t.A, *__restrict__ amp = t.amp;
    float *__restrict__ Of = t.Of;
    int *near_ok = t.near_ok;
    const int N = t.N, L = t.L, D = t.D, Np = t.Np, Lp = t.Lp;
    if (i < Np) {
        double *row = Xs + ((size_t)m * Np + i) * (D + 1);
        if (i < N) {
            double c = log2((double)sf2[m]);
            for (int d = 0; d < D; ++d) {
                const double l = (double)ell[m * D + d];
                const double a = LOG2E / (l * l);
                const double xv = (double)X[(size_t)i * D + d];
                row[d] = a * xv;
                c -= 0.5 * a * xv * xv;
            }
            row[D] = c;
            if (Xn) {
                double *rown = Xn + ((size_t)m * Np + i) * (D + 1);
                for (int d = 0; d < D; ++d) rown[d] = row[d];
                rown[D] = c + 6144.0;
                const double la = log2((double)sf2[m]);
                // the table form needs |c_n| <= 250 and |log2 alpha^2| <= 20 (negated tests: NaN fails them)
                if (!(c >= -250.0) || !(la >= -20.0 && la <= 20.0)) near_ok[0] = 0;
            }
            if (c < -131072.0) {                     // outside the step kernel's range (see gp_step.hip): k = 0
                for (int d = 0; d < D; ++d) row[d] = 0.0;
                row[D] = -2000.0;
            }
        } else {
            for (int d = 0; d < D; ++d) row[d] = 0.0;
            row[D] = -2000.0;
            if (Xn) {                                // padding row of the table form: k = 1, weight 0
                double *rown = Xn + ((size_t)m * Np + i) * (D + 1);
                for (int d = 0; d < D; ++d) rown[d] = 0.0;
                rown[D] = 6144.0;
            }
        }
    }
    if (omega && i < Lp) {
        double *row = Os + ((size_t)m * Lp + i) * (D + 1);
        if (i < L) {
            for (int d = 0; d < D; ++d) row[d] = INV_TWO_PI * (double)omega[((size_t)m * L + i) * D + d];
            row[D] = INV_TWO_PI * (double)phase[(size_t)m * L + i];
        } else {
            for (int d = 0; d <= D; ++d) row[d] = 0.0;
        }
        const int NQ = (D + 3) / 4;
        for (int col = 0; col < 4 * NQ; ++col) {
            const int qd = col >> 2, j = col & 3;
            Of[((((size_t)m * (Lp / 4) + (i >> 2)) * 4 + j) * NQ + qd) * 4 + (i & 3)] = col < D ? (float)row[col] : 0.0f;
        }
    }
    if (i < D) {
        const double l = (double)ell[m * D + i];
        A[m * D + i] = LOG2E / (l * l);
    }
    if (i == 0) amp[m] = sqrt(2.0 * (double)sf2[m] / (double)L);
}

// One 64 x 64 block of a stream, src[S][M][n] -> dst[M][np/4][S] (float4 of four consecutive n, zero past n), through LDS so
// that both sides are contiguous: sample s0 + r, entries q0 ..
__device__ __forceinline__ void pack_block(const float *__restrict__ src, float4 *__restrict__ dst, int S, int M, int n, int np4, int m,
                                           int s0, int q0, float (*t)[65])
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll 4
    for (int r = wave; r < 64; r += 4)
        t[r][lane] = (s0 + r < S && q0 + lane < n) ? src[((size_t)(s0 + r) * M + m) * n + q0 + lane] : 0.0f;
    __syncthreads();
    for (int q = wave; q < 16; q += 4)
        if (q0 / 4 + q < np4 && s0 + lane < S)
            dst[((size_t)m * np4 + q0 / 4 + q) * S + s0 + lane] =
                make_float4(t[lane][4 * q], t[lane][4 * q + 1], t[lane][4 * q + 2], t[lane][4 * q + 3]);
}

// What one call installs: blocks of the model tables, of the two streams and of the inputs, one after the other in the grid
struct install_args {
    model_args t;
    const float *v, *w, *x;
    float4 *v4, *w4;
    double *xbuf;
    int S, B;
    int model_blocks, v_blocks, w_blocks;        // first three parts of the grid; the rest are inputs
};

__global__ __launch_bounds__(256) void install_kernel(install_args a)
{
    __shared__ float t[64][65];
    int blk = blockIdx.x;
    const int M = a.t.M, sb = (a.S + 63) / 64;
    if (blk < a.model_blocks) {
        const int per = a.model_blocks / M;
        build_rows(a.t, blk / per, (blk % per) * 256 + threadIdx.x);
        return;
    }
    blk -= a.model_blocks;
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
    if (b < a.B)
        for (int d = 0; d < a.t.D; ++d) a.xbuf[(size_t)d * a.B + b] = (double)a.x[(size_t)b * a.t.D + d];
}

}  // namespace

hipError_t bagel_launch_install(bagel_ctx *c, const float *X, const float *ell, const float *sf2, const float *omega,
                                const float *phase, const float *w, const float *v, const float *x)
{
    // near_ok starts at 1 and is cleared by any row outside the table form's range (contexts without the
    // table form have no Xn)
    if (c->Xn) hipLaunchKernelGGL(set_flag_kernel, dim3(1), dim3(1), 0, c->stream, c->near_ok, 1);
    install_args a;
    a.t = model_args{X, ell, sf2, omega, phase, c->Xs, c->Xn, c->Os, c->A, c->amp, c->Of, c->near_ok, c->M, c->dm.N, c->dm.L, c->D,
                     c->Np, c->Lp};
    a.v = v; a.w = w; a.x = x;
    a.v4 = c->v4; a.w4 = c->w4; a.xbuf = c->xbuf;
    a.S = c->dm.S; a.B = c->dm.B;
    const int big = c->Np > c->Lp ? c->Np : c->Lp;
    const int64_t sb = (c->dm.S + 63) / 64;
    const int64_t model = (int64_t)c->M * ((big + 255) / 256);
    const int64_t vb = v ? c->M * sb * ((c->Np / 4 + 15) / 16) : 0, wb = w ? c->M * sb * ((c->Lp / 4 + 15) / 16) : 0;
    const int64_t xb = x ? (c->dm.B + 255) / 256 : 0;
    if (model + vb + wb + xb > 0x7fffffff) return hipErrorInvalidValue;
    a.model_blocks = (int)model; a.v_blocks = (int)vb; a.w_blocks = (int)wb;
    hipLaunchKernelGGL(install_kernel, dim3((unsigned)(model + vb + wb + xb)), dim3(256), 0, c->stream, a);
    return hipGetLastError();
}
