// Set-up of the two samplers and hyper-parameter learning: everything that needs K_hat = K + noise I
// (eq. (4), text below eq. (3)) factored.
//   bagel_prepare_impl            v_sm = K_hat_m^-1 (y_m - Phi_m w_sm - eps_sm) for every function sample and output
//                                 (Matheron update of a pathwise sample)
//   bagel_prepare_posterior_impl  K_hat_m^-1 and K_hat_m^-1 y_m (eq. (2), (3))
//   bagel_hyper_impl              log marginal likelihood and its gradient (eq. (5), (6)), Adam ascent on it
// Everything is float64 on the device: the condition number of K_hat is ~ signal/noise variance times N, far
// beyond float32.
//
// Layout.  Np = N rounded up to 64; the padding rows of K_hat are an identity block.  All GP outputs are worked on
// by the same launches (one more grid dimension): the chain of small dependent kernels of a factorisation
// is walked once instead of once per output.  Matrices of one output, row-major with row length Np:
//   K  the upper triangle of K_hat (whole 64 x 64 blocks), updated in place while it is factored;
//   U  the factor, K_hat = U^T U (L = U^T), block rows written as they are finished; with `mirror` also L below;
//   W  L^-1 (lower), V = W^T = U^-1 (upper): the 64 x 64 diagonal blocks come out of the factorisation of the
//      diagonal block, larger blocks from them level by level (triangular_inverse).  Where whole inverses are formed V
//      takes the place of K (inverse_bytes).
// With U, V and W at hand every product has its contraction index as the row of both operands (f64_tile.h).
//
// Factorisation (struct solver): recursive halving with products as deep as half the range down to ranges of
// four blocks; inside a range one launch per block column (chol_step_kernel), which also factors and inverts the
// next diagonal block.  A triangular solve with 64 unknowns is a product with the inverted diagonal block.
#include <math.h>
#include <stdio.h>

#include <new>

#include "bagel_internal.h"
#include "f64_tile.h"

namespace {

constexpr int NB = 64;           // block of the factorisation
constexpr int RB = 4;            // blocks per range that is worked on block column by block column
using f64_tile::d4v;

// ---- K_hat --------------------------------------------------------------------------------------------------
// Hyper-parameters of output m, either as they are (log = 0: ell[M][D], sf2[M], sn2[M]) or as logarithms
// (log = 1: ell[M][D + 2] = log l_1 .. log l_D, log alpha^2, log sigma_n^2).
struct hyper_ptr {
    const float *ell, *sf2, *sn2;
    int log;
};
__device__ __forceinline__ double inv_length(const hyper_ptr &h, int m, int D, int d)
{
    return h.log ? exp(-(double)h.ell[m * (D + 2) + d]) : 1.0 / (double)h.ell[m * D + d];
}
__device__ __forceinline__ double signal_variance(const hyper_ptr &h, int m, int D)
{
    return h.log ? exp((double)h.ell[m * (D + 2) + D]) : (double)h.sf2[m];
}
__device__ __forceinline__ double noise_variance(const hyper_ptr &h, int m, int D)
{
    return h.log ? exp((double)h.ell[m * (D + 2) + D + 1]) : (double)h.sn2[m];
}

// Block (blockIdx.y, blockIdx.x) of the upper triangle of K_hat for output m0 + blockIdx.z; identity on the padding.
// Thread = column and 16 of the rows; inputs of the block's rows and columns in LDS.
__global__ __launch_bounds__(256) void build_khat_kernel(const float *__restrict__ X, hyper_ptr h, double *__restrict__ K,
                                                         size_t sK, int N, int Np, int D, int m0)
{
    if (blockIdx.x < blockIdx.y) return;
    __shared__ double xr[NB][BAGEL_MAX_D], xc[BAGEL_MAX_D][NB + 1], il[BAGEL_MAX_D];
    const int m = m0 + blockIdx.z, i0 = blockIdx.y * NB, j0 = blockIdx.x * NB;
    for (int e = threadIdx.x; e < NB * D; e += 256) {
        const int r = e / D, d = e - r * D;
        xr[r][d] = i0 + r < N ? (double)X[(size_t)(i0 + r) * D + d] : 0.0;
        xc[d][r] = j0 + r < N ? (double)X[(size_t)(j0 + r) * D + d] : 0.0;
    }
    if ((int)threadIdx.x < D) il[threadIdx.x] = inv_length(h, m, D, threadIdx.x);
    __syncthreads();
    const int c = threadIdx.x & 63, r0 = 16 * (threadIdx.x >> 6);
    double s[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) s[e] = 0.0;
    for (int d = 0; d < D; ++d) {
        const double x = xc[d][c], l = il[d];
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const double t = (xr[r0 + e][d] - x) * l;
            s[e] = fma(t, t, s[e]);
        }
    }
    const double sf2 = signal_variance(h, m, D), sn2 = noise_variance(h, m, D);
    double *dst = K + blockIdx.z * sK + (size_t)(i0 + r0) * Np + j0 + c;
    const int j = j0 + c;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        const int i = i0 + r0 + e;
        double v = i == j ? 1.0 : 0.0;
        if (i < N && j < N) {
            v = sf2 * exp(-0.5 * s[e]);
            if (i == j) v += sn2;
        }
        dst[(size_t)e * Np] = v;
    }
}

// ---- diagonal block: factor and inverse -------------------------------------------------------------------------
// Where the 64 x 64 ... 256 x 256 diagonal blocks of V and W are: the whole matrix, or (compact) only the diagonal
// blocks of 256, one after the other.
struct tri_matrix {
    double *p;
    size_t ld;                   // 0: compact, rows of 256
    size_t stride;               // per output
    __device__ __forceinline__ size_t row_length() const { return ld ? ld : (size_t)(NB * RB); }
    __device__ __forceinline__ double *at(int o, int r, int c) const
    {
        return p + o * stride + (ld ? (size_t)r * ld + c : (size_t)r * (NB * RB) + (c & (NB * RB - 1)));
    }
};

struct factor_args {
    double *K, *U;
    size_t sK, sU;               // per output
    tri_matrix V, W;
    double *diag;                // [outputs][Np]: diagonal of U
    int *flag;                   // [outputs]: 0, or 1 + first pivot that is not positive
    int Np;
};

constexpr int LT = 66;           // LDS row stride of a block: even, so that pairs stay aligned

// 1/sqrt(d): hardware estimate (residual 1 - d y^2 below 1.1e-7, measured) and one third-order correction, which
// leaves less than the rounding
__device__ __forceinline__ double inv_sqrt(double d)
{
    const double y = __builtin_amdgcn_rsq(d);
    const double e = fma(-(d * y), y, 1.0);
    return fma(y * e, fma(0.375, e, 0.5), y);
}

// Broadcasts within a row of 16 lanes, as an operand modifier: no trip through LDS or scalar registers.  The hardware
// wants two wait states between the write of a register and its use as such an operand, which the compiler does
// not insert for assembly: every block below starts with them (8 cycles, so the blocks are long).
template <int A, int B>
__device__ __forceinline__ void row_broadcasts(double u, double v, double &a, double &b, double &c)
{
    asm("s_nop 1\n\tv_mov_b64_dpp %0, %3 row_newbcast:%5 row_mask:0xf bank_mask:0xf\n\t"
        "v_mov_b64_dpp %1, %3 row_newbcast:%6 row_mask:0xf bank_mask:0xf\n\t"
        "v_mov_b64_dpp %2, %4 row_newbcast:%6 row_mask:0xf bank_mask:0xf"
        : "=&v"(a), "=&v"(b), "=&v"(c)
        : "v"(u), "v"(v), "n"(A), "n"(B));
}
// x0 -= (v of lane C) * f + (w of lane C) * g, x1 the same with lane C + 1
template <int C>
__device__ __forceinline__ void pivot_update2(double &x0, double &x1, double v, double f, double w, double g)
{
    asm("s_nop 1\n\tv_fmac_f64_dpp %0, -%2, %3 row_newbcast:%6 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %1, -%2, %3 row_newbcast:%7 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, -%4, %5 row_newbcast:%6 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %1, -%4, %5 row_newbcast:%7 row_mask:0xf bank_mask:0xf"
        : "+v"(x0), "+v"(x1)
        : "v"(v), "v"(f), "v"(w), "v"(g), "n"(C), "n"(C + 1));
}
// the same for four columns
template <int C>
__device__ __forceinline__ void pivot_update4(double &x0, double &x1, double &x2, double &x3, double v, double f, double w, double g)
{
    asm("s_nop 1\n\tv_fmac_f64_dpp %0, -%4, %5 row_newbcast:%8 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %1, -%4, %5 row_newbcast:%9 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %2, -%4, %5 row_newbcast:%10 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %3, -%4, %5 row_newbcast:%11 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, -%6, %7 row_newbcast:%8 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %1, -%6, %7 row_newbcast:%9 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %2, -%6, %7 row_newbcast:%10 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %3, -%6, %7 row_newbcast:%11 row_mask:0xf bank_mask:0xf"
        : "+v"(x0), "+v"(x1), "+v"(x2), "+v"(x3)
        : "v"(v), "v"(f), "v"(w), "v"(g), "n"(C), "n"(C + 1), "n"(C + 2), "n"(C + 3));
}
// u and v with the even rows' values in the odd rows too
__device__ __forceinline__ void even_rows(double &u, double &v)
{
    int a = __double2loint(u), b = __double2hiint(u), c = __double2loint(v), d = __double2hiint(v);
    int a1 = a, b1 = b, c1 = c, d1 = d;
    asm("s_nop 1\n\tv_permlane16_swap_b32 %0, %4\n\tv_permlane16_swap_b32 %1, %5\n\t"
        "v_permlane16_swap_b32 %2, %6\n\tv_permlane16_swap_b32 %3, %7"
        : "+v"(a), "+v"(b), "+v"(c), "+v"(d), "+v"(a1), "+v"(b1), "+v"(c1), "+v"(d1));
    u = __hiloint2double(b, a);
    v = __hiloint2double(d, c);
}

// Columns J and J + 1 of the factorisation of a 16 x 16 block, right-looking, and of the inverse of the factor.  Lane
// i of an even row of 16 lanes holds row i of the block in y, lane i of an odd one column i of the identity: what
// a step does to the rows below the pivots, y[c] -= L[c][J] y[J], is also the step of the forward substitution.
// Entries of the block above the diagonal hold nothing and feed nothing.
// Two columns at a time, because the time is the chain of dependent operations from pivot to pivot: with the 2 x 2
// pivot block [a b; b c] and det = a c - b^2, the second pivot's 1/sqrt(c - b^2/a) is a / sqrt(a det), which
// does not wait for 1/sqrt(a).  A pivot that is not positive leaves NaN on the diagonal.
template <int J, int C>
__device__ __forceinline__ void pivot_update(double (&y)[16], double l1, double l2)
{
    if constexpr (C + 4 <= 16) {
        pivot_update4<C>(y[C], y[C + 1], y[C + 2], y[C + 3], l1, y[J], l2, y[J + 1]);
        pivot_update<J, C + 4>(y, l1, l2);
    } else if constexpr (C < 16) {
        pivot_update2<C>(y[C], y[C + 1], l1, y[J], l2, y[J + 1]);
    }
}
template <int J>
__device__ __forceinline__ void pivot_columns(double (&y)[16])
{
    double u = y[J], v = y[J + 1], a, b, c;
    even_rows(u, v);                                                     // the block's two columns, in every row
    row_broadcasts<J, J + 1>(u, v, a, b, c);
    const double det = fma(a, c, -(b * b));
    const double r1 = inv_sqrt(a), r2 = a * inv_sqrt(a * det);
    const double b1 = b * r1;                                            // L[J + 1][J]
    const double l1 = u * r1, l2 = fma(-b1, l1, v) * r2;
    y[J] *= r1;
    y[J + 1] = fma(-b1, y[J], y[J + 1]) * r2;
    pivot_update<J, J + 2>(y, l1, l2);
    if constexpr (J + 2 < 16) pivot_columns<J + 2>(y);
}

// The 16 x 16 diagonal block at T, factored in place, its inverse to Wl; one wave (its two halves do the same)
__device__ __forceinline__ void factor16(double *T, double *Wl, int *flag, int pivot0)
{
    const int lane = threadIdx.x & 63, i = lane & 15;
    const bool block = (lane & 16) == 0;
    double y[16];
#pragma unroll
    for (int c = 0; c < 16; ++c) {
        const double t = T[i * LT + c];
        y[c] = block ? t : (c == i ? 1.0 : 0.0);
    }
    pivot_columns<0>(y);
    if (lane < 16) {
#pragma unroll
        for (int c = 0; c < 16; c += 2)
            *reinterpret_cast<double2 *>(T + i * LT + c) = make_double2(c <= i ? y[c] : 0.0, c + 1 <= i ? y[c + 1] : 0.0);
    } else if (lane < 32) {
#pragma unroll
        for (int c = 0; c < 16; ++c) Wl[c * LT + i] = y[c];
    }
    const unsigned long long bad = __ballot(lane < 16 && !(T[i * (LT + 1)] > 0.0));
    if (bad && lane == 0) atomicCAS(flag, 0, pivot0 + __ffsll(bad));
}

// D[16 x 16] tile of a product of 16 x 16 blocks in LDS: acc += a(i, k) b(k, j), a = A[i][k], b given by rows or by
// columns (transposed)
template <bool NEG, bool BT>
__device__ __forceinline__ d4v block16(d4v acc, const double *A, const double *B)
{
    const int lane = threadIdx.x & 63, i = lane & 15, g = lane >> 4;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        const double a = A[i * LT + g + 4 * s];
        const double b = BT ? B[i * LT + g + 4 * s] : B[(g + 4 * s) * LT + i];
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(NEG ? -a : a, b, acc, 0, 0, 0);
    }
    return acc;
}
// the same with the second operand in accumulator layout (rows g + 4 s of the lane's column): no exchange needed
template <bool NEG>
__device__ __forceinline__ d4v block16_reg(d4v acc, const double *A, const d4v &b)
{
    const int lane = threadIdx.x & 63, i = lane & 15, g = lane >> 4;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        const double a = A[i * LT + g + 4 * s];
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(NEG ? -a : a, b[s], acc, 0, 0, 0);
    }
    return acc;
}
__device__ __forceinline__ d4v load16(const double *C)
{
    const int lane = threadIdx.x & 63, j = lane & 15, g = lane >> 4;
    d4v v;
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = C[(g + 4 * r) * LT + j];
    return v;
}
__device__ __forceinline__ void store16(double *C, const d4v &v)
{
    const int lane = threadIdx.x & 63, j = lane & 15, g = lane >> 4;
#pragma unroll
    for (int r = 0; r < 4; ++r) C[(g + 4 * r) * LT + j] = v[r];
}

// What panel p adds to U, V and W: rows 16 p .. of U and W, columns 16 p .. of V; by waves first .. first + count - 1
__device__ __forceinline__ void emit_panel(const factor_args &f, int o, int k, int p, const double *T, const double *Wl, int first,
                                           int count)
{
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) - first;
    double *Ug = f.U + o * f.sU + (size_t)(NB * k) * f.Np + NB * k;
    const size_t ldv = f.V.row_length();
    double *Vg = f.V.at(o, NB * k, NB * k), *Wg = f.W.at(o, NB * k, NB * k);
    for (int e = wave; e < 16; e += count) {
        const int r = 16 * p + e;
        Ug[(size_t)r * f.Np + lane] = lane >= r ? T[lane * LT + r] : 0.0;
        Wg[(size_t)r * ldv + lane] = lane <= r ? Wl[r * LT + lane] : 0.0;
        const int vr = 4 * e + (lane >> 4), vc = 16 * p + (lane & 15);
        Vg[(size_t)vr * ldv + vc] = vr <= vc ? Wl[vc * LT + vr] : 0.0;
        if (lane == r) f.diag[(size_t)o * f.Np + NB * k + r] = T[r * LT + r];
    }
}

// Diagonal block k of output o, in T (LDS, [64][LT], lower triangle used): its factor to U (upper form) and
// `diag`, the inverse of the factor to W and V.  Wl: LDS of the same size.  256 threads; T is overwritten.
// Four panels of 16 columns.  Wave 0 factors and inverts the panel's 16 x 16 diagonal block; the blocks below it
// are products with that inverse, one wave each; then wave 0 updates the next diagonal block and goes on with it
// while the other waves update the blocks to the right, carry the inverse of the whole block along (wave 1 + j its
// block column j: W(p, j) = -W(p, p) S, S = sum_q L(p, q) W(q, j)) and write out what is finished.
// Bound: the chain of 32 pairs of pivots (4100 cycles per 16 columns, over half of the time): a launch for one block
// takes 14 us (21 us with the broadcasts through scalar registers, the inverse after the factor).
__device__ __forceinline__ void factor_diagonal(const factor_args &f, int o, int k, double *T, double *Wl)
{
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const d4v zero = {0.0, 0.0, 0.0, 0.0};
    const int j = wave - 1;                                  // block column of the inverse
    auto L = [&](int bi, int bj) { return T + 16 * bi * LT + 16 * bj; };
    auto W = [&](int bi, int bj) { return Wl + 16 * bi * LT + 16 * bj; };
    d4v S = zero;
    if (wave == 0) factor16(L(0, 0), W(0, 0), f.flag + o, NB * k);
#pragma unroll 1
    for (int p = 0; p < 4; ++p) {
        __syncthreads();                                     // block p of the diagonal and its inverse are there
        if (wave < 3 - p) {
            double *C = L(p + 1 + wave, p);
            store16(C, block16<false, true>(zero, C, W(p, p)));
        }
        if (j >= 0 && j < p) store16(W(p, j), block16_reg<true>(zero, W(p, p), S));
        __syncthreads();
        if (p == 3) break;
        if (wave == 0) {
            store16(L(p + 1, p + 1), block16<true, true>(load16(L(p + 1, p + 1)), L(p + 1, p), L(p + 1, p)));
            factor16(L(p + 1, p + 1), W(p + 1, p + 1), f.flag + o, NB * k + 16 * (p + 1));
        } else {
            // the other blocks (bi, bj), p < bj <= bi, numbered column by column from the second of the first column
            const int n = 3 - p, count = n * (n + 1) / 2;
            for (int t = wave; t < count; t += 3) {
                int bj = 0, left = t;
                while (left >= n - bj) left -= n - bj++;
                const int bi = p + 1 + bj + left;
                bj += p + 1;
                store16(L(bi, bj), block16<true, true>(load16(L(bi, bj)), L(bi, p), L(bj, p)));
            }
            S = zero;
            for (int q = j; q <= p; ++q) S = block16<false, false>(S, L(p + 1, q), W(q, j));
            emit_panel(f, o, k, p, T, Wl, 1, 3);
        }
    }
    emit_panel(f, o, k, 3, T, Wl, 0, 4);
}

// First diagonal block of a range, for every output (blockIdx.x)
__global__ __launch_bounds__(256) void factor_diagonal_kernel(factor_args f, int k)
{
    __shared__ __align__(16) double T[NB * LT], Wl[NB * LT];
    const int o = blockIdx.x;
    const double *src = f.K + o * f.sK + (size_t)(NB * k) * f.Np + NB * k;
    // row r of the upper triangle is column r of the lower one; all loads before the first use
    const int c = threadIdx.x & 63, r0 = threadIdx.x >> 6;
    double v[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) v[e] = src[(size_t)(r0 + 4 * e) * f.Np + c];
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        const int r = r0 + 4 * e;
        if (c >= r) T[c * LT + r] = v[e];
        if (c > r) T[r * LT + c] = 0.0;
    }
    __syncthreads();
    factor_diagonal(f, o, k, T, Wl);
}

// ---- one block column of the factorisation ------------------------------------------------------------------------
// 64 x 64 block of a row-major matrix to LDS, rows of 64, by direct loads (two rows per wave and instruction)
__device__ __forceinline__ void block_to_lds(const double *src, size_t ld, unsigned lds)
{
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const unsigned off = 16u * (unsigned)(lane & 31) + (unsigned)(lane >> 5) * (unsigned)(ld * 8);
#pragma unroll
    for (int e = 0; e < 8; ++e)
        f64_tile::load_row_to_lds(src + (size_t)(2 * wave + 8 * e) * ld, off, lds + 1024u * (unsigned)wave + 4096u * e);
}

// acc = sum_c A[c][i] B[c][j] over 64 rows in LDS (rows of 64), in the accumulator layout of f64_tile
__device__ __forceinline__ void lds_product(f64_tile::accumulators<64> &acc, const double *A, const double *B)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const double *pa = A + (lane >> 4) * NB + (wave >> 1) * 32 + 2 * (lane & 15);
    const double *pb = B + (lane >> 4) * NB + (wave & 1) * 32 + 2 * (lane & 15);
    f64_tile::clear(acc);
#pragma unroll
    for (int s = 0; s < 16; ++s) {
        const double2 a = *reinterpret_cast<const double2 *>(pa + 4 * s * NB), b = *reinterpret_cast<const double2 *>(pb + 4 * s * NB);
        acc.v[0][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, b.x, acc.v[0][0], 0, 0, 0);
        acc.v[0][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, b.y, acc.v[0][1], 0, 0, 0);
        acc.v[1][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.y, b.x, acc.v[1][0], 0, 0, 0);
        acc.v[1][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.y, b.y, acc.v[1][1], 0, 0, 0);
    }
}

// Block column j = k + 1 + blockIdx.x of output blockIdx.y, with block row k factored on the diagonal:
//   U_kj = L_kk^-1 K_kj, and for the rows i of the range (k < i < k_end, i <= j): K_ij -= U_ki^T U_kj.
// U_ki is computed again by every column that needs it (at most three extra products of 64 x 64 x 64 per workgroup)
// instead of waiting for another launch.  The workgroup of the next diagonal block goes on to factor it.
// Bound: the chain of launches: 2 products and the diagonal block, 16 us per block column for all outputs together,
// where three launches per column and output took 50.
constexpr size_t STEP_LDS = (size_t)4 * NB * NB * sizeof(double);
static_assert(2 * NB * LT <= 4 * NB * NB, "the diagonal block and its inverse take the place of the blocks");
__global__ __launch_bounds__(256) void chol_step_kernel(factor_args f, int k, int k_end)
{
    extern __shared__ __align__(16) double lds[];
    double *Vb = lds, *Jb = lds + NB * NB, *Ib = lds + 2 * NB * NB;       // Ib: two blocks
    const unsigned base = (unsigned)(size_t)(__attribute__((address_space(3))) double *)lds;
    constexpr unsigned BLK = NB * NB * 8;
    const int o = blockIdx.y, j = k + 1 + blockIdx.x;
    const size_t Np = f.Np;
    double *Krow = f.K + o * f.sK + (size_t)(NB * k) * Np;               // block row k of K
    block_to_lds(f.V.at(o, NB * k, NB * k), f.V.row_length(), base);
    block_to_lds(Krow + NB * j, Np, base + BLK);
    const int i_last = j < k_end ? j : k_end - 1;                        // rows k + 1 .. i_last of this column
    if (k + 1 < j && k + 1 <= i_last) block_to_lds(Krow + NB * (k + 1), Np, base + 2 * BLK);
    f64_tile::wait_loads_at_most<0>();
    __syncthreads();
    const f64_tile::lane_pos pos = f64_tile::lane_position<64>();
    f64_tile::accumulators<64> acc;
    lds_product(acc, Vb, Jb);
    __syncthreads();
    double *Urow = f.U + o * f.sU + (size_t)(NB * k) * Np + NB * j;
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int row = pos.row0 + e + 8 * r;
            const double2 v = make_double2(acc.v[e][0][r], acc.v[e][1][r]);
            *reinterpret_cast<double2 *>(Jb + row * NB + pos.col0) = v;
            *reinterpret_cast<double2 *>(Urow + (size_t)row * Np + pos.col0) = v;
        }
    __syncthreads();
    for (int i = k + 1; i <= i_last; ++i) {
        const int s = (i - k - 1) & 1;
        const double *Ui = Jb;
        if (i < j) {
            double *Is = Ib + s * NB * NB;
            // the next row's block goes to the other buffer, which was last read before the barriers above
            if (i + 1 < j && i + 1 <= i_last) block_to_lds(Krow + NB * (i + 1), Np, base + (2 + (s ^ 1)) * BLK);
            lds_product(acc, Vb, Is);
            __syncthreads();
#pragma unroll
            for (int e = 0; e < 2; ++e)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    *reinterpret_cast<double2 *>(Is + (pos.row0 + e + 8 * r) * NB + pos.col0) =
                        make_double2(acc.v[e][0][r], acc.v[e][1][r]);
            __syncthreads();
            Ui = Is;
        }
        double *C = f.K + o * f.sK + (size_t)(NB * i) * Np + NB * j;
        double2 cv[2][4];
#pragma unroll
        for (int e = 0; e < 2; ++e)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                cv[e][r] = *reinterpret_cast<const double2 *>(C + (size_t)(pos.row0 + e + 8 * r) * Np + pos.col0);
        lds_product(acc, Ui, Jb);
        const bool next = i == j && j == k + 1;                          // the next diagonal block: stays here
        if (next) __syncthreads();                                       // (every wave is done with the blocks it overwrites)
#pragma unroll
        for (int e = 0; e < 2; ++e)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = pos.row0 + e + 8 * r;
                const double2 v = make_double2(cv[e][r].x - acc.v[e][0][r], cv[e][r].y - acc.v[e][1][r]);
                if (next) {                                              // upper entry (row, col) is lower entry (col, row)
                    double *T = lds;
                    if (pos.col0 >= row) T[pos.col0 * LT + row] = v.x;
                    if (pos.col0 + 1 >= row) T[(pos.col0 + 1) * LT + row] = v.y;
                    if (pos.col0 > row) T[row * LT + pos.col0] = 0.0;
                    if (pos.col0 + 1 > row) T[row * LT + pos.col0 + 1] = 0.0;
                } else {
                    *reinterpret_cast<double2 *>(C + (size_t)row * Np + pos.col0) = v;
                }
            }
        f64_tile::wait_loads_at_most<0>();                               // the next row's block, if requested, has landed
        __syncthreads();
        if (next) factor_diagonal(f, o, j, lds, lds + NB * LT);
    }
}

// ---- products -----------------------------------------------------------------------------------------------------
// C (ni x nj) -= or = sum_k A[k][i] B[k][j] for every output (blockIdx.z); upper: tiles that lie below the diagonal
// of C are left out (ni <= nj), and the others are numbered row by row, the outputs of a tile one after the other (blockIdx.x).  Workgroups
// go to the eight chiplets in turn: with a grid of all tiles, a chiplet had whole columns and so up to 1.4 times its share
// of the tiles (16 x 16 tiles of 64, K = 1024, four outputs: 167 us, 104 so).
struct gemm_args {
    const double *A, *B;
    double *C;
    size_t lda, ldb, ldc, sA, sB, sC;
    int ni, nj, K;
    int subtract, upper, outputs;            // outputs: set by gemm()
};

template <int T>
__device__ __forceinline__ void upper_tile(const gemm_args &g, int &i, int &j, int &o)
{
    const int columns = (g.nj + T - 1) / T;
    int t = blockIdx.x / g.outputs, row = 0;
    o = blockIdx.x - t * g.outputs;
    while (t >= columns - row) t -= columns - row++;
    i = row;
    j = row + t;
}

template <int T>
__global__ __launch_bounds__(256, T == 128 ? 2 : 3) void gemm_kernel(gemm_args g)
{
    __shared__ __align__(16) double lds[f64_tile::shape<T>::LDS_DOUBLES];
    int ti = blockIdx.y, tj = blockIdx.x, o = blockIdx.z;
    if (g.upper) upper_tile<T>(g, ti, tj, o);
    const int i0 = ti * T, j0 = tj * T;
    f64_tile::accumulators<T> acc;
    f64_tile::clear(acc);
    f64_tile::product<T>(acc, lds, i0, j0, g.ni, g.nj, g.K, g.A + o * g.sA, g.lda, g.B + o * g.sB, g.ldb);
    const f64_tile::lane_pos pos = f64_tile::lane_position<T>();
    constexpr int H = f64_tile::shape<T>::H;
    double *C = g.C + o * g.sC;
#pragma unroll
    for (int x = 0; x < 2 * H; ++x)
#pragma unroll
        for (int h = 0; h < H; ++h)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int gi = i0 + pos.row0 + 32 * (x >> 1) + (x & 1) + 8 * r, gj = j0 + pos.col0 + 32 * h;
                if (gi < g.ni && gj < g.nj) {
                    double2 *dst = reinterpret_cast<double2 *>(C + (size_t)gi * g.ldc + gj);
                    double2 v = make_double2(acc.v[x][2 * h][r], acc.v[x][2 * h + 1][r]);
                    if (g.subtract) {
                        const double2 c = *dst;
                        v = make_double2(c.x - v.x, c.y - v.y);
                    }
                    *dst = v;
                }
            }
}

template <int T>
void launch_gemm(hipStream_t st, const gemm_args &g, long ti, long tj)
{
    const dim3 grid = g.upper ? dim3((ti * tj - ti * (ti - 1) / 2) * g.outputs) : dim3(tj, ti, g.outputs);
    hipLaunchKernelGGL(gemm_kernel<T>, grid, dim3(256), 0, st, g);
}

void gemm(hipStream_t st, int outputs, gemm_args g)
{
    if (g.ni <= 0 || g.nj <= 0 || g.K <= 0) return;
    g.outputs = outputs;
    const long ti = (g.ni + 127) / 128, tj = (g.nj + 127) / 128;
    const long tiles = outputs * (g.upper ? ti * tj - ti * (ti - 1) / 2 : ti * tj);
    if (f64_tile::whole_passes(tiles)) launch_gemm<128>(st, g, ti, tj);
    else launch_gemm<64>(st, g, (g.ni + 63) / 64, (g.nj + 63) / 64);
}

// ---- inverse of the factor -----------------------------------------------------------------------------------------
// One level: in pairs of neighbouring diagonal blocks of h (64-blocks each; the second of the last pair may be
// shorter), with U = [U11 U12; 0 U22], V = U^-1, W = V^T and the diagonal blocks of V and W known,
//   first launch   T[j][i] = sum_c U12[c][j] W11[c][i]            (T = (W11 ... )^T, c >= i)
//   second launch  W21[j][i] = - sum_c V22[c][j] T[c][i] = V12[i][j]  (c <= j)
// blockIdx.y = output * pairs + pair; T goes to the lower triangle of K.  Every level is two launches for all pairs and
// outputs: log2(N / 64) of them instead of a chain of N / 64 block solves.  The sums differ in length: blockIdx.z counts from
// the longest to the shortest, so that these fill the end of the launch and every chiplet has some of each (top level
// of N = 2048, four outputs: 134 and 110 us for the two, 81 and 84 so).
struct level_args {
    const double *U;
    double *T;
    size_t sU, sT;
    tri_matrix V, W;
    int Np, h, pairs;
};

template <bool SECOND>
__global__ __launch_bounds__(256, 3) void inverse_level_kernel(level_args a)
{
    __shared__ __align__(16) double lds[f64_tile::shape<64>::LDS_DOUBLES];
    const int o = blockIdx.y / a.pairs, p = blockIdx.y - o * a.pairs;
    const int r1 = 2 * p * a.h * NB, r2 = r1 + a.h * NB;                     // first rows of the two blocks
    const int n2 = min(a.h * NB, a.Np - r2);
    // row of block 2 and column of block 1: the first product is the longer the smaller i0, the second the larger j0
    const int j0 = NB * (SECOND ? a.h - 1 - (int)blockIdx.z : (int)blockIdx.x), i0 = NB * (SECOND ? blockIdx.x : blockIdx.z);
    if (j0 >= n2) return;
    const size_t Np = a.Np;
    f64_tile::accumulators<64> acc;
    f64_tile::clear(acc);
    const double *U12 = a.U + o * a.sU + (size_t)r1 * Np + r2;
    double *T = a.T + o * a.sT + (size_t)r2 * Np + r1;
    const size_t ldv = a.V.row_length();
    if (!SECOND)
        f64_tile::product<64>(acc, lds, j0, i0, n2, a.h * NB, a.h * NB - i0, U12 + (size_t)i0 * Np, Np,
                              a.W.at(o, r1, r1) + (size_t)i0 * ldv, ldv);
    else
        f64_tile::product<64>(acc, lds, j0, i0, n2, a.h * NB, j0 + NB, a.V.at(o, r2, r2), ldv, T, Np);
    const f64_tile::lane_pos pos = f64_tile::lane_position<64>();
    double *W21 = a.W.at(o, r2, r1) + (size_t)j0 * ldv + i0, *V12 = a.V.at(o, r1, r2) + (size_t)i0 * ldv + j0;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int row = pos.row0 + 8 * r;                                    // rows row, row + 1; columns col0, col0 + 1
        if (!SECOND) {
#pragma unroll
            for (int e = 0; e < 2; ++e)
                *reinterpret_cast<double2 *>(T + (size_t)(j0 + row + e) * Np + i0 + pos.col0) =
                    make_double2(acc.v[e][0][r], acc.v[e][1][r]);
        } else {
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                *reinterpret_cast<double2 *>(W21 + (size_t)(row + e) * ldv + pos.col0) =
                    make_double2(-acc.v[e][0][r], -acc.v[e][1][r]);
                *reinterpret_cast<double2 *>(V12 + (size_t)(pos.col0 + e) * ldv + row) =
                    make_double2(-acc.v[0][e][r], -acc.v[1][e][r]);
            }
        }
    }
}

// U's blocks above the diagonal, transposed, to their places below it
__global__ __launch_bounds__(256) void mirror_factor_kernel(double *__restrict__ U, size_t sU, int Np)
{
    if (blockIdx.x <= blockIdx.y) return;
    __shared__ double t[NB][NB + 1];
    double *src = U + blockIdx.z * sU + (size_t)(blockIdx.y * NB) * Np + blockIdx.x * NB;
    double *dst = U + blockIdx.z * sU + (size_t)(blockIdx.x * NB) * Np + blockIdx.y * NB;
    const int c = threadIdx.x & 63;
    for (int r = threadIdx.x >> 6; r < NB; r += 4) t[r][c] = src[(size_t)r * Np + c];
    __syncthreads();
    for (int r = threadIdx.x >> 6; r < NB; r += 4) dst[(size_t)r * Np + c] = t[c][r];
}

struct solver {
    hipStream_t st;
    factor_args f;
    int nb, outputs;             // 64-blocks per row, outputs worked on

    static int half(int w) { return (w / RB + 1) / 2 * RB; }     // first part of a split, a whole number of ranges

    // block columns [k, k + w) of the factor (block rows of U), for all columns to the right
    void factor(int k, int w)
    {
        if (w > RB) {
            const int h = half(w), r = NB * (k + h);
            factor(k, h);
            const double *P = f.U + (size_t)(NB * k) * f.Np + r;
            gemm_args g = {P, P, f.K + (size_t)r * f.Np + r, (size_t)f.Np, (size_t)f.Np, (size_t)f.Np, f.sU, f.sU, f.sK,
                           NB * (w - h), f.Np - r, NB * h, 1, 1};
            gemm(st, outputs, g);
            factor(k + h, w - h);
            return;
        }
        hipLaunchKernelGGL(factor_diagonal_kernel, dim3(outputs), dim3(256), 0, st, f, k);
        for (int kk = k; kk < k + w && kk + 1 < nb; ++kk)
            hipLaunchKernelGGL(chol_step_kernel, dim3(nb - kk - 1, outputs), dim3(256), STEP_LDS, st, f, kk, k + w);
    }

    // V and W inside diagonal blocks of `size` 64-blocks (K's lower triangle is the work space)
    void triangular_inverse(int size)
    {
        for (int h = 1; h < size && h < nb; h *= 2) {
            const int pairs = (nb + h - 1) / (2 * h);
            level_args a = {f.U, f.K, f.sU, f.sK, f.V, f.W, f.Np, h, pairs};
            const dim3 grid(h, outputs * pairs, h);
            hipLaunchKernelGGL(inverse_level_kernel<false>, grid, dim3(256), 0, st, a);
            hipLaunchKernelGGL(inverse_level_kernel<true>, grid, dim3(256), 0, st, a);
        }
    }

    // right-hand sides of all outputs: [Np][ld] each, `stride` apart
    struct rhs {
        double *p;
        size_t stride, ld;
        double *row(int r) const { return p + (size_t)r * ld; }
    };

    // One range of unknowns [64 k, 64 (k + w)), w <= RB: out = W in (forward: the rows of V are the columns of W) or V in
    void solve_range(bool fwd, int k, int w, const rhs &in, const rhs &out)
    {
        const tri_matrix &M = fwd ? f.V : f.W;
        gemm_args g = {M.p + (size_t)(NB * k) * (NB * RB), in.row(NB * k), out.row(NB * k), (size_t)(NB * RB), in.ld, out.ld,
                       M.stride, in.stride, out.stride, NB * w, (int)in.ld, NB * w, 0, 0};
        gemm(st, outputs, g);
    }

    // Z = L^-1 R on the unknowns of blocks [k, k + w); R's rows below are updated by the caller.  R is used up.
    void forward(int k, int w, const rhs &R, const rhs &Z)
    {
        if (w <= RB) return solve_range(true, k, w, R, Z);
        const int h = half(w), r = NB * (k + h);
        forward(k, h, R, Z);
        gemm_args g = {f.U + (size_t)(NB * k) * f.Np + r, Z.row(NB * k), R.row(r), (size_t)f.Np, Z.ld, R.ld,
                       f.sU, Z.stride, R.stride, NB * (w - h), (int)R.ld, NB * h, 1, 0};
        gemm(st, outputs, g);
        forward(k + h, w - h, R, Z);
    }

    // X = L^-T Z likewise, from the last block up (needs the mirrored factor)
    void backward(int k, int w, const rhs &Z, const rhs &X)
    {
        if (w <= RB) return solve_range(false, k, w, Z, X);
        const int h = half(w), r = NB * (k + h);
        backward(k + h, w - h, Z, X);
        gemm_args g = {f.U + (size_t)r * f.Np + NB * k, X.row(r), Z.row(NB * k), (size_t)f.Np, X.ld, Z.ld,
                       f.sU, X.stride, Z.stride, NB * h, (int)Z.ld, NB * (w - h), 1, 0};
        gemm(st, outputs, g);
        backward(k, h, Z, X);
    }
};

// ---- K_hat^-1 ------------------------------------------------------------------------------------------------------
// out[i] = sum_j A[i][j] v[j] for a triangular matrix of whole 64-blocks (upper: j >= 64 (i / 64), lower: j up to the
// block's end), one wave per row, the lanes' sums added by a fixed butterfly.  v: float y[N] (zero past N) or
// double.  Grid (Np / 4, outputs).
__global__ __launch_bounds__(256) void triangle_times_vector_kernel(tri_matrix A, int upper, const float *__restrict__ yf,
                                                                    const double *__restrict__ v, double *__restrict__ out, int N,
                                                                    int Np, int m0)
{
    const int lane = threadIdx.x & 63, o = blockIdx.y;
    const int i = blockIdx.x * 4 + (threadIdx.x >> 6);
    const int j0 = upper ? i / NB * NB : 0, j1 = upper ? Np : i / NB * NB + NB;
    const double *row = A.at(o, i, 0);
    double s = 0.0;
    for (int j = j0 + lane; j < j1; j += 64)
        s += row[j] * (yf ? (j < N ? (double)yf[(size_t)(m0 + o) * N + j] : 0.0) : v[(size_t)o * Np + j]);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
    if (lane == 0) out[(size_t)o * Np + i] = s;
}

// Lower tile t = (bi, bj), bj <= bi, of the 64-blocks, numbered row by row: the tiles with the longest sums come first
__device__ __forceinline__ void lower_tile(int t, int &bi, int &bj)
{
    bi = (int)((sqrtf(8.0f * (float)t + 1.0f) - 1.0f) * 0.5f);
    while ((bi + 1) * (bi + 2) / 2 <= t) ++bi;
    while (bi * (bi + 1) / 2 > t) --bi;
    bj = t - bi * (bi + 1) / 2;
}

// Block (bi, bj) of K_hat^-1 = W^T W: entry (i, j) sums over k >= 64 bi
__device__ __forceinline__ void inverse_tile(f64_tile::accumulators<64> &acc, double *lds, const tri_matrix &W, int o, int Np,
                                             int bi, int bj)
{
    const double *Wk = W.at(o, NB * bi, 0);
    f64_tile::clear(acc);
    f64_tile::product<64>(acc, lds, NB * bi, NB * bj, Np, Np, Np - NB * bi, Wk, W.ld, Wk, W.ld);
}

// K_hat^-1, both triangles (the posterior cache); the outputs of a tile one after the other (see hyper_grad_tiles_kernel)
__global__ __launch_bounds__(256, 3) void inverse_store_kernel(tri_matrix W, double *__restrict__ Kinv, int Np, int outputs)
{
    __shared__ __align__(16) double lds[f64_tile::shape<64>::LDS_DOUBLES];
    const int tile = blockIdx.x / outputs, o = blockIdx.x - tile * outputs;
    int bi, bj;
    lower_tile(tile, bi, bj);
    f64_tile::accumulators<64> acc;
    inverse_tile(acc, lds, W, o, Np, bi, bj);
    const f64_tile::lane_pos pos = f64_tile::lane_position<64>();
    double *Ko = Kinv + (size_t)o * Np * Np;
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int row = NB * bi + pos.row0 + 8 * r, col = NB * bj + pos.col0;
            *reinterpret_cast<double2 *>(Ko + (size_t)(row + e) * Np + col) = make_double2(acc.v[e][0][r], acc.v[e][1][r]);
            if (bi != bj)
                *reinterpret_cast<double2 *>(Ko + (size_t)(col + e) * Np + row) = make_double2(acc.v[0][e][r], acc.v[1][e][r]);
        }
}

// ---- hyper-parameter learning ----------------------------------------------------------------------------------------
// fixed-order sum of one value per thread over a workgroup of 256 (result valid in thread 0)
__device__ __forceinline__ double block_sum_256(double v, double *sh)
{
    sh[threadIdx.x] = v;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) sh[threadIdx.x] += sh[threadIdx.x + s];
        __syncthreads();
    }
    return sh[0];
}

// lml = -1/2 y^T K_hat^-1 y - sum_i log U_ii - N/2 log(2 pi), with y^T K_hat^-1 y = |z|^2, z = L^-1 y; one workgroup per output
__global__ __launch_bounds__(256) void hyper_lml_kernel(const double *__restrict__ diag, const double *__restrict__ z,
                                                        int N, int Np, float *__restrict__ lml_out)
{
    __shared__ double sh[256];
    const int o = blockIdx.x;
    double ld = 0.0, quad = 0.0;
    for (int i = threadIdx.x; i < Np; i += 256) {
        const double zi = z[(size_t)o * Np + i];
        ld += log(diag[(size_t)o * Np + i]);
        quad += zi * zi;
    }
    const double ld_tot = block_sum_256(ld, sh);
    __syncthreads();
    const double q_tot = block_sum_256(quad, sh);
    if (threadIdx.x == 0) lml_out[o] = (float)(-0.5 * q_tot - ld_tot - 0.5 * (double)N * 1.8378770664093453);
}

// Tile of sum_ij (a_i a_j - Kinv_ij) dK_hat_ij / dphi_c for c = 0 .. D+1 -> partial[o][tile][D+2] (eq. (6) with
// dK/dlog l_d = K (x_d - x'_d)^2 / l_d^2, dK/dlog alpha^2 = K, dK_hat/dlog sigma_n^2 = sigma_n^2 I).  The tile of
// K_hat^-1 is formed here and never written: only these sums of it are needed.  Tiles off the diagonal count
// twice.  The sums are added over a lane's entries, the lanes (fixed butterfly) and the four waves in order.
// The outputs of a tile come one after the other, so that the longest sums of all outputs are started first and the launch ends
// with the shortest (N = 2048, four outputs: output after output 270 us, so 238).
// Three workgroups per compute unit as long as the sums fit their 168 registers: beyond D = 13 they do not, and D = 16 kept 93
// in scratch memory (a call at N = 2048, 8 outputs: 2930 us, 2620 with two workgroups).
template <int D>
__global__ __launch_bounds__(256, D <= 13 ? 3 : 2) void hyper_grad_tiles_kernel(const float *__restrict__ X, const float *__restrict__ log_hyp,
                                                                  tri_matrix W, const double *__restrict__ alpha,
                                                                  double *__restrict__ partial, int N, int Np, int m0, int outputs)
{
    constexpr int LQ = NB + 1, NEED = NB * LQ + 2 * NB * (D + 1) + 4 * (D + 2);
    constexpr int HAVE = f64_tile::shape<64>::LDS_DOUBLES;
    __shared__ __align__(16) double lds[NEED > HAVE ? NEED : HAVE];
    const int tile = blockIdx.x / outputs, o = blockIdx.x - tile * outputs;
    int bi, bj;
    lower_tile(tile, bi, bj);
    f64_tile::accumulators<64> acc;
    inverse_tile(acc, lds, W, o, Np, bi, bj);
    // the tile, and inputs and alpha of its rows and columns, into the LDS the product is done with: thread = column
    // and 16 rows from here on, in a loop that needs few registers
    double *Q = lds, *xr = lds + NB * LQ, *xc = xr + NB * (D + 1), *sums = xc + NB * (D + 1);
    const f64_tile::lane_pos pos = f64_tile::lane_position<64>();
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y)
#pragma unroll
            for (int r = 0; r < 4; ++r) Q[(pos.row0 + x + 8 * r) * LQ + pos.col0 + y] = acc.v[x][y][r];
    const float *lh = log_hyp + (size_t)(m0 + o) * (D + 2);
    for (int e = threadIdx.x; e < 2 * NB * (D + 1); e += 256) {
        const int q = e / (D + 1), d = e - q * (D + 1);
        const int n = q < NB ? NB * bi + q : NB * bj + q - NB;
        xr[e] = n < N ? (d < D ? (double)X[(size_t)n * D + d] : alpha[(size_t)o * Np + n]) : 0.0;
    }
    double il[D];
#pragma unroll
    for (int d = 0; d < D; ++d) il[d] = exp(-(double)lh[d]);
    const double sf2 = exp((double)lh[D]), sn2 = exp((double)lh[D + 1]);
    __syncthreads();
    const int cl = threadIdx.x & 63, r0 = 16 * (threadIdx.x >> 6);
    const int j = NB * bj + cl;
    double xj[D + 1], s[D + 2];
#pragma unroll
    for (int d = 0; d <= D; ++d) xj[d] = xc[cl * (D + 1) + d];
#pragma unroll
    for (int c = 0; c < D + 2; ++c) s[c] = 0.0;
#pragma unroll 2
    for (int r = r0; r < r0 + 16; ++r) {
        const double *ri = xr + r * (D + 1);
        const int i = NB * bi + r;
        double q = 0.0, t2[D];
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const double t = (ri[d] - xj[d]) * il[d];
            t2[d] = t * t;
            q += t2[d];
        }
        double w = ri[D] * xj[D] - Q[r * LQ + cl];
        w = (i < N && j < N) ? w : 0.0;
        const double wk = w * sf2 * exp(-0.5 * q);
#pragma unroll
        for (int d = 0; d < D; ++d) s[d] += wk * t2[d];
        s[D] += wk;
        s[D + 1] += i == j ? w : 0.0;
    }
    s[D + 1] *= sn2;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int c = 0; c < D + 2; ++c) {
        double v = s[c];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
        if (lane == 0) sums[wave * (D + 2) + c] = v;
    }
    __syncthreads();
    const int c = threadIdx.x;
    if (c < D + 2) {
        const double tot = ((sums[c] + sums[(D + 2) + c]) + sums[2 * (D + 2) + c]) + sums[3 * (D + 2) + c];
        partial[((size_t)o * (gridDim.x / outputs) + tile) * (D + 2) + c] = bi == bj ? tot : 2.0 * tot;
    }
}

// grad[c] = 1/2 sum over the tiles; neg_scaled[c] = -grad[c] / N for the Adam update.  One workgroup per hyper-parameter
// and output: thread t adds tiles t, t + 256, ... in order, then a fixed tree over the threads.
__global__ __launch_bounds__(256) void hyper_grad_final_kernel(const double *__restrict__ partial, int tiles, int N, int H2,
                                                               float *__restrict__ grad, float *__restrict__ neg_scaled)
{
    __shared__ double sh[256];
    const int c = blockIdx.x, o = blockIdx.y;
    double s = 0.0;
    for (int i = threadIdx.x; i < tiles; i += 256) s += partial[((size_t)o * tiles + i) * H2 + c];
    s = 0.5 * block_sum_256(s, sh);
    if (threadIdx.x == 0) {
        if (grad) grad[o * H2 + c] = (float)s;
        if (neg_scaled) neg_scaled[o * H2 + c] = (float)(-s / (double)N);
    }
}

// ---- right-hand sides of the sample set-up ---------------------------------------------------------------------------
// PhiT[l][n] = sqrt(2 sf2 / L) cos(omega_l . X_n + phase_l); zero for l >= L (padding of the contraction) and n >= N.
// Grid (Np / 64, Lp / 4, outputs): lane = training point, wave = feature.
__global__ __launch_bounds__(256) void build_phi_kernel(const float *__restrict__ X, const float *__restrict__ omega,
                                                        const float *__restrict__ phase, hyper_ptr h, double *__restrict__ PhiT,
                                                        size_t s_phi, int N, int Np, int L, int D, int m0)
{
    const int m = m0 + blockIdx.z;
    const int n = blockIdx.x * 64 + (threadIdx.x & 63), l = blockIdx.y * 4 + (threadIdx.x >> 6);
    double val = 0.0;
    if (n < N && l < L) {
        const float *om = omega + ((size_t)m * L + l) * D;
        double z = (double)phase[(size_t)m * L + l];
        for (int d = 0; d < D; ++d) z += (double)om[d] * (double)X[(size_t)n * D + d];
        val = sqrt(2.0 * signal_variance(h, m, D) / (double)L) * cos(z);
    }
    PhiT[blockIdx.z * s_phi + (size_t)l * Np + n] = val;
}

// dst[o][q][s] = (y_m ? y_m[q] : 0) +- src[s][m][q] in float64 (plus without y, minus with), zero outside q < n, s < S:
// 64 x 64 blocks through LDS so that both sides are contiguous.  Grid (Sp / 64, rows / 64, outputs).
__global__ __launch_bounds__(256) void transpose_in_kernel(const float *__restrict__ src, const float *__restrict__ y,
                                                           double *__restrict__ dst, size_t s_dst, int n, int S, int Sp, int M,
                                                           int m0)
{
    __shared__ float t[64][65];
    const int m = m0 + blockIdx.z, s0 = blockIdx.x * 64, q0 = blockIdx.y * 64;
    const int lane = threadIdx.x & 63;
    for (int r = threadIdx.x >> 6; r < 64; r += 4)
        t[r][lane] = (s0 + r < S && q0 + lane < n) ? src[((size_t)(s0 + r) * M + m) * n + q0 + lane] : 0.0f;
    __syncthreads();
    for (int r = threadIdx.x >> 6; r < 64; r += 4) {
        const int q = q0 + r, s = s0 + lane;
        double v = (double)t[lane][r];
        if (y) v = (q < n && s < S) ? (double)y[(size_t)m * n + q] - v : 0.0;
        dst[blockIdx.z * s_dst + (size_t)q * Sp + s] = v;
    }
}

// V[n][s] (float64) -> the packed stream v4[m][n4][s] (zero past N) and v_out[s][m][n], both float32, through LDS.
// Grid (ceil(S / 64), ceil(Npk / 64), outputs); Npk: rows of the packed stream, which may be more than Np.
__global__ __launch_bounds__(256) void emit_v_kernel(const double *__restrict__ V, size_t s_v, int Sp, float *__restrict__ v_out,
                                                     float4 *__restrict__ v4, int N, int Npk, int S, int M, int m0)
{
    __shared__ float t[64][65];
    const int m = m0 + blockIdx.z, s0 = blockIdx.x * 64, n0 = blockIdx.y * 64;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int r = wave; r < 64; r += 4)
        t[r][lane] = n0 + r < N ? (float)V[blockIdx.z * s_v + (size_t)(n0 + r) * Sp + s0 + lane] : 0.0f;
    __syncthreads();
    for (int q = wave; q < 16; q += 4)
        if (n0 + 4 * q < Npk && s0 + lane < S)
            v4[((size_t)m * (Npk / 4) + (n0 >> 2) + q) * S + s0 + lane] =
                make_float4(t[4 * q][lane], t[4 * q + 1][lane], t[4 * q + 2][lane], t[4 * q + 3][lane]);
    if (v_out && n0 + lane < N)
        for (int r = wave; r < 64 && s0 + r < S; r += 4) v_out[((size_t)(s0 + r) * M + m) * N + n0 + lane] = t[lane][r];
}

// ---- work space --------------------------------------------------------------------------------------------------------
// What the set-up calls need beyond the context's own buffers: one device allocation that their float64 work
// space is carved from.  It is made by the first set-up call, grown when a later call needs more, kept for the
// next call (a caller's own loop over bagel_hyper_lml_grad, or a redraw of the samples with
// bagel_prepare_samples every few policy updates, allocates nothing after its first pass) and released by
// bagel_destroy.
struct setup_scratch {
    char *arena = nullptr;
    size_t arena_bytes = 0;
    bool limited = false;        // memory for all outputs at once could not be had: an arena that fits one is kept
    bool lds_raised = false;     // the dynamic-LDS limit of chol_step_kernel has been raised on this context's device
};

constexpr size_t ARENA_ALIGN = 256;
size_t arena_round(size_t bytes) { return (bytes + ARENA_ALIGN - 1) / ARENA_ALIGN * ARENA_ALIGN; }

// At least shared_bytes + n * output_bytes of device memory, n = number of outputs worked on by one launch: all
// of them (at most setup_outputs), fewer if the memory for that many cannot be had (one must fit).  The stream is idle when the arena is
// replaced: every set-up call ends with a synchronisation.
hipError_t setup_reserve(bagel_ctx *c, size_t output_bytes, size_t shared_bytes, setup_scratch **out, int *n_outputs)
{
    setup_scratch *sc = static_cast<setup_scratch *>(c->setup);
    if (!sc) {
        sc = new (std::nothrow) setup_scratch();
        if (!sc) return hipErrorOutOfMemory;
        c->setup = sc;
    }
    *out = sc;
    if (!sc->lds_raised) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&chol_step_kernel),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)STEP_LDS);
        if (e != hipSuccess) return e;
        sc->lds_raised = true;
    }
    output_bytes = arena_round(output_bytes);
    shared_bytes = arena_round(shared_bytes);
    const size_t M = (size_t)(c->M < c->setup_outputs ? c->M : c->setup_outputs);
    auto fit = [&]() { return sc->arena_bytes < shared_bytes ? (size_t)0 : (sc->arena_bytes - shared_bytes) / output_bytes; };
    if (fit() < M && !(sc->limited && fit() >= 1)) {
        (void)hipStreamSynchronize(c->stream);
        if (sc->arena) {
            (void)hipFree(sc->arena);
            c->bytes -= (int64_t)sc->arena_bytes;
            sc->arena = nullptr;
            sc->arena_bytes = 0;
        }
        hipError_t e = hipErrorOutOfMemory;
        for (size_t n = M; n >= 1; --n) {
            const size_t need = shared_bytes + n * output_bytes;
            e = hipMalloc((void **)&sc->arena, need);
            if (e == hipSuccess) {
                sc->arena_bytes = need;
                sc->limited = n < M;
                c->bytes += (int64_t)need;
                break;
            }
            sc->arena = nullptr;
            (void)hipGetLastError();
        }
        if (e != hipSuccess) return e;
    }
    *n_outputs = (int)(fit() < M ? fit() : M);
    return hipSuccess;
}

// consecutive pieces of the arena
struct arena_cursor {
    char *p;
    template <class T>
    T *take(size_t count)
    {
        T *r = reinterpret_cast<T *>(p);
        p += arena_round(count * sizeof(T));
        return r;
    }
};

// K_hat of outputs m0 .. m0 + s.outputs - 1 built and factored
void build_and_factor(solver &s, const float *X, const hyper_ptr &h, int N, int D, int m0)
{
    hipLaunchKernelGGL(build_khat_kernel, dim3(s.nb, s.nb, s.outputs), dim3(256), 0, s.st, X, h, s.f.K, s.f.sK, N, s.f.Np, D, m0);
    s.factor(0, s.nb);
}

__global__ void clear_flags_kernel(int *flag, int n)
{
    if ((int)threadIdx.x < n) flag[threadIdx.x] = 0;
}

// The first failure among the outputs of the flags, as (output, pivot); output -1: none.  Synchronises.
hipError_t read_flags(hipStream_t st, const int *flag, int M, int *output, int *pivot)
{
    int h[BAGEL_MAX_STATE];
    *output = -1;
    hipError_t e = hipMemcpyAsync(h, flag, (size_t)M * sizeof(int), hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) return e;
    for (int m = 0; m < M && *output < 0; ++m)
        if (h[m]) {
            *output = m;
            *pivot = h[m] - 1;
        }
    return hipSuccess;
}

#define P_HIP(call)                                                                                          \
    do {                                                                                                     \
        hipError_t e__ = (call);                                                                             \
        if (e__ != hipSuccess) {                                                                             \
            snprintf(c->err, sizeof(c->err), "%s: %s failed: %s", who, #call, hipGetErrorString(e__));       \
            rc = (e__ == hipErrorOutOfMemory) ? BAGEL_ENOMEM : BAGEL_EHIP;                                   \
            goto done;                                                                                       \
        }                                                                                                    \
    } while (0)

}  // namespace

void bagel_release_setup(bagel_ctx *c)
{
    setup_scratch *sc = static_cast<setup_scratch *>(c->setup);
    if (!sc) return;
    if (sc->arena) {
        (void)hipFree(sc->arena);
        c->bytes -= (int64_t)sc->arena_bytes;
    }
    delete sc;
    c->setup = nullptr;
}

int bagel_prepare_impl(bagel_ctx *c, const float *X, const float *y, const float *ell, const float *sf2,
                       const float *sn2, const float *omega, const float *phase, const float *w,
                       const float *eps, float *v_out)
{
    static const char who[] = "bagel_prepare_samples";
    const int N = c->dm.N, L = c->dm.L, S = c->dm.S, M = c->M, D = c->D;
    const int Np = (N + NB - 1) / NB * NB, Sp = (S + 63) / 64 * 64, Lq = (L + 63) / 64 * 64;
    hipStream_t st = c->stream;
    setup_scratch *sc = nullptr;
    int n_out = 1, bad = -1, pivot = 0;
    int rc = BAGEL_OK;
    // PhiT shares its place with U (the product with W comes before the factorisation), W's transpose with Z
    const size_t big = (size_t)(Np > Lq ? Np : Lq);
    const size_t nK = (size_t)Np * Np, nU = (size_t)Np * big, nR = (size_t)Np * Sp, nZ = (size_t)Sp * big, nT = (size_t)Np * NB * RB;
    solver s;
    hyper_ptr h = {ell, sf2, sn2, 0};
    int *flag = nullptr;
    double *R = nullptr, *Z = nullptr;
    P_HIP(setup_reserve(c, arena_round(nK * 8) + arena_round(nU * 8) + arena_round(nR * 8) + arena_round(nZ * 8) +
                               2 * arena_round(nT * 8) + arena_round((size_t)Np * 8),
                        arena_round(BAGEL_MAX_STATE * sizeof(int)), &sc, &n_out));
    {
        arena_cursor cur{sc->arena};
        flag = cur.take<int>(BAGEL_MAX_STATE);
        const size_t n = (size_t)n_out;
        s.st = st;
        s.nb = Np / NB;
        s.f.Np = Np;
        s.f.K = cur.take<double>(n * nK); s.f.sK = nK;
        s.f.U = cur.take<double>(n * nU); s.f.sU = nU;
        R = cur.take<double>(n * nR);
        Z = cur.take<double>(n * nZ);
        s.f.V = tri_matrix{cur.take<double>(n * nT), 0, nT};
        s.f.W = tri_matrix{cur.take<double>(n * nT), 0, nT};
        s.f.diag = cur.take<double>(n * Np);
    }
    hipLaunchKernelGGL(clear_flags_kernel, dim3(1), dim3(64), 0, st, flag, BAGEL_MAX_STATE);
    for (int m0 = 0; m0 < M; m0 += n_out) {
        s.outputs = M - m0 < n_out ? M - m0 : n_out;
        s.f.flag = flag + m0;
        // R = y - eps - Phi W^T
        hipLaunchKernelGGL(build_phi_kernel, dim3(Np / 64, Lq / 4, s.outputs), dim3(256), 0, st, X, omega, phase, h, s.f.U, nU, N,
                           Np, L, D, m0);
        hipLaunchKernelGGL(transpose_in_kernel, dim3(Sp / 64, Lq / 64, s.outputs), dim3(256), 0, st, w, (const float *)nullptr, Z,
                           nZ, L, S, Sp, M, m0);
        hipLaunchKernelGGL(transpose_in_kernel, dim3(Sp / 64, Np / 64, s.outputs), dim3(256), 0, st, eps, y, R, nR, N, S, Sp, M, m0);
        gemm_args g = {s.f.U, Z, R, (size_t)Np, (size_t)Sp, (size_t)Sp, nU, nZ, nR, Np, Sp, Lq, 1, 0};
        gemm(st, s.outputs, g);
        // the range inverses are used as whole squares: what is not written of them must be zero
        P_HIP(hipMemsetAsync(s.f.V.p, 0, s.outputs * nT * 8, st));
        P_HIP(hipMemsetAsync(s.f.W.p, 0, s.outputs * nT * 8, st));
        build_and_factor(s, X, h, N, D, m0);
        s.triangular_inverse(RB);
        hipLaunchKernelGGL(mirror_factor_kernel, dim3(s.nb, s.nb, s.outputs), dim3(256), 0, st, s.f.U, s.f.sU, Np);
        const solver::rhs rR = {R, nR, (size_t)Sp}, rZ = {Z, nZ, (size_t)Sp};
        s.forward(0, s.nb, rR, rZ);
        s.backward(0, s.nb, rZ, rR);
        hipLaunchKernelGGL(emit_v_kernel, dim3(Sp / 64, (c->Np + 63) / 64, s.outputs), dim3(256), 0, st, R, nR, Sp, v_out, c->v4, N,
                           c->Np, S, M, m0);
        P_HIP(hipGetLastError());
    }
    P_HIP(read_flags(st, flag, M, &bad, &pivot));
    if (bad >= 0) {
        snprintf(c->err, sizeof(c->err), "%s: K + noise_var I is not positive definite (output %d, pivot %d)", who, bad, pivot);
        rc = BAGEL_ENOTPD;
    }
done:
    (void)hipStreamSynchronize(st);
    return rc;
}

// The work space of an inverse: U, W and, unless it has a place elsewhere, K [Np][Np], diagonal and two vectors per output.
// V takes the place of K, block by block: V's diagonal block k is written when K's is done with (chol_step_kernel keeps the
// next one in LDS, the products of the recursion touch later ranges only), its blocks above the diagonal after the
// factorisation, and T (inverse_level_kernel) has the blocks below.
static size_t inverse_bytes(int Np, bool with_K)
{
    return (with_K ? 3 : 2) * arena_round((size_t)Np * Np * 8) + 3 * arena_round((size_t)Np * 8);
}

// K, and with it V, of the outputs worked on
static void inverse_place(solver &s, double *K)
{
    s.f.K = K;
    s.f.sK = (size_t)s.f.Np * s.f.Np;
    s.f.V = tri_matrix{K, (size_t)s.f.Np, s.f.sK};
}

static void inverse_carve(solver &s, arena_cursor &cur, int n_out, int Np, bool with_K, double **vec)
{
    const size_t n = (size_t)n_out, nK = (size_t)Np * Np;
    s.nb = Np / NB;
    s.f.Np = Np;
    if (with_K) inverse_place(s, cur.take<double>(n * nK));
    s.f.U = cur.take<double>(n * nK); s.f.sU = nK;
    s.f.W = tri_matrix{cur.take<double>(n * nK), (size_t)Np, nK};
    s.f.diag = cur.take<double>(n * Np);
    *vec = cur.take<double>(2 * n * Np);
}

// z = L^-1 y and alpha = K_hat^-1 y = L^-T z
static void inverse_vectors(solver &s, const float *y, int N, int m0, double *z, double *alpha)
{
    const dim3 grid(s.f.Np / 4, s.outputs);
    hipLaunchKernelGGL(triangle_times_vector_kernel, grid, dim3(256), 0, s.st, s.f.W, 0, y, (const double *)nullptr, z, N, s.f.Np,
                       m0);
    hipLaunchKernelGGL(triangle_times_vector_kernel, grid, dim3(256), 0, s.st, s.f.V, 1, (const float *)nullptr, z, alpha, N,
                       s.f.Np, m0);
}

// Exact posterior cache of the per-step sampler (eq. (2), (3)): for every output alpha = K_hat^-1 y and
// K_hat^-1 itself, float64, padded to Np = multiple of 64 (the padding rows and columns of K_hat are an
// identity block, so they do not couple to the data; padded alpha entries are zero).
int bagel_prepare_posterior_impl(bagel_ctx *c, const float *X, const float *y, const float *ell, const float *sf2,
                                 const float *sn2)
{
    static const char who[] = "bagel_prepare_posterior";
    const int N = c->dm.N, M = c->M, D = c->D, Np = c->post_Np;
    hipStream_t st = c->stream;
    setup_scratch *sc = nullptr;
    int n_out = 1, bad = -1, pivot = 0;
    int rc = BAGEL_OK;
    solver s;
    hyper_ptr h = {ell, sf2, sn2, 0};
    int *flag = nullptr;
    double *vec = nullptr;
    float h_sf2[BAGEL_MAX_STATE];
    P_HIP(setup_reserve(c, inverse_bytes(Np, false), arena_round(BAGEL_MAX_STATE * sizeof(int)), &sc, &n_out));
    {
        arena_cursor cur{sc->arena};
        flag = cur.take<int>(BAGEL_MAX_STATE);
        s.st = st;
        inverse_carve(s, cur, n_out, Np, false, &vec);
    }
    P_HIP(hipMemcpyAsync(h_sf2, sf2, M * sizeof(float), hipMemcpyDeviceToHost, st));
    hipLaunchKernelGGL(clear_flags_kernel, dim3(1), dim3(64), 0, st, flag, BAGEL_MAX_STATE);
    for (int m0 = 0; m0 < M; m0 += n_out) {
        s.outputs = M - m0 < n_out ? M - m0 : n_out;
        s.f.flag = flag + m0;
        inverse_place(s, c->post_Kinv + (size_t)m0 * Np * Np);     // (K and V are done with when K_hat^-1 is written)
        build_and_factor(s, X, h, N, D, m0);
        s.triangular_inverse(s.nb);
        inverse_vectors(s, y, N, m0, vec, c->post_alpha + (size_t)m0 * Np);
        hipLaunchKernelGGL(inverse_store_kernel, dim3(s.nb * (s.nb + 1) / 2 * s.outputs), dim3(256), 0, st, s.f.W,
                           c->post_Kinv + (size_t)m0 * Np * Np, Np, s.outputs);
        P_HIP(hipGetLastError());
    }
    P_HIP(read_flags(st, flag, M, &bad, &pivot));
    for (int m = 0; m < M; ++m) c->post_sf2[m] = (double)h_sf2[m];
    if (bad >= 0) {
        snprintf(c->err, sizeof(c->err), "%s: K + noise_var I is not positive definite (output %d, pivot %d)", who, bad, pivot);
        rc = BAGEL_ENOTPD;
    }
done:
    (void)hipStreamSynchronize(st);
    return rc;
}

static void launch_hyper_grad(const solver &s, int D, const float *X, const float *log_hyp, const double *alpha, double *partial,
                              int N, int m0)
{
    const dim3 grid(s.nb * (s.nb + 1) / 2 * s.outputs);
    switch (D) {
#define CASE(n)                                                                                                                \
    case n:                                                                                                                    \
        hipLaunchKernelGGL(hyper_grad_tiles_kernel<n>, grid, dim3(256), 0, s.st, X, log_hyp, s.f.W, alpha, partial, N, \
                           s.f.Np, m0, s.outputs);                                                                             \
        break;
        CASE(2) CASE(3) CASE(4) CASE(5) CASE(6) CASE(7) CASE(8) CASE(9) CASE(10) CASE(11) CASE(12)
        CASE(13) CASE(14) CASE(15) CASE(16)
#undef CASE
    }
}

// Log marginal likelihood of every output's GP and its gradient in the log hyper-parameters
// (eq. (5), (6)), n_iters > 0: Adam ascent on lml / N for n_iters iterations (Algorithm 1, "learn GP
// transition dynamics").
int bagel_hyper_impl(bagel_ctx *c, const float *X, const float *y, float *log_hyp, float *lml, float *grad,
                     float *adam_m, float *adam_v, int n_iters, int first_step, double lr, double beta1, double beta2,
                     double eps)
{
    static const char who[] = "bagel_hyper";
    const int N = c->dm.N, M = c->M, D = c->D, H2 = c->D + 2;
    const int Np = (N + NB - 1) / NB * NB, nb = Np / NB, tiles = nb * (nb + 1) / 2;
    hipStream_t st = c->stream;
    setup_scratch *sc = nullptr;
    int n_out = 1, bad = -1, pivot = 0;
    int rc = BAGEL_OK;
    solver s;
    hyper_ptr h = {log_hyp, nullptr, nullptr, 1};
    int *flag = nullptr;
    float *gneg = nullptr;
    double *vec = nullptr, *partial = nullptr;
    P_HIP(setup_reserve(c, inverse_bytes(Np, true) + arena_round((size_t)tiles * H2 * 8),
                        arena_round(BAGEL_MAX_STATE * sizeof(int)) + arena_round((size_t)M * H2 * sizeof(float)), &sc, &n_out));
    {
        arena_cursor cur{sc->arena};
        flag = cur.take<int>(BAGEL_MAX_STATE);
        gneg = cur.take<float>((size_t)M * H2);
        s.st = st;
        inverse_carve(s, cur, n_out, Np, true, &vec);
        partial = cur.take<double>((size_t)n_out * tiles * H2);
    }
    hipLaunchKernelGGL(clear_flags_kernel, dim3(1), dim3(64), 0, st, flag, BAGEL_MAX_STATE);
    for (int it = 0; it < (n_iters > 0 ? n_iters : 1); ++it) {
        for (int m0 = 0; m0 < M; m0 += n_out) {
            s.outputs = M - m0 < n_out ? M - m0 : n_out;
            s.f.flag = flag + m0;
            double *z = vec, *alpha = vec + (size_t)n_out * Np;
            build_and_factor(s, X, h, N, D, m0);
            s.triangular_inverse(nb);
            inverse_vectors(s, y, N, m0, z, alpha);
            hipLaunchKernelGGL(hyper_lml_kernel, dim3(s.outputs), dim3(256), 0, st, s.f.diag, z, N, Np,
                               lml + (size_t)it * M + m0);
            if (grad || n_iters > 0) {
                launch_hyper_grad(s, D, X, log_hyp, alpha, partial, N, m0);
                hipLaunchKernelGGL(hyper_grad_final_kernel, dim3(H2, s.outputs), dim3(256), 0, st, partial, tiles, N, H2,
                                   grad ? grad + (size_t)m0 * H2 : nullptr, gneg + (size_t)m0 * H2);
            }
            P_HIP(hipGetLastError());
        }
        if (n_iters > 0) {
            const int step = first_step + it;
            P_HIP(bagel_launch_adam(c, log_hyp, gneg, adam_m, adam_v, M * H2, lr, beta1, beta2, eps,
                                    1.0 - pow(beta1, (double)step), 1.0 - pow(beta2, (double)step)));
        }
    }
    P_HIP(read_flags(st, flag, M, &bad, &pivot));
    if (bad >= 0) {
        snprintf(c->err, sizeof(c->err), "%s: K + noise_var I is not positive definite (output %d, pivot %d)", who, bad, pivot);
        rc = BAGEL_ENOTPD;
    }
done:
    (void)hipStreamSynchronize(st);
    return rc;
}
