// Tile routine of the float64 matrix products: C[i][j] = sum_k A[k][i] B[k][j], both operands with the
// contraction index as the row ("k-major"), contiguous along i and j.  Every product of this library can be
// brought into that form (symmetric matrices, triangular factors kept beside their transposes), and in it a row
// of a tile is one contiguous run of memory that goes to LDS as it is.
//
// A workgroup of 256 threads owns a T x T tile of the result (T = 64 or 128); its four waves own T/2 x T/2
// quarters, made of v_mfma_f64_16x16x4 (D[16x16] += A[16x4] B[4x16]; lane l feeds A[l % 16][l / 16] and
// B[l / 16][l % 16]; register r of lane l holds D[l / 16 + 4 r][l % 16]).  Which rows of the quarter a matrix
// instruction covers is free: instruction x = 2 h + e takes rows 2 (l % 16) + 32 h + e, so that a lane's
// operands for e = 0, 1 are one 16-byte LDS read (16 lanes: one whole pass over the banks, no conflicts), and so
// that a lane's results are pairs of neighbouring columns.
//
// Tiles of TK contraction indices come into LDS through loads that write LDS directly (lane i's 16 bytes land
// at byte 16 i of the wave's kilobyte: one row of 128 doubles or two of 64), NST stages deep: the loads of
// the next stages are in flight under the matrix instructions of the current one, no staging registers, one
// barrier per stage.  The loads are issued from inline assembly because through the compiler's builtin every
// LDS read would wait for all outstanding loads of this kind; the assembly writes no register, and the
// routine waits (vmcnt) itself before the barrier that publishes a stage.
//
// Extents: i, j ranges are multiples of 64 (a tile that hangs over the end by 64 reads its first 64 columns
// twice; the caller drops the surplus results), the contraction is a multiple of 16, rows are 16-byte aligned.
#pragma once
#include <hip/hip_runtime.h>

namespace f64_tile {

typedef double d4v __attribute__((ext_vector_type(4)));

template <int T>
struct shape {
    static constexpr int TK = 16;
    static constexpr int NST = T == 128 ? 2 : 3;             // 64 KB: two workgroups per compute unit; 48 KB: three
    static constexpr int H = T / 64;                         // 32-row groups per wave and direction
    static constexpr int STAGE = 2 * TK * T;                 // doubles per stage: A rows, then B rows
    static constexpr int LDS_DOUBLES = NST * STAGE;
    static constexpr int LOADS = TK * T * 8 / 1024 / 4;      // loads per wave, stage and operand
};

// Do `tiles` tiles of 128 x 128 fill whole passes over the chip?  Two of them share a compute unit, and one alone keeps
// its matrix pipes busy nearly as well, so a product takes 1, 2, 4, 6, ... times the time of one tile as its tiles
// reach 256, 512, 1024, 1536, ... (what is left over after a pass of 512 is not spread one per unit); one of 64 x 64
// takes a quarter of that time and balances by itself, at 5 % less speed.  Measured on the posterior step, 64 against
// 128 (N, B, outputs): 512 tiles (2048, 1024, 4) 556 / 529 us; 256 tiles (2048, 512, 4) 321 / 311, (4096, 512, 2) 577 / 563;
// 384 tiles (2048, 768, 4) 440 / 520; 768 tiles (4000, 500, 6) 1580 / 1944; 64 tiles (1024, 256, 4) 89 / 178.  256 and 512 are
// one and two per compute unit of an MI355X.  The products of the set-up calls, shorter ones among them, go by the same line;
// a set-up of samples (N, L, S, outputs) by it, with 64 and with 128 throughout: (8192, 4096, 8192, 6) 173 / 179 / 178 ms;
// (4096, 2048, 4096, 4) 17.5 / 17.4 / 18.0; (2048, 1024, 4096, 4) 5.12 / 4.96 / 5.35; (4096, 1024, 512, 3) 5.14 / 4.92 / 7.97;
// (1024, 1024, 1024, 4) 0.96 / 0.95 / 1.42.
inline bool whole_passes(long tiles)
{
    if (tiles <= 256) return 100 * tiles >= 95 * 256;
    const long passes = (tiles + 511) / 512;
    return 100 * tiles >= 95 * 512 * passes;
}

template <int T>
struct accumulators {
    d4v v[2 * shape<T>::H][2 * shape<T>::H];                 // [x = 2 h + e][y = 2 h' + e']
};

// Row and column inside the tile of entry v[2 h + e][2 h' + e'][r] of a lane:
// (row0 + 32 h + e + 8 r, col0 + 32 h' + e')
struct lane_pos {
    int row0, col0;
};
template <int T>
__device__ __forceinline__ lane_pos lane_position()
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    return lane_pos{(wave >> 1) * (T / 2) + 2 * (lane >> 4), (wave & 1) * (T / 2) + 2 * (lane & 15)};
}

// lane i's 16 bytes at base + off go to LDS byte address lds + 16 i (base and lds are wave-uniform).  M0 cannot be named as
// clobbered: it is a reserved register, in which the compiler keeps nothing (it would write it right before an
// instruction of its own that reads it; the kernels that call this have none).
__device__ __forceinline__ void load_row_to_lds(const double *base, unsigned off, unsigned lds)
{
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %2" : : "v"(off), "s"(lds), "s"(base) : "memory");
}

// s_waitcnt with only the vector-memory counter set (expcnt and lgkmcnt left at their maxima)
template <int N>
__device__ __forceinline__ void wait_loads_at_most()
{
    static_assert(N >= 0 && N < 64, "vmcnt has six bits");
    __builtin_amdgcn_s_waitcnt(0x0f70 | (N & 15) | ((N >> 4) << 14));
}

// acc (+)= sum_k A[k][i0 + i] B[k][j0 + j] over k in [0, Kd).  A and B point at row 0 of the contraction, column 0;
// ni, nj: extents of i and j (for a tile that hangs over the end).  Ends with a barrier: the LDS may be reused.
// The caller zeroes acc.  No vector-memory operation of the caller may be outstanding that it relies on being
// outstanding afterwards (the routine waits for all of them).
template <int T>
__device__ __forceinline__ void product(accumulators<T> &acc, double *lds, int i0, int j0, int ni, int nj, int Kd,
                                        const double *A, size_t lda, const double *B, size_t ldb)
{
    using S = shape<T>;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) double *)lds;
    // column (and for T = 64 the row within the pair) this lane fetches
    unsigned offa, offb;
    if (T == 128) {
        offa = 16u * (unsigned)(i0 + 64 < ni ? lane : (lane & 31));
        offb = 16u * (unsigned)(j0 + 64 < nj ? lane : (lane & 31));
    } else {
        offa = 16u * (unsigned)(lane & 31) + (unsigned)(lane >> 5) * (unsigned)(lda * 8);
        offb = 16u * (unsigned)(lane & 31) + (unsigned)(lane >> 5) * (unsigned)(ldb * 8);
    }
    constexpr int RPL = T == 128 ? 1 : 2;                    // rows per load
    const double *pa = A + (size_t)(RPL * wave) * lda + i0;
    const double *pb = B + (size_t)(RPL * wave) * ldb + j0;
    const size_t stepa = 4 * RPL * lda, stepb = 4 * RPL * ldb;
    const int nst = Kd / S::TK;
    int issued = 0, slot = 0;
    auto issue = [&]() {
        const unsigned la = lds0 + 8u * (unsigned)(slot * S::STAGE) + 1024u * (unsigned)wave;
        const unsigned lb = la + 8u * (unsigned)(S::TK * T);
#pragma unroll
        for (int e = 0; e < S::LOADS; ++e) {
            load_row_to_lds(pa, offa, la + 4096u * e);
            pa += stepa;
        }
#pragma unroll
        for (int e = 0; e < S::LOADS; ++e) {
            load_row_to_lds(pb, offb, lb + 4096u * e);
            pb += stepb;
        }
        ++issued;
        slot = slot + 1 == S::NST ? 0 : slot + 1;
    };
#pragma unroll
    for (int s = 0; s < S::NST - 1; ++s)
        if (issued < nst) issue();
    const int fa = (lane >> 4) * T + (wave >> 1) * (T / 2) + 2 * (lane & 15);
    const int fb = (lane >> 4) * T + (wave & 1) * (T / 2) + 2 * (lane & 15) + S::TK * T;
    int rd = 0;
    for (int s = 0; s < nst; ++s) {
        // stage s has landed once at most the loads of the later stages are outstanding (loads complete in order)
        if (S::NST > 2 && issued - s > 1) wait_loads_at_most<2 * S::LOADS>();
        else wait_loads_at_most<0>();
        __syncthreads();                                     // ... for every wave; and stage s - 1 has been read
        if (issued < nst) issue();
        const double *st = lds + rd * S::STAGE;
#pragma unroll
        for (int k4 = 0; k4 < S::TK / 4; ++k4) {
            double2 a[S::H], b[S::H];
#pragma unroll
            for (int h = 0; h < S::H; ++h) a[h] = *reinterpret_cast<const double2 *>(st + fa + 4 * k4 * T + 32 * h);
#pragma unroll
            for (int h = 0; h < S::H; ++h) b[h] = *reinterpret_cast<const double2 *>(st + fb + 4 * k4 * T + 32 * h);
#pragma unroll
            for (int x = 0; x < 2 * S::H; ++x)
#pragma unroll
                for (int y = 0; y < 2 * S::H; ++y)
                    acc.v[x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64((x & 1) ? a[x >> 1].y : a[x >> 1].x,
                                                                       (y & 1) ? b[y >> 1].y : b[y >> 1].x, acc.v[x][y], 0, 0, 0);
        }
        rd = rd + 1 == S::NST ? 0 : rd + 1;
    }
    __syncthreads();
}

template <int T>
__device__ __forceinline__ void clear(accumulators<T> &acc)
{
#pragma unroll
    for (int x = 0; x < 2 * shape<T>::H; ++x)
#pragma unroll
        for (int y = 0; y < 2 * shape<T>::H; ++y) acc.v[x][y] = d4v{0.0, 0.0, 0.0, 0.0};
}

}  // namespace f64_tile
