// Block-Jacobi preconditioner of the system matrix D-hat + B-hat^T N^-1 B-hat
// (gfx950): for every tile J, the Cholesky factor of its diagonal block
// A_J = D_JJ + C_JJ, and the application x_J = A_J^-1 r_J.
//
//   k_factor_diag  one wave per tile, in four panels of 16 rows of U.  The upper
//                  triangle's ten 16 x 16 blocks are MFMA accumulators.  A panel
//                  passes through LDS to one column per lane, where 16 steps
//                  (pivot from its lane, row scaled by the pivot's reciprocal as
//                  LAPACK's unblocked factorisation does, the panel's later rows
//                  updated with values broadcast from their lanes) finish its
//                  rows of U; these pass through LDS to MFMA operands and update
//                  the blocks below (FP64 16x16x4).  No workgroup barrier.
//   k_solve_diag   one wave per tile, column l of U in lane l's registers:
//                  U^T y = r as a column sweep (lane l accumulates row l),
//                  then U x = y as a column sweep from the last row, whose
//                  columns reach the other lanes through LDS eight at a time.
//                  Both multiply by the reciprocals of U's diagonal.
//
// Both read only the 128-byte lines that hold part of the upper triangle (5/8 of
// a block) and are then bound by HBM: the factor reads 40 KiB and writes 32 per
// tile, the solve reads 20 KiB and 1 KiB of vectors.
#include <hip/hip_runtime.h>

#include "precond.hpp"

namespace sympix {
namespace {

constexpr int kN = 64;       // pixels per tile (k = 8)
constexpr int kWaves = 4;    // tiles per workgroup, one wave each

// v as held by lane `src` (a constant of the unrolled loops), in every lane.
__device__ __forceinline__ double from_lane(double v, int src) {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)b, src);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(b >> 32), src);
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

typedef double doublex4 __attribute__((ext_vector_type(4)));

// Values pass between the lanes of one wave through LDS: no other wave looks.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Block (I, L), I <= L, of the upper triangle: lane (lr, lk) holds rows 16 I +
// lk + 4 v of column 16 L + lr, as an MFMA result.  The element-by-element form
// this replaces broadcast every multiplier from LDS to the 64 lanes (2016
// doubles per tile, 32 k LDS clocks per four waves) and took 1.88 ms at lmax
// 2048 (97,456 tiles); this takes 1.3, at 5.4 TB/s.  With C the registers do not
// quite hold it: 44 bytes per lane lie in scratch memory.
template <bool WITH_C>
__global__ __launch_bounds__(64 * kWaves) __attribute__((amdgpu_waves_per_eu(3))) void k_factor_diag(const double *__restrict__ D,
                                                             const double *__restrict__ C,
                                                             const int32_t *__restrict__ dblk, int64_t ntiles,
                                                             double *__restrict__ U, int32_t *__restrict__ info) {
    __shared__ double sP[kWaves][16][kN];    // a panel: row, column
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, lr = lane & 15, lk = lane >> 4;
    const int64_t J = (int64_t)blockIdx.x * kWaves + wave;
    if (J >= ntiles) return;                 // the whole wave
    const int64_t base = (int64_t)dblk[J] * (kN * kN);
    double (*panel)[kN] = sP[wave];
    doublex4 a[4][4];                        // [I][L], L >= I
#pragma unroll
    for (int I = 0; I < 4; ++I)
#pragma unroll
        for (int L = I; L < 4; ++L)
#pragma unroll
            for (int v = 0; v < 4; ++v) a[I][L][v] = D[base + (16 * I + lk + 4 * v) * kN + 16 * L + lr];
    if constexpr (WITH_C) {
#pragma unroll
        for (int I = 0; I < 4; ++I) {
            doublex4 t[4];
#pragma unroll
            for (int L = I; L < 4; ++L)
#pragma unroll
                for (int v = 0; v < 4; ++v) t[L][v] = C[base + (16 * I + lk + 4 * v) * kN + 16 * L + lr];
#pragma unroll
            for (int L = I; L < 4; ++L) a[I][L] += t[L];
            __builtin_amdgcn_sched_barrier(0);   // 16 loads of C in flight at most: more would spill
        }
    }
    double *out = U + J * (kN * kN);
    int bad = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        wave_sync();                         // the previous panel's operands have been read
#pragma unroll
        for (int L = k; L < 4; ++L)
#pragma unroll
            for (int v = 0; v < 4; ++v) panel[lk + 4 * v][16 * L + lr] = a[k][L][v];
        wave_sync();
        double u[16];                        // rows 16 k + j of column `lane`
#pragma unroll
        for (int j = 0; j < 16; ++j) u[j] = panel[j][lane];
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const int r = 16 * k + j;
            const double pivot = from_lane(u[j], r);   // A_rr less the earlier steps' updates
            if (bad == 0 && !(pivot > 0.0)) bad = r + 1;
            const double s = sqrt(pivot);
            const double inv = 1.0 / s;
            u[j] = lane == r ? s : u[j] * inv;
#pragma unroll
            for (int i = j + 1; i < 16; ++i) u[i] = fma(-from_lane(u[j], 16 * k + i), u[j], u[i]);
        }
#pragma unroll
        for (int j = 0; j < 16; ++j) {       // zero below the diagonal
            u[j] = 16 * k + j <= lane ? u[j] : 0.0;
            out[(16 * k + j) * kN + lane] = u[j];
        }
        if (k == 3) break;
        wave_sync();
#pragma unroll
        for (int j = 0; j < 16; ++j) panel[j][lane] = u[j];
        wave_sync();
        double op[4][4];                     // [X][t]: U[16 k + 4 t + lk][16 X + lr], either operand of block X
#pragma unroll
        for (int X = k + 1; X < 4; ++X)
#pragma unroll
            for (int t = 0; t < 4; ++t) op[X][t] = panel[4 * t + lk][16 * X + lr];
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int I = k + 1; I < 4; ++I)
#pragma unroll
                for (int L = I; L < 4; ++L)
                    a[I][L] = __builtin_amdgcn_mfma_f64_16x16x4f64(-op[I][t], op[L][t], a[I][L], 0, 0, 0);
    }
    if (lane == 0) info[J] = bad;
}

// r and x may be the same array: a wave reads its tile of r before it writes
// that tile of x.
__global__ __launch_bounds__(64 * kWaves) void k_solve_diag(const double *__restrict__ U, const double *r,
                                                            double *x, int64_t ntiles) {
    __shared__ double sT[kWaves][8][kN];     // eight columns of U: one block of back-substitution steps
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t J = (int64_t)blockIdx.x * kWaves + wave;
    if (J >= ntiles) return;
    const double *ut = U + J * (kN * kN);
    double u[kN];                            // u[c] = U[c][lane], in the lines that hold part of the upper triangle
#pragma unroll
    for (int c = 0; c < kN; ++c) u[c] = 0.0;
#pragma unroll
    for (int c0 = 0; c0 < kN; c0 += 16)
        if (lane >= c0) {
#pragma unroll
            for (int c = c0; c < c0 + 16; ++c) u[c] = ut[c * kN + lane];
        }
    const double rinv = 1.0 / ut[lane * kN + lane];   // 1 / U[lane][lane]
    double z = r[J * kN + lane];
    // U^T y = r, a column sweep: row l of U^T is column l of U, held by lane l
#pragma unroll
    for (int c = 0; c < kN; ++c) {
        const double yc = from_lane(z, c) * from_lane(rinv, c);
        const double m = lane > c ? yc : 0.0;
        z = lane == c ? yc : fma(-u[c], m, z);
    }
    // U x = y, a column sweep from the last row: step i needs U[c][i] in lane c, i.e.
    // column i of U, held by lane i; eight steps at a time take their columns from LDS
    double xv = 0.0;
#pragma unroll
    for (int b = kN / 8 - 1; b >= 0; --b) {
        const int i0 = 8 * b;
        if (lane >= i0 && lane < i0 + 8) {   // rows c < i0 + 8 are the ones these steps update
            double *row = sT[wave][lane - i0];
#pragma unroll
            for (int c = 0; c < i0 + 8; c += 2) *reinterpret_cast<double2 *>(row + c) = make_double2(u[c], u[c + 1]);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
        for (int i = i0 + 7; i >= i0; --i) {
            const double xi = from_lane(z, i) * from_lane(rinv, i);
            if (lane == i) xv = xi;
            const double m = lane < i ? xi : 0.0;
            z = fma(-sT[wave][i - i0][lane], m, z);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    x[J * kN + lane] = xv;
}

}  // namespace

hipError_t launch_factor_diag(const double *D, const double *C, const int32_t *dblk, int64_t ntiles, double *U,
                              int32_t *info, hipStream_t st) {
    if (ntiles == 0) return hipSuccess;
    const int64_t blocks = (ntiles + kWaves - 1) / kWaves;
    if (C) hipLaunchKernelGGL(k_factor_diag<true>, dim3((unsigned)blocks), dim3(64 * kWaves), 0, st, D, C, dblk, ntiles, U, info);
    else hipLaunchKernelGGL(k_factor_diag<false>, dim3((unsigned)blocks), dim3(64 * kWaves), 0, st, D, C, dblk, ntiles, U, info);
    return hipGetLastError();
}

hipError_t launch_solve_diag(const double *U, const double *r, double *x, int64_t ntiles, hipStream_t st) {
    if (ntiles == 0) return hipSuccess;
    const int64_t blocks = (ntiles + kWaves - 1) / kWaves;
    hipLaunchKernelGGL(k_solve_diag, dim3((unsigned)blocks), dim3(64 * kWaves), 0, st, U, r, x, ntiles);
    return hipGetLastError();
}

}  // namespace sympix
