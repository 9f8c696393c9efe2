// HIP kernels for SymPix local-operator sampling on gfx950 (CDNA4, wave64).
//
//   k_tabulate     kernel table of Eq. 10, FP64 Legendre recurrence in y
//   k_eval         table lookups at arbitrary y (interpolation tests)
//   k_unique_eval  one workgroup per unique block (Section 2.3 symmetry keys):
//                  pair geometry, table lookup, radial cut; writes FP64
//                  row-major and FP64 / FP32 copies transposed via LDS
//   k_expand       D-hat: streams each stored block from its unique block
//   k_convolve     pixel-domain convolution g = B-hat f, one FP64 GEMM per
//                  unique block over 32 output tiles
//   k_class_f64    B-hat^T N^-1 B-hat (Eq. 15) in FP64 as one GEMM per class of
//                  blocks that share their contraction pattern; the class
//                  kernels' <true> instantiations also copy D-hat (combined call)
//   k_ninv_f32     N^-1 rounded to FP32
//   k_class_f32    FP32-MFMA contraction as one GEMM per class of blocks that
//                  share their contraction pattern, FP64 accumulation across tiles
//   k_batch_f64    the FP64 class GEMM of many problems in one persistent
//                  launch fed by per-XCD work queues
//   k_batch_f32    the same in FP32
//   k_split_ninv   N^-1 split into BF16 parts
//   k_class_bf16   the same GEMM in split BF16
//   k_batch_bf16   many problems in one persistent launch, split BF16
#include <hip/hip_runtime.h>

#include <mutex>
#include <type_traits>

#include "device.hpp"

namespace sympix {
namespace {

typedef double doublex4 __attribute__((ext_vector_type(4)));
typedef double doublex2 __attribute__((ext_vector_type(2)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint16_t u16x8 __attribute__((ext_vector_type(8)));

constexpr double kInv4Pi = 0.07957747154594767;   // 1 / (4 pi)

// Workgroups are dispatched round-robin over the 8 XCDs (each with its own L2).
// Remap the workgroup index so that every XCD processes one contiguous range of
// the work list: neighbouring items share operands, which then stay in that
// XCD's L2.  A bijection on [0, gridDim.x).
__device__ __forceinline__ int xcd_contiguous_index() {
    const int n = gridDim.x, b = blockIdx.x;
    const int x = b & 7, i = b >> 3;
    const int per = n >> 3, rem = n & 7;
    return x * per + min(x, rem) + i;
}

// ---------------------------------------------------------------------------
// a6: kernel table.  Node i holds b at s = |i - 1| h, y = s^2 (node 0 mirrors
// node 2: the kernel is even in s).  Recurrence in y with D_l = P_l - P_{l-1}.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_tabulate(const double *__restrict__ coef, int lmax,
                                                  double h, double *__restrict__ table,
                                                  int n_nodes, int32_t *__restrict__ overflow) {
    if (blockIdx.x == 0 && threadIdx.x == 0) *overflow = 0;   // set by k_unique_eval, next on the stream
    // Per-degree factors of the recurrence, staged in LDS a chunk of degrees
    // at a time by the whole workgroup: step l takes d <- A_l d - B_l y p with
    // A_l = l / (l + 1), B_l = (2l + 1) / (l + 1), then p <- p + d (now
    // P_{l+1}(1 - y)), and adds C_l p, C_l = (2l + 3) coef_{l+1} / 4 pi.
    constexpr int kChunk = 1024;
    __shared__ double sA[kChunk], sB[kChunk], sC[kChunk];
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const double s = (double)(i > 0 ? i - 1 : 1) * h;
    const double y = s * s;
    double p = 1.0;
    double acc = coef[0] * kInv4Pi;
    double d = 0.0;                      // step 0 gives d = -y (A_0 = 0, B_0 = 1)
    for (int l0 = 0; l0 < lmax; l0 += kChunk) {
        const int n = min(kChunk, lmax - l0);
        __syncthreads();                 // the previous chunk is used up
        for (int t = threadIdx.x; t < n; t += blockDim.x) {
            const int l = l0 + t;
            sA[t] = (double)l / (double)(l + 1);
            sB[t] = (double)(2 * l + 1) / (double)(l + 1);
            sC[t] = (double)(2 * l + 3) * coef[l + 1] * kInv4Pi;
        }
        __syncthreads();
        for (int t = 0; t < n; ++t) {
            d = sA[t] * d - sB[t] * y * p;
            p = p + d;
            acc += sC[t] * p;
        }
    }
    if (i < n_nodes) table[i] = acc;
}

// 4-point Lagrange interpolation in s = sqrt(y) on nodes -1, 0, 1, 2 around
// the interval containing s; zero beyond the radial cut.
__device__ __forceinline__ double lookup(const KTable &kt, double y) {
    if (!(y <= kt.y_cut)) return 0.0;
    double u = sqrt(y) * kt.inv_h;
    u = fmin(u, (double)(kt.n_nodes - 3));
    int i = (int)u;
    i = min(i, kt.n_nodes - 4);
    const double t = u - (double)i;
    const double *T = kt.table + i;
    const double tp1 = t + 1.0, tm1 = t - 1.0, tm2 = t - 2.0;
    const double w0 = -t * tm1 * tm2 * (1.0 / 6.0);
    const double w1 = tp1 * tm1 * tm2 * 0.5;
    const double w2 = -tp1 * t * tm2 * 0.5;
    const double w3 = tp1 * t * tm1 * (1.0 / 6.0);
    return w0 * T[0] + w1 * T[1] + w2 * T[2] + w3 * T[3];
}

__global__ __launch_bounds__(256) void k_eval(KTable kt, const double *__restrict__ y,
                                              double *__restrict__ out, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = lookup(kt, y[i]);
}

__device__ __forceinline__ uint16_t bf16_bits(float x) {
    __bf16 b = (__bf16)x;   // round to nearest even
    return __builtin_bit_cast(uint16_t, b);
}

__device__ __forceinline__ float bf16_value(uint16_t b) {
    return __builtin_bit_cast(float, (uint32_t)b << 16);
}

// ---------------------------------------------------------------------------
// a7: unique blocks (the 64 pairs of columns and the 64 pairs of rings hold all
// sines: computed per element they took most of 70 us at lmax 1500).  Element (p, q): row pixel p = c*8 + r of tile I, column
// pixel q of tile J.  dphi = pi N / (n_i n_j) with N reduced exactly into
// (-n_i n_j, n_i n_j]; y = 2 [sin^2(dtheta/2) + sin th1 sin th2 sin^2(dphi/2)].
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_unique_eval(KTable kt, const UInfo *__restrict__ uinfo,
                                                     const double *__restrict__ ring_theta,
                                                     const double *__restrict__ ring_sin,
                                                     double *__restrict__ u64,
                                                     double *__restrict__ u64t,
                                                     float *__restrict__ ut32, UnitMasks um) {
    __shared__ double tile[64][65];
    __shared__ double ssp[64], ssd[64], sss[64];
    __shared__ uint32_t scols[4];
    if (threadIdx.x < 4) scols[threadIdx.x] = 0;
    const int64_t uid = blockIdx.x;
    const UInfo inf = uinfo[uid];
    const int64_t M = (int64_t)inf.n_i * inf.n_j;
    const double inv2M = 1.0 / (double)(2 * M);
    double *dst = u64 + uid * kBlockElems;
    if (threadIdx.x < 64) {              // columns (c, c2): sin(dphi / 2)
        const int c = threadIdx.x >> 3, c2 = threadIdx.x & 7;
        int64_t N = (int64_t)(2 * (inf.p0_j + c2) + 1) * inf.n_i -
                    (int64_t)(2 * (inf.p0_i + c) + 1) * inf.n_j;
        while (N > M) N -= 2 * M;
        while (N <= -M) N += 2 * M;
        ssp[threadIdx.x] = sinpi((double)N * inv2M);
    } else if (threadIdx.x < 128) {      // rings (r, r2): sin(dtheta / 2) and the product of the sines
        const int r = threadIdx.x >> 3 & 7, r2 = threadIdx.x & 7;
        const int j1 = inf.ring0_i + r, j2 = inf.ring0_j + r2;
        ssd[8 * r + r2] = sin(0.5 * (ring_theta[j1] - ring_theta[j2]));
        sss[8 * r + r2] = ring_sin[j1] * ring_sin[j2];
    }
    __syncthreads();
    for (int e = threadIdx.x; e < kBlockElems; e += 256) {
        const int p = e >> 6, q = e & 63;
        const int c = p >> 3, r = p & 7, c2 = q >> 3, r2 = q & 7;
        const double sp = ssp[8 * c + c2], sd = ssd[8 * r + r2];
        const double y = 2.0 * (sd * sd + sss[8 * r + r2] * (sp * sp));
        const double v = lookup(kt, y);
        dst[e] = v;
        tile[p][q] = v;
    }
    __syncthreads();
    const int64_t base = uid * kBlockElems;
    for (int e = threadIdx.x; e < kBlockElems; e += 256) {
        const int q = e >> 6, p = e & 63;   // transposed layout [q][p]
        const double v = tile[p][q];
        u64t[base + e] = v;
        ut32[base + e] = (float)v;
        // rings of each half of the tile (four columns) that are not all zero in column q
        const uint64_t nzp = __ballot(v != 0.0);
        uint32_t lo = (uint32_t)nzp, hi = (uint32_t)(nzp >> 32);
        lo |= lo >> 16;
        hi |= hi >> 16;
        const uint32_t nz = ((lo | lo >> 8) & 255u) | ((hi | hi >> 8) & 255u) << 8;
        const bool over = __any(!(fabsf((float)v) < INFINITY));
        if (p == 0) {
            um.units[uid * 64 + q] = (uint16_t)nz;
            atomicOr(&scols[q >> 4], nz);
            if (over) atomicOr(um.overflow, 1);
        }
    }
    __syncthreads();
    if (threadIdx.x < 4) um.cols[uid * 4 + threadIdx.x] = (uint16_t)scols[threadIdx.x];
}

// ---------------------------------------------------------------------------
// a8: D-hat expansion.  Each stored block is a 32 KiB copy of its unique block.
// A workgroup holds one unique block in registers (2 x 16 bytes per thread)
// and writes it to up to 64 stored blocks with 16-byte non-temporal stores,
// so the unique blocks are read once and the kernel only streams writes.  The
// stored blocks of a band's unique blocks interleave in memory: each XCD takes
// one contiguous range of the items, and 1024 threads write a block in two
// stores each, so that what is written together lies together.  Measured with
// its tabulation against 256 threads and items in turn over the XCDs: lmax 400
// 211 -> 204 us, 900 717 -> 697; at 1500 (8.5 GB) the gain, 1.68 -> 1.57 ms, is
// less than runs of either differ by (12%).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(1024) void k_expand(const double *__restrict__ u64,
                                                const int32_t *__restrict__ items,
                                                const int32_t *__restrict__ exp_blk,
                                                double *__restrict__ out) {
    const int item = xcd_contiguous_index();
    const int32_t uid = items[4 * item], first = items[4 * item + 1];
    const int32_t count = items[4 * item + 2];
    const doublex2 *src = (const doublex2 *)(u64 + (int64_t)uid * kBlockElems);
    doublex2 v[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) v[j] = src[threadIdx.x + 1024 * j];
    for (int n = 0; n < count; ++n) {
        doublex2 *dst = (doublex2 *)(out + (int64_t)exp_blk[first + n] * kBlockElems);
#pragma unroll
        for (int j = 0; j < 2; ++j) __builtin_nontemporal_store(v[j], &dst[threadIdx.x + 1024 * j]);
    }
}

// ---------------------------------------------------------------------------
// Pixel-domain convolution g = B-hat f (Section 4.1): g_J = sum_{K in nbr(J)}
// B_JK f_K.  One workgroup per chunk of kConvTiles (32) consecutive output
// tiles of a band, wave i computing output rows 16 i .. 16 i + 15 of all of
// them, as two 16-column MFMA tiles.  For every unique block u the chunk uses
// (a slot), one FP64 GEMM C += U_u F_u with C[p][j] the outputs of tile J0 + j
// and F_u[q][j] = f of the input tile that tile J0 + j multiplies with u
// (zero when it does not), so each unique block is read once per 32 tiles.
// F_u (32 tiles x 64 values) is loaded once by the workgroup into one of two
// LDS buffers, one barrier per slot; each wave loads only its own 16 rows of
// U_u.  Loads of the next slot go out before the current slot's MFMAs.  MFMA
// 16x16x4 FP64, MFMA m = 2 x + t with contraction index q = 8 x + 2 lk + t:
// lane (lr, lk) holds U[16 i + lr][q] and F[q][16 cg + lr]; its result holds
// rows 16 i + lk + 4 v of column 16 cg + lr.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_convolve(const double *__restrict__ u64, const int32_t *__restrict__ chunks,
                                                  const int32_t *__restrict__ slots, const double *__restrict__ f,
                                                  double *__restrict__ g) {
    constexpr int NT = kConvTiles, SW = 1 + kConvTiles;   // tiles per chunk, ints per slot
    constexpr int NCG = NT / 16, NFR = NT / 8;             // 16-column MFMA tiles, F chunks per thread
    static_assert(NT % 16 == 0 && NT <= 64, "16-column MFMA tiles, at most 64 KiB of staged F");
    // F of one slot: tile t's 64 values as 32 chunks of 16 bytes, chunk c at
    // 32 t + (c ^ (t & 15)), so each 16-lane read phase (16 tiles, one c)
    // touches 16 different bank groups
    __shared__ doublex2 sF[2][NT * 32];
    const int ch = xcd_contiguous_index();
    const int J0 = chunks[4 * ch], n = chunks[4 * ch + 1];
    const int s0 = chunks[4 * ch + 2], ns = chunks[4 * ch + 3];
    const int tid = threadIdx.x;
    const int i = __builtin_amdgcn_readfirstlane(tid >> 6);   // this wave's rows 16 i .. 16 i + 15
    const int lane = tid & 63, lr = lane & 15, lk = lane >> 4;
    // F staging: thread tid takes chunks tid + 256 r (r < NT / 8): tile (tid >> 5) + 8 r, chunk tid & 31
    const int ft = tid >> 5, fc = tid & 31;
    struct Ops { doublex2 a[8], fs[NFR]; };
    // The block and the input tiles of the next slot to load, read a slot ahead: read with the
    // slot's data they held up the current slot's MFMAs for a load's latency (476 -> 364 us at
    // lmax 3000, 98 -> 77 at 1000, 47 -> 40 at 300).
    int32_t uid, K[NFR];
    auto next = [&](int sl) {
        const int32_t *slot = slots + SW * (int64_t)(s0 + min(sl, ns - 1));
#pragma unroll
        for (int r = 0; r < NFR; ++r) K[r] = slot[1 + ft + 8 * r];
        uid = slot[0];
    };
    next(0);
    auto load = [&](int sl, Ops &o) {
#pragma unroll
        for (int r = 0; r < NFR; ++r)
            o.fs[r] = K[r] >= 0 ? *(const doublex2 *)(f + (int64_t)K[r] * 64 + 2 * fc) : doublex2{0.0, 0.0};
        const doublex2 *up = (const doublex2 *)(u64 + (int64_t)uid * kBlockElems + (16 * i + lr) * 64 + 2 * lk);
#pragma unroll
        for (int x = 0; x < 8; ++x) o.a[x] = up[4 * x];   // the four lanes of a row read 64 contiguous bytes
        next(sl + 1);
    };
    auto stage = [&](const Ops &o, int buf) {
#pragma unroll
        for (int r = 0; r < NFR; ++r) {
            const int t = ft + 8 * r;
            sF[buf][32 * t + (fc ^ (t & 15))] = o.fs[r];
        }
    };
    doublex4 c[NCG];
#pragma unroll
    for (int cg = 0; cg < NCG; ++cg) c[cg] = doublex4{0.0, 0.0, 0.0, 0.0};
    auto mfmas = [&](const Ops &o, int buf) {
#pragma unroll
        for (int cg = 0; cg < NCG; ++cg) {
            const int t = 16 * cg + lr;
#pragma unroll
            for (int x = 0; x < 8; ++x) {
                const doublex2 bf = sF[buf][32 * t + ((4 * x + lk) ^ (t & 15))];
                c[cg] = __builtin_amdgcn_mfma_f64_16x16x4f64(o.a[x][0], bf[0], c[cg], 0, 0, 0);
                c[cg] = __builtin_amdgcn_mfma_f64_16x16x4f64(o.a[x][1], bf[1], c[cg], 0, 0, 0);
            }
        }
    };
    Ops o0, o1;
    load(0, o0);
    stage(o0, 0);
    __syncthreads();
    // slot sl computes from buffer sl & 1 with its U rows in registers; the
    // next slot's loads go out first and its F is staged after the MFMAs
    for (int sl = 0; sl < ns; sl += 2) {
        load(sl + 1, o1);
        mfmas(o0, 0);
        stage(o1, 1);
        __syncthreads();
        if (sl + 1 >= ns) break;
        load(sl + 2, o0);
        mfmas(o1, 1);
        stage(o0, 0);
        __syncthreads();
    }
#pragma unroll
    for (int cg = 0; cg < NCG; ++cg) {
        const int j = 16 * cg + lr;
        if (j < n) {
            double *o = g + (int64_t)(J0 + j) * 64 + 16 * i + lk;
#pragma unroll
            for (int v = 0; v < 4; ++v) o[4 * v] = c[cg][v];
        }
    }
}

// ---------------------------------------------------------------------------
// D-hat copies made by a class-GEMM launch for the stored blocks of its tile
// (the combined call): each stored block gets its unique D-hat block
// (row-major FP64).  Chunk c of a tile is 16 bytes (c & 2047) of member row
// c >> 11; a wave's 64 chunks lie in one row, so the row is uniform.  Step stp
// of a workgroup of NT threads loads chunks [N NT stp, N NT (stp + 1)), N per
// thread (past the tile's last chunk it reloads the first row's and stores
// nothing).  The FP32 and split-BF16 forms store them one step later, right after
// that step's loads: stores and loads share one wait counter, and a store placed
// there is waited for only by the next step's operand wait.  The FP64 form
// stores them at the end of their own step, after its barrier, where the
// compiler's wait for them also empties the operand loads ahead of them.
// sBlk[m] is the stored block of member row m (-1: none), sBlk[64 + m] its unique
// D-hat block.
// ---------------------------------------------------------------------------
template <int N>
struct DCopy {
    doublex2 v[N];
    double *dst[N];            // uniform: where the chunk row goes (nullptr: nowhere)
    __device__ __forceinline__ void clear() {
#pragma unroll
        for (int r = 0; r < N; ++r) dst[r] = nullptr;
    }
};

template <int NT, int N>
__device__ __forceinline__ void dcopy_load(const double *__restrict__ du64, double *__restrict__ outD,
                                           const int32_t *sBlk, int nchunks, int stp, int wave, int lane,
                                           DCopy<N> &dc) {
#pragma unroll
    for (int r = 0; r < N; ++r) {
        const int c0 = __builtin_amdgcn_readfirstlane((N * stp + r) * NT + 64 * wave);
        const bool ok = c0 < nchunks;
        const int m = ok ? c0 >> 11 : 0;
        const int blk = __builtin_amdgcn_readfirstlane(sBlk[m]);
        const int uid = __builtin_amdgcn_readfirstlane(sBlk[64 + m]);
        const int base = 2 * (c0 & 2047);
        const double *src = du64 + (int64_t)uid * kBlockElems + base;
        dc.v[r] = *(const doublex2 *)(src + 2 * lane);
        dc.dst[r] = ok && blk >= 0 ? outD + (int64_t)blk * kBlockElems + base : nullptr;
    }
}

template <int N>
__device__ __forceinline__ void dcopy_store(const DCopy<N> &dc, int lane) {
#pragma unroll
    for (int r = 0; r < N; ++r)
        if (dc.dst[r]) __builtin_nontemporal_store(dc.v[r], (doublex2 *)(dc.dst[r] + 2 * lane));
}

// The thread's index.  Where a kernel loops over work items (BATCH) it is opaque to
// the compiler: what a tile's body derives from it (swizzles, staging offsets, of
// every tile height and form) would otherwise be computed once ahead of the loop
// and held in registers through all bodies, which spilled (104 bytes per lane in
// FP64, 256 in BF16x6).
template <bool BATCH>
__device__ __forceinline__ int thread_index() {
    int t = threadIdx.x;
    if constexpr (BATCH) asm volatile("" : "+v"(t));
    return t;
}

// A class without contraction terms: between two grids, when the auxiliary
// grid is the coarser one, a stored block (J, K) can have no tile I that
// neighbours both J and K, so the sum of Eq. 15 is empty and the block is
// zero.  The workgroup clears the member tile's blocks (and gives them their
// D-hat copies), without LDS; the caller returns right after.
template <int NT, bool WD, class PD>
__device__ __forceinline__ void empty_class_tile(const PD &pd, const DevClass &cl, int m0, int rows) {
    constexpr int kChunks = kBlockElems / 2;            // 16-byte chunks of a block
    const int nm = min(rows, cl.nblocks - m0);
    for (int c = threadIdx.x; c < nm * kChunks; c += NT) {
        const int m = c / kChunks, q = c - m * kChunks;
        const int64_t blk = pd.cblk[cl.blk0 + m0 + m];
        __builtin_nontemporal_store(doublex2{0.0, 0.0}, (doublex2 *)(pd.out + blk * kBlockElems) + q);
        if constexpr (WD) {
            const int64_t u = pd.blk_uid[blk];
            __builtin_nontemporal_store(*((const doublex2 *)(pd.du64 + u * kBlockElems) + q),
                                        (doublex2 *)(pd.outD + blk * kBlockElems) + q);
        }
    }
}

// ---------------------------------------------------------------------------
// a9, FP64 MFMA class GEMM (the class decomposition is described with the
// FP32 form below).  W = N^-1 as given, M = B_IJ[p][a] B_IK[p][b] formed in
// FP64 from the transposed FP64 unique blocks.  MFMA 16x16x4 FP64: lane
// (lr, lk) holds W[16 i + lr][p] and M[p][16 j + lr], its result members 16 i +
// lk + 4 v of column b = 16 j + lr.  The MFMA accumulates in FP64 across all
// terms of an output row, so there is no separate accumulation step.
//
// Blocks cut at a radius are largely zero: a 3-pixel beam cut at three FWHM
// leaves 44% of the elements of the unique blocks, and 27% of the products
// B[p][a] B[p][b] of a contraction.  So only products that can be nonzero are
// formed, in whole MFMAs.  An MFMA's four pixels are a unit, four columns of
// one ring of the tile (pixel lk of the unit at lane lk), and bit masks written
// with the unique blocks say in which units a column a, or a group of 16
// columns, is not all zero.  A step is one term's group of 4 x 4 pixels (MFMA t
// takes its ring t), the four waves of a workgroup take R consecutive rows a
// through the same steps, listed beforehand (those in which any of the rows and
// any column can be nonzero), and each wave runs only the MFMAs whose row and
// column group are not all zero in unit t.  What is left out are products with
// an exact zero, so the sums are those of the full contraction bit for bit,
// whatever rows and members share a tile.  A tile whose N^-1 holds an infinity
// or NaN, and a kernel whose table overflowed, run the full lists, since there
// a zero factor does not give a zero product.  MFMAs left (lmax 256, beam 3
// pixels): 48%; units of four rings of a column would leave 55%.  A kernel without
// a cut skips the masks and runs the full lists.
//
// The operands of a step are staged through LDS for all four waves (W of the
// tile's rows, the B_IK values of all columns, the B_IJ values of the rows), by
// loads that write LDS directly, three steps ahead into three buffers, one
// barrier per step.  With so few MFMAs per step, operands loaded by each wave on
// its own were bound by L2 (16 bytes per clock and CU).  Wave w takes column
// group (w + r) mod 4 of row r: 16 accumulators, so that two workgroups share a
// CU (one's MFMAs run while the other waits or stores), and the four waves'
// shares of a step are nearly equal (one column group per wave: the longest of
// the four is 11% above their mean, one row per wave 18%, this 1%).
//
// Symmetric classes (every term pairs a unique block with itself: the blocks
// (J, J)) give C[a][b] = C[b][a] bit for bit, since the products B[p][a]
// B[p][b] are the same numbers either way round.  Row a then computes only
// the column groups j >= a / 16 (10 of the 16 16x16 tiles) and writes the
// tiles below the diagonal as mirror images (plain stores: a mirrored row
// gets its 16 values from 16 rows a at different times, and L2 merges them,
// where streaming stores would send each 8 bytes out as a partial line).
// There wave w takes row w of every four, with all column groups it needs: the
// rows run in four phases whose first column group JLO is a compile-time
// constant, and a step takes more rows the fewer column groups they have.
// Measured (MI355X, beam 3 pixels; the full contraction in 4-wave workgroups,
// operands loaded per wave, before): contraction alone 46.1 -> 26.8 ms at lmax
// 3000 and 12.0 -> 6.8 ms at 1500, with D-hat 48.1 -> 29.3 ms at lmax 3000; the
// MFMAs left take 18 ms at the FP64 matrix rate.  Beam 2 pixels (lmax 2048):
// 23.5 -> 6.6 ms, 5 pixels (91% of the MFMAs left): 23.6 -> 21.8 ms.
// ---------------------------------------------------------------------------
// Rows per row group and of them per wave: R rows by all waves, or in phase JLO
// of a symmetric class 4 f64_sym_rows, one in four per wave: as many as keep 16
// accumulators busy (and lie in the phase).
__host__ __device__ constexpr int f64_rows(int ni) { return ni == 4 ? 4 : 8; }
__host__ __device__ constexpr int f64_sym_rows(int ni, int jlo) { return jlo == 3 ? 4 : jlo == 2 ? (ni == 4 ? 2 : 4) : ni == 4 ? 1 : 2; }
constexpr int kLastStep = 0x8000, kLastOfRows = 0x4000;   // the last step of a list, of a row group

// LDS of an FP64 class tile, f64_lds_bytes(S, rows) of it for up to S terms per
// class and `rows` members per tile.  The staging buffers come first: three,
// holding W (64 rows of 128 bytes, 32 in tiles of fewer members), B_IK (64
// columns) and B_IJ (16 rows).
struct F64Lds {
    char *stage;
    int32_t *blk;               // [192]: stored block per member row; its D-hat source block; and the stored
                                // blocks again, at 16 i + 4 lk + v that of row 16 i + lk + 4 v
    uint16_t *mask;             // [64 * S]: units of (term, row a) in which B_IJ is not all zero
    uint16_t *cols;             // [4 * S]: units of (term, column group j) in which B_IK is not all zero
    uint32_t *on;               // [4][3][kListSteps]: per wave, three lists' steps: bit 4 q + t for MFMA t of accumulator q
    uint16_t *code;             // [4][3][kListSteps]: 4 term + pixel group of these steps, and kLastStep, kLastOfRows
    int32_t *term;              // [2 * S]: unique-block pairs of the class
    int32_t *tile;              // [rows * stride]: tile I of (member row, term)
    int stride;
};

__device__ __forceinline__ F64Lds f64_lds(char *p, int S, int rows) {
    F64Lds l;
    l.stage = p;
    l.blk = (int32_t *)(p + 3 * f64_stage_bytes(rows));
    l.mask = (uint16_t *)(l.blk + 192);          // 8-byte aligned, as cols: read four at a time
    l.cols = l.mask + 64 * S;
    l.code = l.cols + 4 * S;
    l.term = (int32_t *)(l.code + 12 * kListSteps);
    l.on = (uint32_t *)(l.term + 2 * S);
    l.tile = (int32_t *)(l.on + 12 * kListSteps);
    l.stride = S | 1;                        // odd: rows fall on different banks
    return l;
}

// One 16-byte load per lane straight into LDS: lane l's value goes to byte lds +
// 16 l (uniform lds).  Counted in vmcnt; the compiler knows of neither, so the
// waits are written out where the staged data change hands.
// It writes m0, which the compiler does not let an asm name as clobbered: nothing
// else in these kernels uses it (LDS instructions do not on gfx950, and no
// register array is indexed by a variable).
__device__ __forceinline__ void load_to_lds(const void *src, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(__builtin_amdgcn_readfirstlane(lds)), "v"(src) : "memory");
}
// The same with a uniform address and a byte offset per lane.  A vector memory
// instruction may read a scalar register that a vector instruction wrote (the
// address comes from v_readfirstlane) only five wait states later; the compiler
// does not see the load, so the asm brings all five (s_mov one, s_nop 3 four).
__device__ __forceinline__ void load_to_lds(const void *uniform_src, uint32_t offset, uint32_t lds) {
    const uint64_t p = (uint64_t)(uintptr_t)uniform_src;
    const uint64_t src = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)p) |
                         (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(p >> 32)) << 32;
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 3\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(__builtin_amdgcn_readfirstlane(lds)), "v"(offset), "s"(src) : "memory");
}

// Every load but the N youngest memory operations done, and LDS traffic too;
// then the workgroup's barrier.
template <int N>
__device__ __forceinline__ void wait_and_barrier() {
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

__device__ __forceinline__ bool not_finite(double v) {
    return ((uint32_t)(__builtin_bit_cast(uint64_t, v) >> 32) & 0x7ff00000u) == 0x7ff00000u;
}

template <int NI, bool WD, bool ALL, bool BATCH>
__device__ __forceinline__ void class_f64_tile(const ProblemDesc64 &pd, int item, int part, int parts, const F64Lds &lds) {
    constexpr int R = f64_rows(NI);
    constexpr int kWRows = NI == 4 ? 64 : 32;    // rows of W staged
    constexpr int kStageU2 = kWRows * 128, kStageU1 = kStageU2 + 64 * 128, kStage = f64_stage_bytes(kWRows);
    const double *__restrict__ ut = pd.u64t;
    const double *__restrict__ wv = pd.w;
    double *__restrict__ out = pd.out;
    const int tid = thread_index<BATCH>();
    const int cls = pd.mtiles[4 * item], m0 = pd.mtiles[4 * item + 1];
    const DevClass cl = pd.classes[cls];
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63, lr = lane & 15, lk = lane >> 4;
    const int nterms = __builtin_amdgcn_readfirstlane(cl.nterms);
    const int32_t *terms = pd.cterms + 2 * cl.term0;
    if (nterms == 0) {
        if (part == 0) empty_class_tile<256, WD>(pd, cl, m0, 16 * NI);
        return;
    }

    for (int x = tid; x < 16 * NI * nterms; x += 256) {
        const int r = x / nterms, e = x - r * nterms;
        const int m = min(m0 + r, cl.nblocks - 1);   // rows past the class repeat its last member
        lds.tile[r * lds.stride + e] = pd.citab[cl.itab0 + (int64_t)m * nterms + e];
    }
    if (tid < 64) {
        const int blk = lane < 16 * NI && m0 + lane < cl.nblocks ? pd.cblk[cl.blk0 + m0 + lane] : -1;
        lds.blk[lane] = blk;
        lds.blk[128 + (lane & 48) + 4 * (lane & 3) + (lane >> 2 & 3)] = blk;
        if constexpr (WD) lds.blk[64 + lane] = blk >= 0 ? pd.blk_uid[blk] : 0;   // D-hat source block
    }
    for (int x = tid; x < 2 * nterms; x += 256) lds.term[x] = terms[x];
    // A kernel without a cut has no zeros worth a look: every step runs in full,
    // and nothing is asked of N^-1 (lmax 256 with 512: 3363 -> 3287 us)
    bool all = ALL || pd.cut == 0;
    if (!all) {
        for (int x = tid; x < 32 * nterms; x += 256)                       // 64 masks of 2 bytes per term
            ((uint32_t *)lds.mask)[x] = ((const uint32_t *)pd.units)[(int64_t)terms[2 * (x >> 5)] * 32 + (x & 31)];
        for (int x = tid; x < 4 * nterms; x += 256)
            lds.cols[x] = pd.unit_cols[(int64_t)terms[2 * (x >> 2) + 1] * 4 + (x & 3)];
        __syncthreads();
        bool bad = *pd.overflow != 0;    // sixteen threads per (member row, term), four pixels each
        for (int r = tid >> 4; r < 16 * NI; r += 16)
            for (int e = 0; e < nterms; e += 4) {    // four loads in flight
                doublex4 v[4];
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    v[i] = *(const doublex4 *)(wv + (int64_t)lds.tile[r * lds.stride + min(e + i, nterms - 1)] * 64 + 4 * lr);
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int t = 0; t < 4; ++t) bad |= not_finite(v[i][t]);
            }
        all = __syncthreads_or(bad) != 0;
    }
    if (all) {
        for (int x = tid; x < 32 * nterms; x += 256) ((uint32_t *)lds.mask)[x] = 0xffffffffu;
        for (int x = tid; x < 2 * nterms; x += 256) ((uint32_t *)lds.cols)[x] = 0xffffffffu;
        __syncthreads();
    }

    // Row groups: R rows each, or the phases of a symmetric class one after the
    // other (phase p in groups of 4 f64_sym_rows rows, from group first[p] on).
    constexpr int kRows[4] = {4 * f64_sym_rows(NI, 0), 4 * f64_sym_rows(NI, 1), 4 * f64_sym_rows(NI, 2), 4 * f64_sym_rows(NI, 3)};
    constexpr int kFirst[5] = {0, 16 / kRows[0], 16 / kRows[0] + 16 / kRows[1], 16 / kRows[0] + 16 / kRows[1] + 16 / kRows[2],
                               16 / kRows[0] + 16 / kRows[1] + 16 / kRows[2] + 16 / kRows[3]};
    const bool sym = __builtin_amdgcn_readfirstlane(cl.sym) != 0;
    auto phase_of = [&](int g) { return !sym || g < kFirst[1] ? 0 : g < kFirst[2] ? 1 : g < kFirst[3] ? 2 : 3; };
    auto rows_of = [&](int g) { const int p = phase_of(g); return !sym ? R : p == 0 ? kRows[0] : p == 1 ? kRows[1] : p == 2 ? kRows[2] : kRows[3]; };
    auto row0_of = [&](int g) {
        const int p = phase_of(g);
        return !sym ? R * g : 16 * p + rows_of(g) * (g - (p == 0 ? 0 : p == 1 ? kFirst[1] : p == 2 ? kFirst[2] : kFirst[3]));
    };
    const int ng = sym ? kFirst[4] : 64 / R;
    parts = min(parts, ng);
    if (part >= parts) return;
    const int g_begin = ng * part / parts, g_end = ng * (part + 1) / parts;   // this workgroup's groups

    // A unit: 16 terms of a row group.  Its steps, and this wave's MFMAs of them,
    // into list `slot`: lane l looks at pixel group l & 3 of the unit's term l / 4.
    // Every wave builds its own (the steps are the same for all).  At least two
    // steps: the first pixel group left out fills up, with no MFMA.
    struct Unit { int g, k; };
    const int units = (nterms + 15) >> 4;        // per row group
    auto after_unit = [&](const Unit &u) { return u.k + 1 < units ? Unit{u.g, u.k + 1} : Unit{u.g + 1, 0}; };
    uint16_t *const codes = lds.code + 3 * kListSteps * wave;
    uint32_t *const ons = lds.on + 3 * kListSteps * wave;
    auto build = [&](const Unit &u, int slot) __attribute__((always_inline)) {
        uint16_t *code = codes + kListSteps * slot;
        uint32_t *on = ons + kListSteps * slot;
        const int a0 = row0_of(u.g), nr = rows_of(u.g), jlo = phase_of(u.g);
        const int e0 = 16 * u.k + (lane >> 2), e = min(e0, nterms - 1), G = lane & 3;
        // bits 16 j + t of c: column group j; bits 16 r + t of m: row r of four
        const uint64_t nib = 0x000f000f000f000full;
        uint64_t c = *(const uint64_t *)(lds.cols + 4 * e) >> (4 * G) & nib;
        if (jlo > 0) c = c >> (16 * jlo) << (16 * jlo);
        uint32_t any_c = (uint32_t)c | (uint32_t)(c >> 32), bits = 0, any_m = 0;
        any_c |= any_c >> 16;
        if (!sym) {
            if (wave != 0) c = c >> (16 * wave) | c << (64 - 16 * wave);   // column group (w + r) mod 4 to place r
#pragma unroll
            for (int r = 0; r < R; r += 4) {
                const uint64_t m = *(const uint64_t *)(lds.mask + 64 * e + a0 + r) >> (4 * G) & nib, x = m & c;
                any_m |= (uint32_t)m | (uint32_t)(m >> 32);
                const uint32_t lo = (uint32_t)x, hi = (uint32_t)(x >> 32);
                bits |= (((lo | lo >> 12) & 255u) | ((hi | hi >> 12) & 255u) << 8) << (4 * r);
            }
        } else {
            const int nj = 4 - jlo;
            for (int r = 0; r < nr; r += 4) {
                const uint64_t m = *(const uint64_t *)(lds.mask + 64 * e + a0 + r) >> (4 * G) & nib;
                any_m |= (uint32_t)m | (uint32_t)(m >> 32);
                const uint32_t own = (uint32_t)(m >> (16 * wave)) & 15u;
                for (int j = jlo; j < 4; ++j) bits |= (own & (uint32_t)(c >> (16 * j))) << (4 * (r / 4 * nj + j - jlo));
            }
        }
        any_m |= any_m >> 16;
        const bool in = e0 < nterms && (any_m & any_c & 15u) != 0;
        const uint64_t in_b = __ballot(in);
        const int n = __popcll(in_b), first = kListSteps * u.k;   // code of lane 0: 4 term + pixel group
        const int end = kLastStep | (u.k + 1 == units ? kLastOfRows : 0);
        if (in) {
            const int i = __builtin_amdgcn_mbcnt_hi((uint32_t)(in_b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)in_b, 0));
            code[i] = (uint16_t)((first + lane) | (i > 0 && i == n - 1 ? end : 0));
            on[i] = bits;
        }
        if (lane < 2 - n) {
            code[n + lane] = (uint16_t)((first + __ffsll((unsigned long long)~in_b) - 1) | (n + lane == 1 ? end : 0));
            on[n + lane] = 0;
        }
        // read by other lanes of this wave
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };

    // Staging of one step, 16 bytes per lane and load: row r (a member row of W,
    // a column of B_IK, a row of B_IJ) keeps its 16-byte chunk c (pixels 8 (c /
    // 2) + 2 (c mod 2) and the next of the group's) at 8 r + (c ^ (r & 7)), so
    // that the eight lanes of a read phase fall on different banks.  Wave w
    // loads rows 16 w + 8 k + lane / 8 (k = 0, 1) of W (8 w + lane / 8 of 32)
    // and B_IK, and half of the rows of B_IJ.  Rows past the tile repeat its last
    // member, rows past the group its own (no wave reads them).
    const int lrow = lane >> 3, lchunk = (lane & 7) ^ lrow;
    const int lpix = 8 * (lchunk >> 1) + 2 * (lchunk & 1);
    const int wrow0 = min(kWRows / 4 * wave + lrow, 16 * NI - 1) * lds.stride;
    const int wrow1 = min(16 * wave + 8 + lrow, 16 * NI - 1) * lds.stride;      // (kWRows 64)
    const uint32_t stage0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)lds.stage;
    constexpr int kLoads = NI == 4 ? 5 : 4;      // per wave and step
    // where a step (g, code) finds its operands: its term's unique blocks, and this lane's tiles I
    struct Src { int g, code, tile0, tile1, uid1, uid2; };
    auto source = [&](int g, int code) __attribute__((always_inline)) {
        const int e = (code & (kLastOfRows - 1)) >> 2;
        return Src{g, code, lds.tile[wrow0 + e], NI == 4 ? lds.tile[wrow1 + e] : 0, lds.term[2 * e], lds.term[2 * e + 1]};
    };
    const uint32_t off2 = 8 * (lrow * 64 + lpix);                     // lane offsets into B_IK and B_IJ
    const uint32_t off1 = 8 * (((8 * (wave & 1) + lrow) & (R - 1)) * 64 + lpix);
    struct Addr { const double *w0, *w1, *u2, *u1; uint32_t off1; };
    auto addresses = [&](const Src &q) __attribute__((always_inline)) {
        const int pix = 32 * (q.code >> 1 & 1) + 4 * (q.code & 1);
        const double *w = wv + pix;
        return Addr{w + ((int64_t)q.tile0 * 64 + lpix), w + ((int64_t)q.tile1 * 64 + lpix),
                    ut + (int64_t)__builtin_amdgcn_readfirstlane(q.uid2) * kBlockElems + (16 * wave * 64 + pix),
                    ut + (int64_t)__builtin_amdgcn_readfirstlane(q.uid1) * kBlockElems + (row0_of(q.g) * 64 + pix),
                    sym ? 8 * (((8 * (wave & 1) + lrow) & (rows_of(q.g) - 1)) * 64 + lpix) : off1};
    };
    auto stage = [&](const Addr &q, uint32_t at) __attribute__((always_inline)) {
        load_to_lds(q.w0, at + 32 * kWRows * wave);
        if constexpr (NI == 4) load_to_lds(q.w1, at + 2048 * wave + 1024);
        load_to_lds(q.u2, off2, at + kStageU2 + 2048 * wave);
        load_to_lds(q.u2 + 8 * 64, off2, at + kStageU2 + 2048 * wave + 1024);
        load_to_lds(q.u1, q.off1, at + kStageU1 + 1024 * (wave & 1));   // two waves write the same
    };
    // pixels 8 lk + 2 h, 8 lk + 2 h + 1 of a staged row
    auto staged = [&](const char *rows, int r, int h) __attribute__((always_inline)) {
        return *(const doublex2 *)(rows + 128 * r + 16 * ((2 * lk + h) ^ (r & 7)));
    };

    // Steps in order: a step of group g at place `at` of the lists is followed by
    // the next place, or if it is its list's last by the next list's first; past
    // the last group it repeats (its loads go where no step reads).
    struct Cursor { int g, at; };
    auto after = [&](const Cursor &c, int code) __attribute__((always_inline)) {
        if (!(code & kLastStep)) return Cursor{c.g, c.at + 1};
        const int g = (code & kLastOfRows) ? c.g + 1 : c.g, at = (c.at & -kListSteps) + kListSteps;
        return g < g_end ? Cursor{g, at == 3 * kListSteps ? 0 : at} : c;
    };
    auto code_at = [&](const Cursor &c) __attribute__((always_inline)) { return (int)codes[c.at]; };
    auto on_at = [&](const Cursor &c) __attribute__((always_inline)) { return (int)ons[c.at]; };
    auto uniform = [&](int x) __attribute__((always_inline)) { return __builtin_amdgcn_readfirstlane(x); };

    constexpr int kDChunks = 16 * NI * 2048;   // D-hat chunks of the tile
    int stp = kDChunks / 512 * part / parts;   // steps done, counted from the first of this part's chunks
    const int dchunks = kDChunks / 512 * (part + 1) / parts * 512;
    DCopy<2> dpend;
    Unit next_unit{g_begin, 0};          // the next to be listed, and where
    int slot = 0;
    for (; slot < 3 && next_unit.g < g_end; ++slot) {
        build(next_unit, slot);
        next_unit = after_unit(next_unit);
    }
    slot = 0;
    bool begun = false;                  // past the first unit
    int code0, code1, code2, code3;
    uint32_t on;                         // on: this wave's MFMAs of this step
    Cursor c1, c2, c3;                   // the next three steps
    {
        const Cursor c0{g_begin, 0};
        code0 = uniform(code_at(c0));
        on = uniform(on_at(c0));
        c1 = after(c0, code0);
        code1 = uniform(code_at(c1));
        c2 = after(c1, code1);
        code2 = uniform(code_at(c2));
        c3 = after(c2, code2);
        code3 = uniform(code_at(c3));
        stage(addresses(source(c0.g, code0)), stage0);
        stage(addresses(source(c1.g, code1)), stage0 + kStage);
        stage(addresses(source(c2.g, code2)), stage0 + 2 * kStage);
    }
    uint32_t at = 0;                     // this step's buffer
    // The row groups [gb, ge) of this part.  SYM false: accumulator q is row q,
    // column group (w + q) mod 4; SYM true: column groups >= JLO of the rows w, w + 4, ...
    auto groups = [&](auto symt, auto jt, int gb, int ge) __attribute__((always_inline)) {
        constexpr bool SYM = decltype(symt)::value;
        constexpr int JLO = decltype(jt)::value, NR = SYM ? f64_sym_rows(NI, JLO) : R, NJ = SYM ? 4 - JLO : 1;
        auto row = [&](int q) { return SYM ? wave + 4 * (q / NJ) : q; };
        auto col = [&](int q) { return SYM ? JLO + q % NJ : (wave + q) & 3; };
        for (int g = max(gb, g_begin); g < min(ge, g_end); ++g) {
            const int a0 = row0_of(g);
            doublex4 acc[NR * NJ][NI];
#pragma unroll
            for (int q = 0; q < NR * NJ; ++q)
#pragma unroll
                for (int i = 0; i < NI; ++i) acc[q][i] = doublex4{0.0, 0.0, 0.0, 0.0};
            for (bool done = false; !done;) {
            if (begun && next_unit.g < g_end) {      // listed two units ahead, in the place of the one just done
                build(next_unit, slot);
                next_unit = after_unit(next_unit);
                slot = slot == 2 ? 0 : slot + 1;
            }
            begun = true;
            for (bool last = false; !last;) {
                // read now, used after the MFMAs: what the loads of three steps on need, the code of the step
                // after that, the next step's masks
                const Src src = source(c3.g, code3);
                const Cursor c4 = after(c3, code3);
                const int code4 = code_at(c4);
                const int on1 = on_at(c1);
                if constexpr (WD) {
                    dcopy_load<256>(pd.du64, pd.outD, lds.blk, dchunks, stp, wave, lane, dpend);
                    ++stp;
                }
                const char *sw = lds.stage + at, *su2 = sw + kStageU2, *su1 = sw + kStageU1;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    constexpr int NC = SYM ? NJ : 4;
                    doublex2 u1[NR], u2[NC], w[NI];
#pragma unroll
                    for (int r = 0; r < NR; ++r) u1[r] = staged(su1, row(r * NJ), h);
#pragma unroll
                    for (int j = 0; j < NC; ++j) u2[j] = staged(su2, 16 * (SYM ? JLO + j : (wave + j) & 3) + lr, h);
#pragma unroll
                    for (int i = 0; i < NI; ++i) w[i] = staged(sw, 16 * i + lr, h);
#pragma unroll
                    for (int t = 0; t < 2; ++t)
#pragma unroll
                        for (int q = 0; q < NR * NJ; ++q)
                            if (ALL || (on & (1u << (4 * q + 2 * h + t)))) {
                                const double bv = u1[q / NJ][t] * u2[SYM ? q % NJ : q & 3][t];
#pragma unroll
                                for (int i = 0; i < NI; ++i)
                                    acc[q][i] = __builtin_amdgcn_mfma_f64_16x16x4f64(w[i][t], bv, acc[q][i], 0, 0, 0);
                            }
                }
                const Addr ad = addresses(src);
                last = (code0 & kLastStep) != 0;
                done = (code0 & kLastOfRows) != 0;
                c1 = c2;
                c2 = c3;
                c3 = c4;
                code0 = code1;
                code1 = code2;
                code2 = code3;
                code3 = uniform(code4);
                on = uniform(on1);
                // the next step's loads are done in every wave, and nobody reads this step's buffer any more
                wait_and_barrier<kLoads + (WD ? 2 : 0)>();
                if constexpr (WD) dcopy_store(dpend, lane);
                stage(ad, stage0 + at);
                at = at == 2 * kStage ? 0 : at + kStage;
            }
            }
            // store the group's rows (and their mirror images below the diagonal in a symmetric class)
            typedef int32_t intx4 __attribute__((ext_vector_type(4)));
            intx4 blk[NI];
#pragma unroll
            for (int i = 0; i < NI; ++i) blk[i] = *(const intx4 *)(lds.blk + 128 + 16 * i + 4 * lk);
#pragma unroll
            for (int i = 0; i < NI; ++i)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    if (blk[i][v] >= 0) {
                        double *ob = out + (int64_t)blk[i][v] * kBlockElems;
#pragma unroll
                        for (int q = 0; q < NR * NJ; ++q) {
                            const int a = a0 + row(q), b = 16 * col(q) + lr;
                            __builtin_nontemporal_store(acc[q][i][v], &ob[a * 64 + b]);
                            if (SYM && q % NJ > 0) ob[b * 64 + a] = acc[q][i][v];
                        }
                    }
                }
        }
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;
    using I3 = std::integral_constant<int, 3>;
    if (sym) {
        wait_and_barrier<2 * kLoads>();
        groups(std::true_type(), I0(), kFirst[0], kFirst[1]);
        groups(std::true_type(), I1(), kFirst[1], kFirst[2]);
        groups(std::true_type(), I2(), kFirst[2], kFirst[3]);
        groups(std::true_type(), I3(), kFirst[3], kFirst[4]);
    } else {
        wait_and_barrier<2 * kLoads>();
        groups(std::false_type(), I0(), 0, 64 / R);
    }
    wait_and_barrier<0>();               // no load into LDS outlives the tile
    if constexpr (WD) {                  // the chunks past the last step
        for (; 512 * stp < dchunks; ++stp) {
            DCopy<2> dc;
            dcopy_load<256>(pd.du64, pd.outD, lds.blk, dchunks, stp, wave, lane, dc);
            dcopy_store(dc, lane);
        }
    }
}

// ALL: for kernels without a cut, every MFMA and no test of them.  Measured
// against tests that all say yes / the full contraction that loaded its operands
// per wave: lmax 1500 11.42 / 12.0 -> 11.15 ms, lmax 512 with 1126 24.2 / 22.3 ->
// 21.7, 256 with 589 5.85 / 5.70 -> 5.27.
template <bool WD, bool ALL>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
void k_class_f64(ProblemDesc64 pd) {
    extern __shared__ __align__(16) char smem[];
    const F64Lds lds = f64_lds(smem, pd.max_terms, pd.tile_rows);
    const int item = blockIdx.x;        // pd.mtiles: a dispatch table, slot per workgroup
    const int groups = pd.mtiles[4 * item + 2];
    if (groups == 0) return;            // an empty slot
    if (groups == 4) class_f64_tile<4, WD, ALL, false>(pd, item, blockIdx.y, gridDim.y, lds);
    else if (groups == 2) class_f64_tile<2, WD, ALL, false>(pd, item, blockIdx.y, gridDim.y, lds);
    else class_f64_tile<1, WD, ALL, false>(pd, item, blockIdx.y, gridDim.y, lds);
}

// Queue draining shared by the persistent batch kernels: thread 0 takes the
// next item from queue home, then steals from the others in order; -1 once
// every queue is empty.  Counters only grow, so every workgroup leaves.  Every
// item is taken in `parts` parts: the result is parts times the item, plus the part.
__device__ __forceinline__ int batch_next_item(const int32_t *__restrict__ qb, int32_t nq,
                                               int32_t *__restrict__ counters, int home, int &tried, int parts = 1) {
    int it = -1;
    while (tried < nq) {
        const int q = (home + tried) % nq;
        const int c = atomicAdd(&counters[q], 1);
        if (c < (qb[q + 1] - qb[q]) * parts) {
            it = qb[q] * parts + c;
            break;
        }
        ++tried;
    }
    return it;
}

// a10 in FP64: the FP64 class GEMM of many problems in one persistent launch
// (two 4-wave workgroups per CU, as k_class_f64), fed by the same queues as the
// FP32 and split-BF16 batch kernels below.
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
void k_batch_f64(const ProblemDesc64 *__restrict__ probs, const int32_t *__restrict__ items,
                 const int32_t *__restrict__ qb, int32_t nq, int32_t *__restrict__ counters, int32_t max_terms,
                 int32_t parts) {
    extern __shared__ __align__(16) char smem[];
    __shared__ int32_t sItem;
    const F64Lds lds = f64_lds(smem, max_terms, 64);
    const int home = blockIdx.x % nq;
    int tried = 0;                       // queues found empty (thread 0)
    for (;;) {
        if (threadIdx.x == 0) sItem = batch_next_item(qb, nq, counters, home, tried, parts);
        __syncthreads();
        const int it = __builtin_amdgcn_readfirstlane(sItem);   // uniform: descriptors in scalar registers
        __syncthreads();                 // every thread has read sItem before it changes
        if (it < 0) break;
        const int at = it / parts, part = it % parts;
        const ProblemDesc64 pd = probs[items[2 * at]];
        const int item = items[2 * at + 1];
        const int groups = pd.mtiles[4 * item + 2];
        if (groups == 4) class_f64_tile<4, false, false, true>(pd, item, part, parts, lds);
        else if (groups == 2) class_f64_tile<2, false, false, true>(pd, item, part, parts, lds);
        else class_f64_tile<1, false, false, true>(pd, item, part, parts, lds);
    }
}

// ---------------------------------------------------------------------------
// a9, FP32 MFMA class GEMM.  Same decomposition as the split-BF16 form below:
// C[m][(a,b)] = sum_(e,p) W[m][(e,p)] M[(e,p)][(a,b)], W = N^-1 rounded to FP32,
// M = B_IJ[p][a] B_IK[p][b] formed as the FP32 product of the FP32 copies.
// The same schedule as the split-BF16 kernel: eight waves per member tile,
// wave w the output rows a = w mod 4 and the column half w / 4, two waves per
// SIMD; W and the B_IK values of a step (32 pixels) staged through four LDS
// buffers two steps ahead, one barrier per term.  MFMA 16x16x4 FP32, MFMA g
// of a step taking the pixels 8 lk + g; the result lane holds members
// 16 i + 4 lk + v of column b = 16 j + lr.  A term's FP32 sum over its 64
// pixels is added to FP64 accumulators, which are stored and cleared at the
// end of every row a.
// ---------------------------------------------------------------------------
// What a member tile of the FP32 and split-BF16 kernels leaves out, in LDS: the
// masks of its class's terms (as in the FP64 form) and, row quad by row quad (a
// = 4 x .. 4 x + 3, one row per row phase), the terms in which any of the four
// rows and any column can be nonzero, 256 x + term, at least one per quad.  A
// term's steps and its sum stay together, so the results are those of the
// full contraction bit for bit.  An FP32 wave tests each MFMA (a unit of one
// column group), a split-BF16 one each half term (its products are split and
// scheduled together).  Measured, beam 3 pixels, lmax 1500, contraction: FP32
// 7.00 -> 5.57 ms, BF16x6 4.78 -> 4.47; FP32 on the two-hop pattern (lmax 701,
// 2.3 pixels) 3.05 -> 1.78.
struct SkipLds {
    uint16_t mask[kMaxClassTerms * 64];   // units of (term, row a) in which B_IJ is not all zero
    uint16_t cols[kMaxClassTerms * 4];    // units of (term, column group j) in which B_IK is not all zero
    uint16_t list[16 * kMaxClassTerms];
};

// Fills it (512 threads; sTerm and the tile's W are there): w_finite(r, e, c)
// tells whether pixels 4 c .. 4 c + 3 of member row r, term e are finite.  Only
// the row quads of this part of the tile are listed.  Returns the length of the
// list.
template <int NI, class PD, class Finite>
__device__ __forceinline__ int build_skip(const PD &pd, int nterms, int part, int parts, const int32_t *sTerm, SkipLds &sk,
                                          const Finite &w_finite) {
    const int tid = threadIdx.x, lane = tid & 63;
    for (int x = tid; x < 32 * nterms; x += 512)
        ((uint32_t *)sk.mask)[x] = ((const uint32_t *)pd.units)[(int64_t)sTerm[2 * (x >> 5)] * 32 + (x & 31)];
    for (int x = tid; x < 4 * nterms; x += 512) sk.cols[x] = pd.unit_cols[(int64_t)sTerm[2 * (x >> 2) + 1] * 4 + (x & 3)];
    bool bad = *pd.overflow != 0;        // sixteen threads per (member row, term), four pixels each
    for (int r = tid >> 4; r < 16 * NI; r += 32)
        for (int e = 0; e < nterms; e += 8) {        // eight loads in flight
            bool b[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) b[i] = !w_finite(r, min(e + i, nterms - 1), tid & 15);
#pragma unroll
            for (int i = 0; i < 8; ++i) bad |= b[i];
        }
    if (__syncthreads_or(bad)) {
        for (int x = tid; x < 32 * nterms; x += 512) ((uint32_t *)sk.mask)[x] = 0xffffffffu;
        for (int x = tid; x < 2 * nterms; x += 512) ((uint32_t *)sk.cols)[x] = 0xffffffffu;
        __syncthreads();
    }
    // every wave writes the same list, and reads what it wrote itself
    int total = 0;
    for (int x = 16 * part / parts; x < 16 * (part + 1) / parts; ++x) {
        const int first = total;
        for (int e0 = 0; e0 < nterms; e0 += 64) {
            const int e = min(e0 + lane, nterms - 1);
            const uint64_t m = *(const uint64_t *)(sk.mask + 64 * e + 4 * x), c = *(const uint64_t *)(sk.cols + 4 * e);
            uint32_t mm = (uint32_t)m | (uint32_t)(m >> 32), cc = (uint32_t)c | (uint32_t)(c >> 32);
            mm |= mm >> 16;
            cc |= cc >> 16;
            const bool take = e0 + lane < nterms && (mm & cc & 0xffffu) != 0;
            const uint64_t b = __ballot(take);
            if (take)
                sk.list[total + __builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, 0))] =
                    (uint16_t)(256 * x + e);
            total += __popcll(b);
        }
        if (total == first) {
            if (lane == 0) sk.list[total] = (uint16_t)(256 * x);
            ++total;
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    return __builtin_amdgcn_readfirstlane(total);
}

__global__ __launch_bounds__(256) void k_ninv_f32(const double *__restrict__ ninv, int64_t n,
                                                  float *__restrict__ wf) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) wf[i] = (float)ninv[i];
}

// One member tile (item) of one problem with NI groups of 16 member rows; all
// 512 threads of the workgroup take part.  sTile / sBlk / sTerm are the
// workgroup's LDS tables, sW / sU its four staging buffers.
template <int NI, bool WD, bool SKIP, bool BATCH>
__device__ __forceinline__ void class_f32_tile(const ProblemDesc &pd, int item, int part, int parts, int32_t *sTile,
                                               int32_t *sBlk, int32_t *sTerm, floatx4 *sW, floatx4 *sU, SkipLds *sk) {
    const float *__restrict__ ut32 = pd.ut32;
    double *__restrict__ out = pd.out;
    constexpr int NW = 8, NT = 64 * NW, RP = NW / 2;
    const int tid = thread_index<BATCH>();
    const int cls = pd.mtiles[4 * item], m0 = pd.mtiles[4 * item + 1];
    const DevClass cl = pd.classes[cls];
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rw = wave % RP, ch = wave / RP;          // row phase, column half
    const int lane = tid & 63, lr = lane & 15, lk = lane >> 4;
    const int nterms = cl.nterms;
    const int32_t *terms = pd.cterms + 2 * cl.term0;
    if (nterms == 0) {
        if (part == 0) empty_class_tile<NT, WD>(pd, cl, m0, 16 * NI);
        return;
    }

    for (int x = tid; x < 16 * NI * nterms; x += NT) {
        const int r = x / nterms, e = x - r * nterms;
        const int m = min(m0 + r, cl.nblocks - 1);   // rows past the class repeat its last member
        sTile[r * kTileStride + e] = pd.citab[cl.itab0 + (int64_t)m * nterms + e];
    }
    if (tid < 64) {
        const int blk = lane < 16 * NI && m0 + lane < cl.nblocks ? pd.cblk[cl.blk0 + m0 + lane] : -1;
        sBlk[lane] = blk;
        if constexpr (WD) sBlk[64 + lane] = blk >= 0 ? pd.blk_uid[blk] : 0;   // D-hat source block
    }
    if (tid < 2 * nterms) sTerm[tid] = terms[tid];   // unique-block pairs of the class
    __syncthreads();
    // SKIP false: every term of every row, in order
    const int quad0 = 16 * part / parts;
    int total = (16 * (part + 1) / parts - quad0) * nterms;
    if constexpr (SKIP) total = build_skip<NI>(pd, nterms, part, parts, sTerm, *sk, [&](int r, int e, int c) {
        const floatx4 v = *(const floatx4 *)(pd.wf + (int64_t)sTile[r * kTileStride + e] * 64 + 4 * c);
        return fabsf(v[0]) < INFINITY && fabsf(v[1]) < INFINITY && fabsf(v[2]) < INFINITY && fabsf(v[3]) < INFINITY;
    });

    // Staging of one step (32 pixels of a term): W of the tile's 64 rows and
    // the B_IK values of its 64 columns, FP32, 8 chunks of 16 bytes per row
    // each; thread t takes W chunk t (row t >> 3) and B_IK chunk t.  Rows past
    // the tile's 16 NI members load the last member's values into LDS rows no
    // wave reads.  LDS row r keeps its chunk c at 8 r + (c ^ usw(r)).
    auto usw = [](int b) { return ((b >> 1) ^ (b << 2)) & 7; };
    const int srow = tid >> 3, sch = tid & 7;
    const int wrow = min(srow, 16 * NI - 1) * kTileStride;
    const int sdst = srow * 8 + (sch ^ usw(srow));
    struct SAddr { int64_t wo; const float *u2; };
    struct OAddr { const float *p1; };
    auto saddr = [&](int e, int h) {
        SAddr r;
        r.wo = (int64_t)sTile[wrow + e] * 64 + 32 * h + 4 * sch;
        r.u2 = ut32 + (int64_t)__builtin_amdgcn_readfirstlane(sTerm[2 * e + 1]) * kBlockElems + 32 * h;
        return r;
    };
    // this lane's B_IJ values of row a: pixels 32 h + 8 lk + g, g = 0..7
    auto oaddr = [&](int a, int e, int h) {
        OAddr r;
        r.p1 = ut32 + (int64_t)__builtin_amdgcn_readfirstlane(sTerm[2 * e]) * kBlockElems + a * 64 + 32 * h + 8 * lk;
        return r;
    };
    struct Stage { floatx4 w, u; };
    struct Own { floatx4 u1[2]; };
    auto stage_load = [&](const SAddr &ad, Stage &st) {
        st.w = *(const floatx4 *)(pd.wf + ad.wo);
        st.u = *(const floatx4 *)(ad.u2 + srow * 64 + 4 * sch);
    };
    auto own_load = [&](const OAddr &ad, Own &o) {
        o.u1[0] = *(const floatx4 *)ad.p1;
        o.u1[1] = *(const floatx4 *)(ad.p1 + 4);
    };
    auto stage_store = [&](const Stage &st, int buf) {
        sW[buf * 512 + sdst] = st.w;
        sU[buf * 512 + sdst] = st.u;
    };
    // this part's D-hat chunks of the tile, two per thread and step: steps dstep .. dchunks / (2 NT)
    constexpr int kDSteps = 16 * NI * 2048 / (2 * NT);
    const int dstep = kDSteps * part / parts, dchunks = kDSteps * (part + 1) / parts * 2 * NT;

    doublex4 acc[NI][2];
    floatx4 psum[NI][2];
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = doublex4{0.0, 0.0, 0.0, 0.0};
    // One step, in three scheduling regions as in the split-BF16 form.  MFMA
    // g (g = 0..7) of a step takes the pixels 8 lk + g: lane (lr, lk) holds
    // W[16 i + lr][8 lk + g] and M[8 lk + g][16 j + lr].
    auto step = [&](const Own &oc, int buf, const SAddr &sa, const OAddr &oa, int sbuf, Stage &stn, Own &on,
                    int h, uint32_t on0, uint32_t on1, bool bar, int nse, int nsh, int noa, int noe, int noh, SAddr &sa_n, OAddr &oa_n,
                    int stp, DCopy<2> &dprev, auto symt, int ng, int g0, int g1) {
        constexpr bool S = decltype(symt)::value;
        stage_load(sa, stn);
        own_load(oa, on);
        if constexpr (WD) {
            DCopy<2> dc;
            dcopy_load<NT>(pd.du64, pd.outD, sBlk, dchunks, stp, wave, lane, dc);
            dcopy_store(dprev, lane);
            dprev = dc;
        }
        __builtin_amdgcn_sched_barrier(0);
        floatx4 wfr[NI][2];
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int r = 16 * i + lr;
#pragma unroll
            for (int hh = 0; hh < 2; ++hh) wfr[i][hh] = sW[buf * 512 + r * 8 + ((2 * lk + hh) ^ usw(r))];
        }
#pragma unroll
        for (int jj = 0; jj < 2; ++jj) {
            // bit g: ring g of this half's four columns can be nonzero
            const uint32_t rings = (jj ? on1 : on0) >> (8 * h) & 255u;
            if (SKIP ? rings == 0 : S && jj >= ng) continue;   // symmetric class: this wave's groups of the row
            const int b = S ? 16 * (jj ? g1 : g0) + lr : 32 * ch + 16 * jj + lr;
            float m[8];
#pragma unroll
            for (int hh = 0; hh < 2; ++hh) {
                const floatx4 u2 = sU[buf * 512 + b * 8 + ((2 * lk + hh) ^ usw(b))];
#pragma unroll
                for (int t = 0; t < 4; ++t) m[4 * hh + t] = oc.u1[hh][t] * u2[t];
            }
#pragma unroll
            for (int g = 0; g < 8; ++g)
                if (!SKIP || (rings & (1u << g)) != 0) {
#pragma unroll
                    for (int i = 0; i < NI; ++i)
                        psum[i][jj] = __builtin_amdgcn_mfma_f32_16x16x4f32(wfr[i][g >> 2][g & 3], m[g],
                                                                           !SKIP && h == 0 && g == 0 ? floatx4{0.f, 0.f, 0.f, 0.f} : psum[i][jj], 0, 0, 0);
                }
        }
        sa_n = saddr(nse, nsh);
        oa_n = oaddr(noa, noe, noh);
        __builtin_amdgcn_sched_barrier(0);
        stage_store(stn, sbuf);
        if (bar) __syncthreads();
        __builtin_amdgcn_sched_barrier(0);
    };

    // Four LDS buffers: iteration it (one term of one row) computes from
    // buffers 2 (it & 1) + h, fills the other pair for iteration it + 1, and
    // ends with the only barrier of the term.
    // entry it of the list (past its end the last one), and this wave's MFMAs of
    // an entry, read one iteration ahead: bit 8 h + g of a column group
    auto entry = [&](int it, int before) {   // before: entry it - 1
        if constexpr (SKIP) return (int)sk->list[min(it, total - 1)];
        else if (it == 0) return 256 * quad0;
        else if (it >= total) return before;
        else return (before & 255) + 1 < nterms ? before + 1 : (before | 255) + 1;
    };
    auto uniform = [&](int v) { return __builtin_amdgcn_readfirstlane(v); };
    struct Groups { int ng, g0, g1; };
    auto groups_of = [&](auto symt, int x) {
        Groups q{2, 2 * ch, 2 * ch + 1};
        if constexpr (decltype(symt)::value) {
            const int p = x >> 2;
            if (p == 1 && ch == 0) q = Groups{1, 1, 1};
            else if (p == 2) q = Groups{1, 2 + ch, 2 + ch};
            else if (p == 3) q = Groups{ch, 3, 3};
        }
        return q;
    };
    auto on_of = [&](int c, const Groups &q, uint32_t &o0, uint32_t &o1) {
        if constexpr (SKIP) {
            const uint32_t m = sk->mask[64 * (c & 255) + rw + RP * (c >> 8)];
            o0 = q.ng > 0 ? m & sk->cols[4 * (c & 255) + q.g0] : 0u;
            o1 = q.ng > 1 ? m & sk->cols[4 * (c & 255) + q.g1] : 0u;
        }
    };
    Stage s0, s1;
    Own o0, o1;
    int c0 = uniform(entry(0, 0)), c1 = uniform(entry(1, c0));   // this iteration and the next
    {
        Stage t0, t1;
        stage_load(saddr(c0 & 255, 0), t0);
        stage_load(saddr(c0 & 255, 1), t1);
        own_load(oaddr(rw + RP * (c0 >> 8), c0 & 255, 0), o0);
        stage_store(t0, 0);
        stage_store(t1, 1);
    }
    SAddr sa = saddr(c1 & 255, 0);
    OAddr oa = oaddr(rw + RP * (c0 >> 8), c0 & 255, 1);
    DCopy<2> dpend;                           // D-hat chunks loaded, not yet stored
    dpend.clear();
    __syncthreads();
    // Symmetric classes (every term pairs a unique block with itself: the
    // blocks (J, J), with C[a][b] = C[b][a] bit for bit since the products
    // B[p][a] B[p][b] are the same numbers either way round): row a needs only
    // the column groups j >= a / 16 (= x / 4, as a = rw + 4 x); the tiles
    // below the diagonal are written as mirror images.  The groups a row needs
    // are shared out so that the two waves of a row phase (column halves 0
    // and 1) do at most two groups each and one each where two are left:
    // x / 4 = 0: {0, 1} | {2, 3};  1: {1} | {2, 3};  2: {2} | {3};  3: {} | {3}.
    auto rows = [&](auto symt) {
        constexpr bool S = decltype(symt)::value;
        Groups gr = groups_of(symt, c0 >> 8);
        uint32_t on0 = 0, on1 = 0;           // (SKIP)
        on_of(c0, gr, on0, on1);
        on0 = uniform(on0);
        on1 = uniform(on1);
        for (int it = 0; it < total; ++it) {
            const int raw2 = entry(it + 2, c1);
            const int x = c0 >> 8, x1 = c1 >> 8, e1 = c1 & 255, p = x >> 2;
            const int a = rw + RP * x, a1 = rw + RP * x1;
            const int ng = gr.ng, g0 = gr.g0, g1 = gr.g1;
            const Groups gn = groups_of(symt, x1);
            uint32_t raw_on0 = 0, raw_on1 = 0;
            on_of(c1, gn, raw_on0, raw_on1);
            if constexpr (SKIP) {
#pragma unroll
                for (int i = 0; i < NI; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j) psum[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
            }
            const int ib = 2 * (it & 1), nb = 2 - ib;
            step(o0, ib, sa, oa, nb, s1, o1, 0, on0, on1, false, e1, 1, a1, e1, 0, sa, oa, dstep + 2 * it, dpend, symt, ng, g0, g1);
            const int c2 = uniform(raw2);
            step(o1, ib + 1, sa, oa, nb + 1, s0, o0, 1, on0, on1, true, c2 & 255, 0, a1, e1, 1, sa, oa, dstep + 2 * it + 1, dpend, symt,
                 ng, g0, g1);
#pragma unroll
            for (int i = 0; i < NI; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    if (SKIP ? (j ? on1 : on0) != 0 : !S || j < ng) {
#pragma unroll
                        for (int v = 0; v < 4; ++v) acc[i][j][v] += (double)psum[i][j][v];
                    }
            if (x1 != x || it + 1 == total) {    // end of output row a: store, clear
#pragma unroll
                for (int i = 0; i < NI; ++i)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int blk = sBlk[16 * i + 4 * lk + v];
                        if (blk >= 0) {
                            double *ob = out + (int64_t)blk * kBlockElems;
#pragma unroll
                            for (int j = 0; j < 2; ++j) {
                                if (S && j >= ng) continue;
                                const int G = S ? (j ? g1 : g0) : 2 * ch + j;
                                __builtin_nontemporal_store(acc[i][j][v], &ob[a * 64 + 16 * G + lr]);
                                if (S && G > p) ob[(16 * G + lr) * 64 + a] = acc[i][j][v];
                            }
                        }
                    }
#pragma unroll
                for (int i = 0; i < NI; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j) acc[i][j] = doublex4{0.0, 0.0, 0.0, 0.0};
            }
            c0 = c1;
            c1 = c2;
            on0 = uniform(raw_on0);
            on1 = uniform(raw_on1);
            gr = gn;
        }
    };
    if (cl.sym != 0) rows(std::true_type());
    else rows(std::false_type());
    if constexpr (WD) {                  // the last step's chunks, then those past the last step
        dcopy_store(dpend, lane);
        for (int stp = dstep + 2 * total; 2 * NT * stp < dchunks; ++stp) {
            DCopy<2> dc;
            dcopy_load<NT>(pd.du64, pd.outD, sBlk, dchunks, stp, wave, lane, dc);
            dcopy_store(dc, lane);
        }
    }
}

template <bool WD, bool SKIP, bool BATCH>
__device__ __forceinline__ void class_f32_item(const ProblemDesc &pd, int item, int part, int parts, int32_t *sTile, int32_t *sBlk,
                                               int32_t *sTerm, floatx4 *sW, floatx4 *sU, SkipLds *sk) {
    const int groups = pd.mtiles[4 * item + 2];
    if (groups == 0) return;            // an empty slot of a dispatch table
    if (groups == 4) class_f32_tile<4, WD, SKIP, BATCH>(pd, item, part, parts, sTile, sBlk, sTerm, sW, sU, sk);
    else if (groups == 2) class_f32_tile<2, WD, SKIP, BATCH>(pd, item, part, parts, sTile, sBlk, sTerm, sW, sU, sk);
    else class_f32_tile<1, WD, SKIP, BATCH>(pd, item, part, parts, sTile, sBlk, sTerm, sW, sU, sk);
}

// SKIP: products that the cut makes zero are left out (a kernel of its own: with
// both forms in one, the full form at lmax 1500 took 7.04 ms, alone 6.93).
template <bool WD, bool SKIP>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
void k_class_f32(ProblemDesc pd) {
    __shared__ int32_t sTile[64 * kTileStride];   // tile I of (member row, term)
    __shared__ int32_t sBlk[128];                    // stored block per member row; D-hat source block
    __shared__ int32_t sTerm[2 * kMaxClassTerms];     // unique-block pairs of the class
    __shared__ floatx4 sW[4 * 512];                  // staged W, four buffers
    __shared__ floatx4 sU[4 * 512];                  // staged B_IK values, four buffers
    SkipLds *sk = nullptr;
    if constexpr (SKIP) {
        __shared__ SkipLds lists;
        sk = &lists;
    }
    class_f32_item<WD, SKIP, false>(pd, blockIdx.x, blockIdx.y, gridDim.y, sTile, sBlk, sTerm, sW, sU, sk);
}

// ---------------------------------------------------------------------------
// a10: many problems in one persistent launch.  Work items (problem, member
// tile) sit in nq queues, queue q holding items [qb[q], qb[q+1]).  Workgroup b
// drains queue b mod nq first (with one queue per XCD and items in natural
// order, the tiles an XCD runs together share operands in its L2), then steals
// from the others.  Counters only grow, so every workgroup leaves once all
// queues are empty.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(64) void k_fill_i32(int32_t *p, int32_t n, int32_t v) {
    for (int i = threadIdx.x; i < n; i += 64) p[i] = v;
}

__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
void k_batch_f32(const ProblemDesc *__restrict__ probs, const int32_t *__restrict__ items,
                 const int32_t *__restrict__ qb, int32_t nq, int32_t *__restrict__ counters, int32_t parts) {
    __shared__ int32_t sTile[64 * kTileStride];
    __shared__ int32_t sBlk[128];
    __shared__ int32_t sTerm[2 * kMaxClassTerms];     // unique-block pairs of the class
    __shared__ floatx4 sW[4 * 512];
    __shared__ floatx4 sU[4 * 512];
    __shared__ SkipLds sk;
    __shared__ int32_t sItem;
    const int home = blockIdx.x % nq;
    int tried = 0;                       // queues found empty (thread 0)
    for (;;) {
        if (threadIdx.x == 0) sItem = batch_next_item(qb, nq, counters, home, tried, parts);
        __syncthreads();
        const int it = __builtin_amdgcn_readfirstlane(sItem);   // uniform: descriptors in scalar registers
        __syncthreads();                 // every thread has read sItem before it changes
        if (it < 0) break;
        const int at = it / parts;
        const ProblemDesc pd = probs[items[2 * at]];
        if (pd.skip != 0) class_f32_item<false, true, true>(pd, items[2 * at + 1], it % parts, parts, sTile, sBlk, sTerm, sW, sU, &sk);
        else class_f32_item<false, false, true>(pd, items[2 * at + 1], it % parts, parts, sTile, sBlk, sTerm, sW, sU, &sk);
    }
}

// ---------------------------------------------------------------------------
// a9, split BF16.  A value is split into NP BF16 parts, each rounded to nearest
// even from the exact FP32 remainder of the previous ones: three parts
// represent an FP32 value exactly, two parts to 2^-17 relative, and every
// part has a sign independent of the value's, so the products left out
// (NP = 3: ml, lm, ll; NP = 2: mm) are unbiased.  Products kept: NP = 3: mm,
// lh, hl, mh, hm, hh (all of order >= 2^-16); NP = 2: mh, hm, hh.  FP32 MFMA
// accumulation over the 64 pixels of one contraction tile, FP64 across tiles.
// ---------------------------------------------------------------------------
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {   // round to nearest even
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((floatx2){a, b}, bf16x2));
}

template <int NP>
__device__ __forceinline__ void split_pair(float y0, float y1, uint32_t *out) {
    const uint32_t h = pack_bf16(y0, y1);
    out[0] = h;
    const float r0 = y0 - __uint_as_float(h << 16);
    const float r1 = y1 - __uint_as_float(h & 0xffff0000u);
    const uint32_t m = pack_bf16(r0, r1);
    out[1] = m;
    if constexpr (NP == 3) {
        const float l0 = r0 - __uint_as_float(m << 16);
        const float l1 = r1 - __uint_as_float(m & 0xffff0000u);
        out[2] = pack_bf16(l0, l1);
    }
}

// N^-1 split into three BF16 parts (hi, mid, lo) from FP64, read directly as
// MFMA operands by the class GEMM.
__global__ __launch_bounds__(256) void k_split_ninv(const double *__restrict__ ninv, int64_t n,
                                                    uint16_t *__restrict__ w0, uint16_t *__restrict__ w1,
                                                    uint16_t *__restrict__ w2) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double v = ninv[i];
    const uint16_t h = bf16_bits((float)v);
    const double r1 = v - (double)bf16_value(h);
    const uint16_t m = bf16_bits((float)r1);
    w0[i] = h;
    w1[i] = m;
    w2[i] = bf16_bits((float)(r1 - (double)bf16_value(m)));
}

__device__ __forceinline__ const uint16_t *one_of(int k, const uint16_t *a, const uint16_t *b, const uint16_t *c) {
    return k == 0 ? a : k == 1 ? b : c;
}

// Split-BF16 class GEMM (the decomposition of the FP32 form above): W = N^-1
// split into NP BF16 parts, M = B_IJ[p][a] B_IK[p][b] formed as an FP32
// product and split into NP parts in registers; NP = 3 keeps the products hh,
// hm, mh, hl, lh, mm (smallest first), NP = 2 keeps hh, hm, mh.  MFMA
// 16x16x32 BF16: lane (lr, lk) holds W[16 i + lr][p0 + 8 lk + 0..7] and
// M[p0 + 8 lk + 0..7][16 j + lr]; the result holds members 16 i + 4 lk + v.
// Eight waves per member tile, two on each SIMD: a wave's own VALU work
// (forming and splitting M, the FP64 accumulation) does not overlap its
// MFMAs, but it does overlap those of the other wave on its SIMD.  Wave w
// takes the output rows a = w mod 4 and the column half w / 4, so each wave
// holds half the columns of its rows.  The operands all waves share (W of the tile's
// rows, the B_IK values of a step) are staged through LDS.  A step is 32
// pixels (half a term); a term's FP32 sums are added to the FP64 accumulators
// after its second step.
// With WD the launch also writes D-hat: the D-hat block of every stored block
// of the tile is its unique block, copied in 16-byte chunks, two per thread
// and step (loaded with one step's loads, stored after the next step's), so
// that these writes proceed under the contraction's arithmetic; chunks left
// after the last step are copied at the end of the tile.
template <int NP, int NI, bool WD, bool SKIP, bool BATCH>
__device__ __forceinline__ void class_bf16_tile(const ProblemDescB &pd, int item, int part, int parts, int32_t *sTile,
                                                int32_t *sBlk, int32_t *sTerm, u16x8 *sW, floatx4 *sU, SkipLds &sk) {
    const float *__restrict__ ut32 = pd.ut32;
    double *__restrict__ out = pd.out;
    const int cls = pd.mtiles[4 * item], m0 = pd.mtiles[4 * item + 1];
    const DevClass cl = pd.classes[cls];
    const int tid = thread_index<BATCH>();
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    constexpr int NW = 8, NT = 64 * NW;              // waves, threads
    constexpr int RP = NW / 2;                       // row phases
    const int rw = wave % RP, ch = wave / RP;          // row phase, column half
    const int lane = tid & 63, lr = lane & 15, lk = lane >> 4;
    const int nterms = cl.nterms;
    const int32_t *terms = pd.cterms + 2 * cl.term0;
    if (nterms == 0) {
        if (part == 0) empty_class_tile<NT, WD>(pd, cl, m0, 16 * NI);
        return;
    }

    for (int x = tid; x < 16 * NI * nterms; x += NT) {
        const int r = x / nterms, e = x - r * nterms;
        const int m = min(m0 + r, cl.nblocks - 1);   // rows past the class repeat its last member
        sTile[r * kTileStride + e] = pd.citab[cl.itab0 + (int64_t)m * nterms + e];
    }
    if (tid < 64) {
        const int blk = lane < 16 * NI && m0 + lane < cl.nblocks ? pd.cblk[cl.blk0 + m0 + lane] : -1;
        sBlk[lane] = blk;
        if constexpr (WD) sBlk[64 + lane] = blk >= 0 ? pd.blk_uid[blk] : 0;   // D-hat source block
    }
    if (tid < 2 * nterms) sTerm[tid] = terms[tid];   // unique-block pairs of the class
    __syncthreads();
    // SKIP false: every term of every row, in order
    const int quad0 = 16 * part / parts;
    int total = (16 * (part + 1) / parts - quad0) * nterms;
    if constexpr (SKIP) total = build_skip<NI>(pd, nterms, part, parts, sTerm, sk, [&](int r, int e, int c) {
        // the leading parts: exponents of two BF16 values per word, all ones if not finite
        const uint64_t v = *(const uint64_t *)(pd.w[0] + (int64_t)sTile[r * kTileStride + e] * 64 + 4 * c);
        uint64_t inf = 0;
        for (int i = 0; i < 4; ++i) inf |= (v >> (16 * i) & 0x7f80u) == 0x7f80u;
        return inf == 0;
    });

    // Staging: W is 256 NP chunks of 16 bytes (part c >> 8, row (c & 255) >> 2,
    // chunk c & 3), B_IK of one step 512 chunks (row c >> 3, chunk c & 7).
    // Thread t takes W chunks t + NT r and B_IK chunks t + NT q; with 512
    // threads and NP = 3 the threads past the last W chunk repeat one (same
    // value to the same LDS place), so every thread issues the same loads.
    // Rows past the tile's 16 NI members load the last member's values into
    // LDS rows no wave reads.
    constexpr int NWC = (256 * NP + NT - 1) / NT, NUC = 512 / NT;
    const uint16_t *wsrc[NWC];
    int wrow[NWC], wdst[NWC];
    auto wsw = [](int r) { return ((r >> 1) ^ (r >> 3)) & 3; };
    auto usw = [](int b) { return ((b >> 1) ^ (b << 2)) & 7; };
#pragma unroll
    for (int r = 0; r < NWC; ++r) {
        int c = tid + NT * r;
        if (c >= 256 * NP) c -= 256;
        const int k = __builtin_amdgcn_readfirstlane(c >> 8), q = c & 255, row = q >> 2, sub = q & 3;
        // (an index into a copied descriptor's array would keep it in scratch memory)
        if constexpr (BATCH) wsrc[r] = one_of(k, pd.w[0], pd.w[1], pd.w[2]) + 8 * sub;
        else wsrc[r] = pd.w[k] + 8 * sub;
        wrow[r] = min(row, 16 * NI - 1) * kTileStride;
        // LDS layouts, in 16-byte chunks: W row r (64 bytes) keeps its chunk c at
        // 4 r + (c ^ wsw(r)), a B_IK row b (128 bytes) its chunk c at 8 b + (c ^
        // usw(b)); every read and write phase then touches distinct banks,
        // whether a 16-byte access is served 8 lanes at a time over 32 banks or
        // 16 lanes at a time over 64 banks.
        wdst[r] = (k * 64 + row) * 4 + (sub ^ wsw(row));
    }
    int usrc[NUC], udst[NUC];
#pragma unroll
    for (int q = 0; q < NUC; ++q) {
        const int c = tid + NT * q, ub = c >> 3, uc = c & 7;
        usrc[q] = ub * 64 + 4 * uc;
        udst[q] = ub * 8 + (uc ^ usw(ub));
    }

    // Addresses of one step (term e, half h) for the staged operands (W
    // offsets of this thread's chunks, B_IK rows), and of this lane's B_IJ
    // values of row a.
    struct SAddr { int64_t wo[NWC]; const float *u2; };
    struct OAddr { const float *p1; };
    auto saddr = [&](int e, int h) {
        SAddr r;
#pragma unroll
        for (int q = 0; q < NWC; ++q) r.wo[q] = (int64_t)sTile[wrow[q] + e] * 64 + 32 * h;
        r.u2 = ut32 + (int64_t)__builtin_amdgcn_readfirstlane(sTerm[2 * e + 1]) * kBlockElems + 32 * h;
        return r;
    };
    auto oaddr = [&](int a, int e, int h) {
        OAddr r;
        r.p1 = ut32 + (int64_t)__builtin_amdgcn_readfirstlane(sTerm[2 * e]) * kBlockElems + a * 64 + 32 * h + 8 * lk;
        return r;
    };
    struct Stage { u16x8 w[NWC]; floatx4 u[NUC]; };
    struct Own { floatx4 u1[2]; };        // B_IJ values of this wave's output row (not shared)
    auto stage_load = [&](const SAddr &ad, Stage &st) {
#pragma unroll
        for (int q = 0; q < NWC; ++q) st.w[q] = *(const u16x8 *)(wsrc[q] + ad.wo[q]);
#pragma unroll
        for (int q = 0; q < NUC; ++q) st.u[q] = *(const floatx4 *)(ad.u2 + usrc[q]);
    };
    auto own_load = [&](const OAddr &ad, Own &o) {
        o.u1[0] = *(const floatx4 *)ad.p1;
        o.u1[1] = *(const floatx4 *)(ad.p1 + 4);
    };
    auto stage_store = [&](const Stage &st, int buf) {
#pragma unroll
        for (int q = 0; q < NWC; ++q) sW[buf * NP * 256 + wdst[q]] = st.w[q];
#pragma unroll
        for (int q = 0; q < NUC; ++q) sU[buf * 512 + udst[q]] = st.u[q];
    };
    // this part's D-hat chunks of the tile, two per thread and step: steps dstep .. dchunks / (2 NT)
    constexpr int kDSteps = 16 * NI * 2048 / (2 * NT);
    const int dstep = kDSteps * part / parts, dchunks = kDSteps * (part + 1) / parts * 2 * NT;

    doublex4 acc[NI][2];
    floatx4 psum[NI][2];
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = doublex4{0.0, 0.0, 0.0, 0.0};
    constexpr int NPROD = NP == 3 ? 6 : 3;
    // One step, in three scheduling regions: (1) the loads of the staged
    // operands of the step two ahead and of this wave's B_IJ values of the
    // next step; (2) the MFMAs of this step from LDS buffer buf (W fragments,
    // and M formed from the staged B_IK values and this wave's B_IJ values),
    // with the addresses the next step needs read meanwhile; (3) the staged
    // operands written to buffer sbuf, and, at the end of a term, a barrier.
    auto step = [&](const Own &oc, int buf, const SAddr &sa, const OAddr &oa, int sbuf, Stage &stn, Own &on,
                    int h, uint32_t on0, uint32_t on1, bool bar, int nse, int nsh, int noa, int noe, int noh, SAddr &sa_n, OAddr &oa_n,
                    int stp, DCopy<2> &dprev) {
        stage_load(sa, stn);
        own_load(oa, on);
        if constexpr (WD) {
            DCopy<2> dc;
            dcopy_load<NT>(pd.du64, pd.outD, sBlk, dchunks, stp, wave, lane, dc);
            dcopy_store(dprev, lane);
            dprev = dc;
        }
        __builtin_amdgcn_sched_barrier(0);
        const bool any = !SKIP || ((on0 | on1) >> (8 * h) & 255u) != 0;   // some of this wave's products can be nonzero
        if (any) {
        bf16x8 wf[NI][NP];
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int k = 0; k < NP; ++k)
                wf[i][k] = __builtin_bit_cast(bf16x8, sW[((buf * NP + k) * 64 + 16 * i + lr) * 4 + (lk ^ wsw(16 * i + lr))]);
#pragma unroll
        for (int jj = 0; jj < 2; ++jj) {
            const int b = 32 * ch + 16 * jj + lr;
            const floatx4 u2a = sU[buf * 512 + b * 8 + ((2 * lk) ^ usw(b))];
            const floatx4 u2b = sU[buf * 512 + b * 8 + ((2 * lk + 1) ^ usw(b))];
            typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
            u32x4 words[NP];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int hh = q >> 1, y = 2 * (q & 1);
                const floatx4 &u2 = hh ? u2b : u2a;
                uint32_t parts[NP];
                split_pair<NP>(oc.u1[hh][y] * u2[y], oc.u1[hh][y + 1] * u2[y + 1], parts);
#pragma unroll
                for (int k = 0; k < NP; ++k) words[k][q] = parts[k];
            }
            bf16x8 bfr[NP];
#pragma unroll
            for (int k = 0; k < NP; ++k) bfr[k] = __builtin_bit_cast(bf16x8, words[k]);
            constexpr int pa3[6] = {1, 2, 0, 1, 0, 0}, pb3[6] = {1, 0, 2, 0, 1, 0};
            constexpr int pa2[3] = {1, 0, 0}, pb2[3] = {0, 1, 0};
#pragma unroll
            for (int pr = 0; pr < NPROD; ++pr) {
                const int qa = NP == 3 ? pa3[pr] : pa2[pr];
                const int qb = NP == 3 ? pb3[pr] : pb2[pr];
#pragma unroll
                for (int i = 0; i < NI; ++i)
                    psum[i][jj] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                        wf[i][qa], bfr[qb], (h == 0 && pr == 0) ? floatx4{0.f, 0.f, 0.f, 0.f} : psum[i][jj], 0, 0, 0);
            }
        }
        if constexpr (!SKIP) {
            sa_n = saddr(nse, nsh);
            oa_n = oaddr(noa, noe, noh);
        }
        __builtin_amdgcn_sched_group_barrier(0x100, NI * NP + 6 + NWC, 0);   // LDS reads
#pragma unroll
        for (int x = 0; x < 2 * NPROD * NI; ++x) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);             // one MFMA
            __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);             // two VALU
        }
        __builtin_amdgcn_sched_barrier(0);
        } else if (h == 0) {                 // the term's sum starts from the second half
#pragma unroll
            for (int i = 0; i < NI; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j) psum[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
        }
        if constexpr (SKIP) {                // among the MFMAs they cost up to 3% where halves are left out
            sa_n = saddr(nse, nsh);
            oa_n = oaddr(noa, noe, noh);
        }
        stage_store(stn, sbuf);
        if (bar) __syncthreads();
        __builtin_amdgcn_sched_barrier(0);
    };

    // Four LDS buffers: iteration it (one term of one row) computes from
    // buffers 2 (it & 1) + h, fills the other pair for iteration it + 1, and
    // ends with the only barrier of the term.  Cursors: row index x
    // (a = rw + RP x) and term e; past the last row they repeat (harmless
    // reloads into buffers no step reads).
    auto entry = [&](int it, int before) {   // before: entry it - 1
        if constexpr (SKIP) return __builtin_amdgcn_readfirstlane((int)sk.list[min(it, total - 1)]);
        else if (it == 0) return 256 * quad0;
        else if (it >= total) return before;
        else return (before & 255) + 1 < nterms ? before + 1 : (before | 255) + 1;
    };
    Stage s0, s1;
    Own o0, o1;
    int c0 = entry(0, 0), c1 = entry(1, c0);   // this iteration and the next
    {
        Stage t0, t1;
        stage_load(saddr(c0 & 255, 0), t0);
        stage_load(saddr(c0 & 255, 1), t1);
        own_load(oaddr(rw + RP * (c0 >> 8), c0 & 255, 0), o0);
        stage_store(t0, 0);
        stage_store(t1, 1);
    }
    SAddr sa = saddr(c1 & 255, 0);
    OAddr oa = oaddr(rw + RP * (c0 >> 8), c0 & 255, 1);
    DCopy<2> dpend;                           // D-hat chunks loaded, not yet stored
    dpend.clear();
    __syncthreads();
    // Symmetric classes (the blocks (J, J)) are computed in full here: sharing
    // out the column groups on and above the diagonal, as the FP32 form does,
    // cost more (branches inside the step's scheduling regions, code size)
    // than the skipped groups saved (measured).
    {
        for (int it = 0; it < total; ++it) {
            const int c2 = entry(it + 2, c1);
            const int x = c0 >> 8, e = c0 & 255, x1 = c1 >> 8, e1 = c1 & 255, e2 = c2 & 255;
            const int a = rw + RP * x, a1 = rw + RP * x1;
            uint32_t on0 = 0xffffu, on1 = 0xffffu;
            if constexpr (SKIP) {
                const uint32_t rowm = sk.mask[64 * e + a];
                on0 = __builtin_amdgcn_readfirstlane(rowm & sk.cols[4 * e + 2 * ch]);
                on1 = __builtin_amdgcn_readfirstlane(rowm & sk.cols[4 * e + 2 * ch + 1]);
            }
            const int ib = 2 * (it & 1), nb = 2 - ib;
            step(o0, ib, sa, oa, nb, s1, o1, 0, on0, on1, false, e1, 1, a1, e1, 0, sa, oa, dstep + 2 * it, dpend);
            step(o1, ib + 1, sa, oa, nb + 1, s0, o0, 1, on0, on1, true, e2, 0, a1, e1, 1, sa, oa, dstep + 2 * it + 1, dpend);
            if (!SKIP || (on0 | on1) != 0) {
#pragma unroll
                for (int i = 0; i < NI; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j)
#pragma unroll
                        for (int v = 0; v < 4; ++v) acc[i][j][v] += (double)psum[i][j][v];
            }
            if (x1 != x || it + 1 == total) {    // end of output row a: store, clear
#pragma unroll
                for (int i = 0; i < NI; ++i)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int blk = sBlk[16 * i + 4 * lk + v];
                        if (blk >= 0) {
                            double *ob = out + (int64_t)blk * kBlockElems;
#pragma unroll
                            for (int j = 0; j < 2; ++j) {
                                __builtin_nontemporal_store(acc[i][j][v], &ob[a * 64 + 32 * ch + 16 * j + lr]);
                            }
                        }
                    }
#pragma unroll
                for (int i = 0; i < NI; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j) acc[i][j] = doublex4{0.0, 0.0, 0.0, 0.0};
            }
            c0 = c1;
            c1 = c2;
        }
    }
    if constexpr (WD) {                  // the last step's chunks, then those past the last step
        dcopy_store(dpend, lane);
        for (int stp = dstep + 2 * total; 2 * NT * stp < dchunks; ++stp) {
            DCopy<2> dc;
            dcopy_load<NT>(pd.du64, pd.outD, sBlk, dchunks, stp, wave, lane, dc);
            dcopy_store(dc, lane);
        }
    }
}

// One member tile (item) of one problem; sTile, sBlk, sTerm, sW and sU are the
// workgroup's LDS tables and staging buffers.  FORM kFull or kSkip: the form of
// every problem of the launch; kEither: each problem's own.
enum Form { kFull, kSkip, kEither };

template <int NP, bool WD, int FORM = kEither, bool BATCH = false>
__device__ __forceinline__ void class_bf16_item(const ProblemDescB &pd, int item, int part, int parts, int32_t *sTile, int32_t *sBlk,
                                                int32_t *sTerm, u16x8 *sW, floatx4 *sU, SkipLds &sk) {
    const int groups = pd.mtiles[4 * item + 2];
    if (groups == 0) return;            // an empty slot of a dispatch table
    auto tile = [&](auto skip) {
        constexpr bool SKIP = decltype(skip)::value;
        if (groups == 4) class_bf16_tile<NP, 4, WD, SKIP, BATCH>(pd, item, part, parts, sTile, sBlk, sTerm, sW, sU, sk);
        else if (groups == 2) class_bf16_tile<NP, 2, WD, SKIP, BATCH>(pd, item, part, parts, sTile, sBlk, sTerm, sW, sU, sk);
        else class_bf16_tile<NP, 1, WD, SKIP, BATCH>(pd, item, part, parts, sTile, sBlk, sTerm, sW, sU, sk);
    };
    if constexpr (FORM != kEither) tile(std::bool_constant<FORM == kSkip>());
    else if (pd.skip != 0) tile(std::true_type());
    else tile(std::false_type());
}

template <int NP, bool WD>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
void k_class_bf16(ProblemDescB pd) {
    __shared__ int32_t sTile[64 * kTileStride];
    __shared__ int32_t sBlk[128];                    // stored block per member row; D-hat source block
    __shared__ int32_t sTerm[2 * kMaxClassTerms];     // unique-block pairs of the class
    __shared__ u16x8 sW[4 * NP * 64 * 4];            // staged W, four buffers
    __shared__ floatx4 sU[4 * 512];                  // staged B_IK values, four buffers
    __shared__ SkipLds sk;
    class_bf16_item<NP, WD>(pd, blockIdx.x, blockIdx.y, gridDim.y, sTile, sBlk, sTerm, sW, sU, sk);
}

// Many problems in one persistent launch, split BF16 (the queues and their
// draining as in k_batch_f32; one 8-wave workgroup per CU).  A kernel per form,
// with bodies of its own (thread_index), and one for batches of both, which runs
// the bodies of the single launches: with the thread's index opaque in those too
// BF16x6 alone took 446 us at lmax 300 (437 before), and a batch of both forms
// gains nothing by it.  That kernel spills 100 bytes per lane in BF16x6.  Four
// levels from lmax 512 down, one spilling kernel for all / this: BF16x6 at beams
// of 2.5 pixels 1542 / 1519 us, at 3 (both forms) 1684 / 1616, at 5 1692 / 1657;
// BF16x3 1133 / 1099, 1155 / 1124 and 1159 / 1124.
template <int NP, int FORM>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
void k_batch_bf16(const ProblemDescB *__restrict__ probs, const int32_t *__restrict__ items,
                  const int32_t *__restrict__ qb, int32_t nq, int32_t *__restrict__ counters, int32_t parts) {
    __shared__ int32_t sTile[64 * kTileStride];
    __shared__ int32_t sBlk[128];
    __shared__ int32_t sTerm[2 * kMaxClassTerms];
    __shared__ u16x8 sW[4 * NP * 64 * 4];
    __shared__ floatx4 sU[4 * 512];
    __shared__ SkipLds sk;
    __shared__ int32_t sItem;
    const int home = blockIdx.x % nq;
    int tried = 0;                       // queues found empty (thread 0)
    for (;;) {
        if (threadIdx.x == 0) sItem = batch_next_item(qb, nq, counters, home, tried, parts);
        __syncthreads();
        const int it = __builtin_amdgcn_readfirstlane(sItem);   // uniform: descriptors in scalar registers
        __syncthreads();                 // every thread has read sItem before it changes
        if (it < 0) break;
        const int at = it / parts;
        using Desc = std::conditional_t<FORM != kEither, const ProblemDescB, const ProblemDescB &>;
        Desc pd = probs[items[2 * at]];
        class_bf16_item<NP, false, FORM, FORM != kEither>(pd, items[2 * at + 1], it % parts, parts, sTile, sBlk, sTerm, sW, sU, sk);
    }
}

// Scratch of the allocation-free entry point: N^-1 in the MFMA operand format
// (three BF16 parts or FP32) for up to kNoAllocMaxPix pixels.  Each device
// that loads this code object holds one copy until the process ends.
static __device__ __align__(256) uint16_t scratch[3 * kNoAllocMaxPix];

}  // namespace

hipError_t noalloc_scratch(int device, void **ptr) {
    // the array's name is a host-side stand-in: its device address comes from
    // the runtime, once per device, with that device current
    static std::mutex mu;
    static void *addr[kNoAllocMaxDevices] = {};
    if (device < 0 || device >= kNoAllocMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[device]) {
        int cur = -1;
        hipError_t e = hipGetDevice(&cur);
        if (e != hipSuccess) return e;
        if (cur != device) return hipErrorInvalidDevice;
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        addr[device] = p;
    }
    *ptr = addr[device];
    return hipSuccess;
}

hipError_t launch_tabulate(const double *coef, int32_t lmax, double h, double *table,
                           int32_t n_nodes, int32_t *overflow, hipStream_t st) {
    const int threads = 256;
    const int blocks = (n_nodes + threads - 1) / threads;
    hipLaunchKernelGGL(k_tabulate, dim3(blocks), dim3(threads), 0, st, coef, lmax, h, table, n_nodes, overflow);
    return hipGetLastError();
}

hipError_t launch_eval(KTable kt, const double *y, double *out, int64_t n, hipStream_t st) {
    if (n == 0) return hipSuccess;
    const int64_t blocks = (n + 255) / 256;
    hipLaunchKernelGGL(k_eval, dim3((unsigned)blocks), dim3(256), 0, st, kt, y, out, n);
    return hipGetLastError();
}

hipError_t launch_unique_eval(KTable kt, const UInfo *uinfo, int64_t nunique, const double *ring_theta,
                              const double *ring_sin, double *u64, double *u64t, float *ut32, const UnitMasks &um,
                              hipStream_t st) {
    if (nunique == 0) return hipSuccess;
    hipLaunchKernelGGL(k_unique_eval, dim3((unsigned)nunique), dim3(256), 0, st, kt, uinfo, ring_theta,
                       ring_sin, u64, u64t, ut32, um);
    return hipGetLastError();
}

hipError_t launch_expand(const double *u64, const int32_t *items, int64_t nitems, const int32_t *exp_blk,
                         double *out, hipStream_t st) {
    if (nitems == 0) return hipSuccess;
    hipLaunchKernelGGL(k_expand, dim3((unsigned)nitems), dim3(1024), 0, st, u64, items, exp_blk, out);
    return hipGetLastError();
}

// Dynamic LDS past 64 KiB is allowed per kernel: up to the largest class the
// kernels hold, whatever this launch needs, so that launches do not lower each
// other's limit.
static hipError_t f64_allow_lds(const void *kernel, int bytes) {
    if (bytes <= 64 * 1024) return hipSuccess;
    return hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, f64_lds_bytes(kMaxClassTerms, 64));
}

// A short launch splits each tile's row groups over up to eight workgroups, to
// have two per CU (each repeats the tile's tables).  Measured, D-hat and
// contraction, one / two / four / eight parts: 57 tiles (lmax 64) 518 / 322 /
// 236 / 178 us, 208 (128) 460 / 308 / 265, 350 (256) 879 / 557 / 547, 987 (512)
// 1270 / 1278 / 1321, 8848 (2048) 13373 / 13562 / 13916.  Where a class has many
// terms (two grids) its tiles are long and unlike, a part's share of the tables
// is small, and the launch's end costs more: 1072 tiles of up to 36 terms (lmax
// 256 with 512, beam 5 pixels) one / two / four parts 3301 / 3119 / 3039 us, 320
// of up to 42 (60 with 120) four / eight 1441 / 1194 (the full contraction on
// whole tiles: 1293), 564 of up to 16 (256 with 307) two / four / eight 1246 /
// 1126 / 1164.
static unsigned f64_parts(int64_t tiles, int terms) {
    const int64_t enough = terms > 12 ? 128 * terms : 1024;
    unsigned parts = 1;
    while (parts < 8 && tiles * parts < enough) parts *= 2;
    return parts;
}

// The same for the FP32 and split-BF16 forms, one workgroup per CU: BF16x6 with
// D-hat at lmax 100 (about 100 tiles) 349 -> 117 us.
static unsigned tile_parts(int64_t tiles) {
    unsigned parts = 1;
    while (parts < 8 && tiles * parts < 512) parts *= 2;
    return parts;
}

// The kernel of one FP64 launch: with D-hat or without, with the cut's tests or
// without.
static void (*class_f64_kernel(const ProblemDesc64 &d))(ProblemDesc64) {
    if (d.outD) return d.cut ? k_class_f64<true, false> : k_class_f64<true, true>;
    return d.cut ? k_class_f64<false, false> : k_class_f64<false, true>;
}

// One launch of the FP32 class GEMM: with D-hat or without, with the cut's tests
// or in full.
static void run_class_f32(const ProblemDesc &d, dim3 grid, hipStream_t st) {
    if (d.outD && d.skip) hipLaunchKernelGGL((k_class_f32<true, true>), grid, dim3(512), 0, st, d);
    else if (d.outD) hipLaunchKernelGGL((k_class_f32<true, false>), grid, dim3(512), 0, st, d);
    else if (d.skip) hipLaunchKernelGGL((k_class_f32<false, true>), grid, dim3(512), 0, st, d);
    else hipLaunchKernelGGL((k_class_f32<false, false>), grid, dim3(512), 0, st, d);
}

hipError_t launch_btnb(int prec, const BtnbArgs &a, hipStream_t st) {
    if (a.nblocks == 0) return hipSuccess;
    if (prec == 0) {
        ProblemDesc64 pd{a.mtiles, a.classes, a.class_terms, a.class_blk, a.class_itab, a.u64t, a.ninv, a.out,
                         a.du64, a.blk_uid, a.outD, a.masks.units, a.masks.cols, a.masks.overflow, a.max_terms, a.tile_rows, a.cut};
        const int lds = f64_lds_bytes(a.max_terms, a.tile_rows);
        const auto k = class_f64_kernel(pd);
        const hipError_t e = f64_allow_lds((const void *)k, lds);
        if (e != hipSuccess) return e;
        const dim3 grid((unsigned)a.nmtiles, f64_parts(a.nmtiles, a.max_terms));
        hipLaunchKernelGGL(k, grid, dim3(256), lds, st, pd);
        return hipGetLastError();
    }
    if (prec == 1) {
        hipLaunchKernelGGL(k_ninv_f32, dim3((unsigned)((a.npix + 255) / 256)), dim3(256), 0, st, a.ninv,
                           a.npix, a.wf32);
        ProblemDesc pd{a.mtiles, a.classes, a.class_terms, a.class_blk, a.class_itab, a.ut32, a.wf32, a.out,
                       a.du64, a.blk_uid, a.outD, a.masks.units, a.masks.cols, a.masks.overflow, a.skip};
        run_class_f32(pd, dim3((unsigned)a.nmtiles, tile_parts(a.nmtiles)), st);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_split_ninv, dim3((unsigned)((a.npix + 255) / 256)), dim3(256), 0, st, a.ninv,
                       a.npix, a.wsplit[0], a.wsplit[1], a.wsplit[2]);
    const dim3 grid((unsigned)a.nmtiles, tile_parts(a.nmtiles));
    ProblemDescB pd{a.mtiles, a.classes, a.class_terms, a.class_blk, a.class_itab, a.ut32,
                    {a.wsplit[0], a.wsplit[1], a.wsplit[2]}, a.out, a.du64, a.blk_uid, a.outD,
                    a.masks.units, a.masks.cols, a.masks.overflow, a.skip};
    if (a.outD) {
        if (prec == 2) hipLaunchKernelGGL((k_class_bf16<2, true>), grid, dim3(512), 0, st, pd);
        else hipLaunchKernelGGL((k_class_bf16<3, true>), grid, dim3(512), 0, st, pd);
    } else {
        if (prec == 2) hipLaunchKernelGGL((k_class_bf16<2, false>), grid, dim3(512), 0, st, pd);
        else hipLaunchKernelGGL((k_class_bf16<3, false>), grid, dim3(512), 0, st, pd);
    }
    return hipGetLastError();
}

template <int NP>
static void run_batch_bf16(const BatchLaunch &b, dim3 grid, int32_t parts, hipStream_t st) {
    int skips = 0;
    for (int p = 0; p < b.nprob; ++p) skips += b.host_descb[p].skip != 0;
    auto run = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, dim3(512), 0, st, b.descb, b.items, b.qb, b.nq, b.counters, parts);
    };
    if (skips == 0) run(k_batch_bf16<NP, kFull>);
    else if (skips == b.nprob) run(k_batch_bf16<NP, kSkip>);
    else run(k_batch_bf16<NP, kEither>);
}

hipError_t launch_batch(const BatchLaunch &b, hipStream_t st) {
    hipLaunchKernelGGL(k_fill_i32, dim3(1), dim3(64), 0, st, b.counters, b.nq, 0);
    if (b.prec == 0) {                   // FP64: N^-1 is read as given
        if (b.persistent) {
            if (b.nitems > 0)
                hipLaunchKernelGGL(k_batch_f64, dim3((unsigned)b.nworkgroups), dim3(256), f64_lds_bytes(b.max_terms, 64), st,
                                   b.desc64, b.items, b.qb, b.nq, b.counters, b.max_terms, (int32_t)f64_parts(b.nitems, b.max_terms));
        } else {
            for (int p = 0; p < b.nprob; ++p) {
                if (b.ngtiles[p] == 0) continue;
                ProblemDesc64 d = b.host_desc64[p];
                d.mtiles = b.gtiles[p];
                hipLaunchKernelGGL(class_f64_kernel(d), dim3((unsigned)b.ngtiles[p], f64_parts(b.ngtiles[p], b.max_terms)), dim3(256),
                                   f64_lds_bytes(d.max_terms, d.tile_rows), st, d);
            }
        }
        return hipGetLastError();
    }
    const bool bf16 = b.prec != 1;
    for (int p = 0; p < b.nprob; ++p) {
        if (b.npix[p] == 0) continue;
        const dim3 g((unsigned)((b.npix[p] + 255) / 256));
        if (!bf16) {
            hipLaunchKernelGGL(k_ninv_f32, g, dim3(256), 0, st, b.ninv[p], b.npix[p], b.host_desc[p].wf);
        } else {
            uint16_t *const *w = b.wsplit + 3 * p;
            hipLaunchKernelGGL(k_split_ninv, g, dim3(256), 0, st, b.ninv[p], b.npix[p], w[0], w[1], w[2]);
        }
    }
    if (b.persistent) {
        if (b.nitems > 0) {
            const dim3 g((unsigned)b.nworkgroups);
            const int32_t parts = (int32_t)tile_parts(b.nitems);
            if (!bf16)
                hipLaunchKernelGGL(k_batch_f32, g, dim3(512), 0, st, b.desc, b.items, b.qb, b.nq, b.counters, parts);
            else if (b.prec == 2)
                run_batch_bf16<2>(b, g, parts, st);
            else
                run_batch_bf16<3>(b, g, parts, st);
        }
    } else {
        for (int p = 0; p < b.nprob; ++p) {
            if (b.ngtiles[p] == 0) continue;
            const dim3 g((unsigned)b.ngtiles[p], tile_parts(b.ngtiles[p]));
            if (!bf16) {
                ProblemDesc d = b.host_desc[p];
                d.mtiles = b.gtiles[p];
                run_class_f32(d, g, st);
            } else {
                ProblemDescB d = b.host_descb[p];
                d.mtiles = b.gtiles[p];
                if (b.prec == 2) hipLaunchKernelGGL((k_class_bf16<2, false>), g, dim3(512), 0, st, d);
                else hipLaunchKernelGGL((k_class_bf16<3, false>), g, dim3(512), 0, st, d);
            }
        }
    }
    return hipGetLastError();
}

hipError_t batch_prepare(int prec, int max_terms, int *workgroups_per_cu) {
    if (prec == 0) {
        const int lds = f64_lds_bytes(max_terms, 64);
        hipError_t e = f64_allow_lds((const void *)k_batch_f64, lds);
        if (e == hipSuccess) e = f64_allow_lds((const void *)k_class_f64<false, false>, lds);
        if (e == hipSuccess) e = f64_allow_lds((const void *)k_class_f64<false, true>, lds);
        if (e != hipSuccess) return e;
        return hipOccupancyMaxActiveBlocksPerMultiprocessor(workgroups_per_cu, k_batch_f64, 256, lds);
    }
    if (prec == 1) return hipOccupancyMaxActiveBlocksPerMultiprocessor(workgroups_per_cu, k_batch_f32, 512, 0);
    if (prec == 2) return hipOccupancyMaxActiveBlocksPerMultiprocessor(workgroups_per_cu, k_batch_bf16<2, kEither>, 512, 0);
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(workgroups_per_cu, k_batch_bf16<3, kEither>, 512, 0);
}

hipError_t launch_convolve(const double *u64, const int32_t *chunks, int64_t nchunks, const int32_t *slots,
                           const double *f, double *g, hipStream_t st) {
    if (nchunks == 0) return hipSuccess;
    hipLaunchKernelGGL(k_convolve, dim3((unsigned)nchunks), dim3(256), 0, st, u64, chunks, slots, f, g);
    return hipGetLastError();
}

}  // namespace sympix
