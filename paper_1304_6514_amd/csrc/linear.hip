// Affine basis propagator for the heat equation of sec. 6 (include/nv_linear.h).
//
// Computation phase, two launches:
//   lin_coef_kernel   one thread per (slice, step): the Thomas coefficients
//                     w_i, c_i of that step's tridiagonal matrix (a chain of M
//                     divisions that every solve of the slice shares);
//   lin_build_kernel<MP>
//                     one workgroup per slice, one lane per solve: lane 0 the
//                     forced solve from 0, lane k the homogeneous solve from
//                     e_k; each lane's vector lives in registers (the sweeps
//                     unrolled over MP rows), a step's coefficients in the
//                     lanes of the wave.
// Communication phase: lin_chain_kernel, one workgroup of eight waves, wave r
// forming the partial sums of residue r of the fixed summation order for
// every component from table values prefetched into its registers several
// slices ahead; one LDS exchange and one barrier per slice.  From kBlockedFrom
// slices on it runs through products of the slices' maps, formed by
// lin_many_kernel, which also carries many chains at once.
#include "launch_limits.h"
#include "nv_internal.h"
#include "nv_linear.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstring>
#include <new>
#include <system_error>
#include <thread>
#include <utility>
#include <vector>

using nv::fail;
using nv::lin::kBlock;

#define NV_HIP(expr)                                                                    \
    do {                                                                                \
        hipError_t e_ = (expr);                                                         \
        if (e_ != hipSuccess)                                                           \
            return fail(NV_ERR_HIP, "%s failed: %s", #expr, hipGetErrorString(e_));     \
    } while (0)

namespace {

constexpr int kMaxM = NV_LIN_MAX_POINTS;

struct CoefArgs {
    const double *step;         // [n_slices * S_tot][2]: r, h beta
    double *w, *c;              // [n_slices * S_tot][M]
    long long count;            // n_slices * S_tot
    int M;
};

// A thread's coefficients lie M values apart from the next thread's, so they go
// through LDS kCoefRows rows at a time and leave as runs of consecutive values.
// 20,480 steps of 99 rows: 38 -> 22 us.
constexpr int kCoefRows = 16;

__global__ __launch_bounds__(64) void lin_coef_kernel(CoefArgs a) {
#pragma clang fp contract(off)
    __shared__ double tile[2][64][kCoefRows + 1];
    const int lane = int(threadIdx.x), M = a.M;
    const long long q0 = (long long)blockIdx.x * 64;
    const long long q = q0 + lane < a.count ? q0 + lane : a.count - 1;
    const double r = a.step[2 * q];
    const double diag = 1.0 + 2.0 * r, off = -r;
    double cp = 0.0;
    for (int i0 = 0; i0 < M; i0 += kCoefRows) {
        const int rows = M - i0 < kCoefRows ? M - i0 : kCoefRows;
        for (int i = 0; i < rows; ++i) {
            const double den = i0 + i == 0 ? diag : diag - off * cp;
            const double w = 1.0 / den;
            cp = off * w;
            tile[0][lane][i] = w;
            tile[1][lane][i] = cp;
        }
        __syncthreads();
        const int i = lane % kCoefRows;
        if (i < rows)
            for (int t = lane / kCoefRows; t < 64; t += 64 / kCoefRows)
                if (q0 + t < a.count) {
                    a.w[(q0 + t) * M + i0 + i] = tile[0][t][i];
                    a.c[(q0 + t) * M + i0 + i] = tile[1][t][i];
                }
        __syncthreads();
    }
}

// Device table of slice j: T[j][k Ms + i] = G_j[i][k] (column-major), then
// T[j][M Ms + i] = c_j[i], with the column stride Ms = M rounded up to even
// (the padding row holds 0.0): one contiguous block of Ms (M + 1) values per
// slice, every column 16-byte aligned.
struct BuildArgs {
    const double *step;         // [n_slices * S_tot][2]
    const double *w, *c;        // [n_slices * S_tot][M]
    const double *s;            // [M] sin(pi x_i)
    double *T;                  // [n_slices][Ms (M + 1)]
    int M, S_tot, forcing;
};

__host__ __device__ inline int lin_stride(int M) { return M + (M & 1); }

__device__ inline double lin_readlane(double v, int l) {
    const long long b = __double_as_longlong(v);
    const unsigned lo = unsigned(__builtin_amdgcn_readlane(int(b & 0xffffffffLL), l));
    const unsigned hi = unsigned(__builtin_amdgcn_readlane(int(b >> 32), l));
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// Value i of 128 that the wave's lanes hold two each (i in lane i, 64 + i in
// lane i again), in scalar registers.
__device__ inline double lin_pick(const double (&v)[2], int i) { return lin_readlane(v[i >> 6], i & 63); }

// One backward Euler step of the lane's solve: the Thomas sweeps over MP >= M
// rows, a row's coefficients taken from the lanes that hold them.  Rows M ..
// MP-1 have coefficients 0 and stay 0, so that row M-1 of the back substitution
// subtracts c * 0 and is x itself.  Forced: the lane's right-hand side is f + m
// fs, m being 1 in the lane of the forced solve and 0 in the others: the
// product is exact, so the fused operation rounds once, as f + fs does, and
// leaves f alone elsewhere.
template <int MP, bool Forced>
__device__ inline void lin_step(double (&x)[MP], double off, const double (&w)[2],
                                const double (&c)[2], const double (&fs)[2], double m) {
#pragma clang fp contract(off)
    double fp = 0.0;
#pragma unroll
    for (int i = 0; i < MP; ++i) {
        double f = x[i];
        if constexpr (Forced) f = fma(m, lin_pick(fs, i), f);
        fp = i == 0 ? f * lin_pick(w, 0) : (f - off * fp) * lin_pick(w, i);
        x[i] = fp;
    }
    double y = x[MP - 1];
#pragma unroll
    for (int i = MP - 2; i >= 0; --i) {
        y = x[i] - lin_pick(c, i) * y;
        x[i] = y;
    }
}

// What bounds it: the issue of each wave's FP64 operations, five per row and
// step, and of the four lane reads that bring the row's two coefficients into
// scalar registers (with the coefficients staged in LDS, two to four waves per
// SIMD waited for a read every other row: 226 us at M = 99, 1024 slices of 20
// steps, where this takes 115 us; M = 127, 512 slices: 1059 -> 124 us).  Up to
// MP = 104 two waves share a SIMD; above, a wave has the SIMD's registers to itself.
template <int MP>
__global__ __launch_bounds__(128, MP <= 104 ? 2 : 1) void lin_build_kernel(BuildArgs a) {
#pragma clang fp contract(off)
    const int solve = int(threadIdx.x), lane = solve & 63, M = a.M;
    const int j = int(blockIdx.x);
    const bool forced = a.forcing && solve < 64;     // the wave of the forced solve
    const double m = solve == 0 ? 1.0 : 0.0;
    const long long q0 = (long long)j * a.S_tot;
    double x[MP];
#pragma unroll
    for (int i = 0; i < MP; ++i) x[i] = i == solve - 1 ? 1.0 : 0.0;
    // rows lane and 64 + lane of a step's coefficients (0 past row M - 1)
    const int r0 = lane < M ? lane : M - 1, r1 = 64 + lane < M ? 64 + lane : M - 1;
    const bool in0 = lane < M, in1 = 64 + lane < M;
    // a forcing that is not finite: m times it would reach every lane, so it takes no
    // part in the sweeps; the forced solve, and it alone, is not finite from there on
    double lost = 0.0;
    const double s[2] = {in0 ? a.s[r0] : 0.0, in1 ? a.s[r1] : 0.0};
    double w[2], c[2];
    w[0] = a.w[q0 * M + r0];
    w[1] = a.w[q0 * M + r1];
    c[0] = a.c[q0 * M + r0];
    c[1] = a.c[q0 * M + r1];
    for (int st = 0; st < a.S_tot; ++st) {
        const long long q = q0 + st;
        const double off = -a.step[2 * q], hb_step = a.step[2 * q + 1];
        const double hb = isfinite(hb_step) ? hb_step : 0.0;
        if (!isfinite(hb_step)) lost = hb_step;
        // the next step's coefficients (the last step reloads its own)
        const long long qn = st + 1 < a.S_tot ? q + 1 : q;
        const double wn[2] = {a.w[qn * M + r0], a.w[qn * M + r1]};
        const double cn[2] = {a.c[qn * M + r0], a.c[qn * M + r1]};
        const double ww[2] = {in0 ? w[0] : 0.0, in1 ? w[1] : 0.0};
        const double cc[2] = {in0 ? c[0] : 0.0, in1 ? c[1] : 0.0};
        const double fs[2] = {hb * s[0], hb * s[1]};
        if (forced)
            lin_step<MP, true>(x, off, ww, cc, fs, m);
        else
            lin_step<MP, false>(x, off, ww, cc, fs, m);
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            w[u] = wn[u];
            c[u] = cn[u];
        }
    }
    if (solve > M) return;
    const int Ms = lin_stride(M);
    double *blk = a.T + (long long)j * Ms * (M + 1);
    double2 *col = reinterpret_cast<double2 *>(solve == 0 ? blk + Ms * M : blk + (solve - 1) * Ms);
#pragma unroll
    for (int i = 0; i < MP; i += 2)             // row M of an odd M is padding: 0
        if (i < M) col[i / 2] = double2{x[i], x[i + 1]};
    if (solve == 0 && lost != 0.0)
        for (int i = 0; i < M; ++i) blk[Ms * M + i] = lost;
}

template <int MP>
void lin_launch_build(const BuildArgs &a, int n_slices, hipStream_t st) {
    hipLaunchKernelGGL(lin_build_kernel<MP>, dim3(unsigned(n_slices)),
                       dim3(unsigned(64 * ((a.M + 1 + 63) / 64))), 0, st, a);
}

using BuildLaunch = void (*)(const BuildArgs &, int, hipStream_t);
template <int... K>
constexpr void build_fill(BuildLaunch *t, std::integer_sequence<int, K...>) {
    ((t[K] = &lin_launch_build<8 * (K + 1)>), ...);
}

// lin_build.f[k - 1] launches the build for ceil(M/8) = k
struct LinBuildTable {
    BuildLaunch f[16];
    LinBuildTable() { build_fill(f, std::make_integer_sequence<int, 16>{}); }
};
const LinBuildTable lin_build;

// ---- blocks of slices ------------------------------------------------------
//
// The chain of N affine maps takes N dependent steps, whatever the chip could
// do at once.  Composition is associative, so the maps are first multiplied
// together in blocks of kBlock (every block on its own, as matrix products),
// the blocks' maps again in blocks while there are more than kTopMaps of them,
// and the states run through the few maps of the top level; the states inside
// a block, where they are asked for, then follow from the state at its start,
// every block on its own again.  A level's maps lie in memory as the slices'
// do, so the same kernels run on all of them.  At M = 99, N = 1024 a chain's
// dependent steps fall from 1024 to 7 + 7 + 16 (+ 7 + 7 for the inner states).
//
// Rounding.  a(t) is positive, so every G_j is the inverse of an M-matrix:
// non-negative, with row sums of at most 1.  Products of such matrices have no
// cancellation: a block's map carries a relative error of at most kBlock
// gamma_M in every entry, and a state formed with it stays within the rounding
// bound of any other order of the same sums.
//
// A state or a map that exceeds kLargest (or is not finite) is reported by the
// kernels, and the chains are then run slice by slice, which names the slice.
constexpr int kTopMaps = 16;            // fewer maps are not worth another level's launches
constexpr int kBlockedFrom = 64;        // slices; below, the launches cost what the steps save
constexpr double kLargest = 1e300;
constexpr int kNoSlice = 0x7fffffff;

// Which maps a launch runs through: block b of the level starts at map
// b kBlock (one block of all `maps` maps when whole); map m of the level
// starts at slice m stride.
struct LevelArgs {
    const double *T;            // the level's maps, [maps][Ms (M + 1)]
    int M, N;                   // interior points; slices of the whole chain
    int maps, stride;
    int whole;
    double largest;             // a state beyond it is reported
};

struct LevelRange {
    int first, count;           // the block's maps
    __device__ LevelRange(const LevelArgs &a, int b) {
        first = a.whole ? 0 : b * kBlock;
        count = a.whole ? a.maps : (a.maps - first < kBlock ? a.maps - first : kBlock);
    }
};

// The slice a state lies at after t maps of the block.
__device__ inline long long level_slice(const LevelArgs &a, int first, int t) {
    const long long s = (long long)(first + t) * a.stride;
    return s < a.N ? s : a.N;
}

struct ComposeArgs {
    LevelArgs lv;
    const double *y0;           // device [M]: the state at slice 0 (whole level)
    double *boundary;           // device [(N+1)][M]
    int *bad;                   // a whole level sets it: the first map whose state is beyond the
                                // limit, or -1; blocks set it to 0 when one of theirs is
};

// third word of a buffer resource on gfx9-family chips (32-bit data format,
// no swizzle): raw buffer loads then read num_records bytes from the base
constexpr int kBufferWord3 = 0x00020000;

// The chain, built around the summation order itself.  Wave r (r = 0..7)
// forms the partial sums p_r = G_i,r l_r + G_i,r+8 l_r+8 + ... (left to right
// from 0) of every component i, lane l taking the two rows 2l and 2l + 1 (so
// one wave covers M <= 128), from table values that were loaded straight into
// its registers D slices ahead: per slice, KM = ceil(M/8) 16-byte loads of a
// row pair (column fragments of 128 consecutive doubles per wave: coalesced,
// and no table value passes through LDS).  The partial sums go to LDS; after
// the one barrier of the slice, lane m < KM of wave r combines the eight
// partial sums of component r + 8m in the fixed tree and adds c, which yields
// exactly the new state components that wave r needs for the next slice, and
// v_readlane hands them to the whole wave.  The partial-sum buffer is double
// buffered, so one barrier per slice suffices.  Each wave stores its own
// components of the boundary states; a store is always younger than the loads
// the next slices wait for, so it never delays them (the memory counter is in
// order).
template <int KM, int D>
__global__ __launch_bounds__(512) void lin_chain_kernel(ComposeArgs a) {
#pragma clang fp contract(off)
    constexpr int kRow = 128;
    __shared__ double part[2][8][kRow];
    __shared__ int bad_s;
    const int tid = int(threadIdx.x), lane = tid & 63;
    const int r = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int M = a.lv.M, Ms = lin_stride(M), per = Ms * (M + 1);
    const LevelRange rg(a.lv, int(blockIdx.x));
    // a block ends one map early: the state after it is the next block's first
    const int N = a.lv.whole ? rg.count : rg.count - 1;
    if (N < 1) return;
    const double *T = a.lv.T + (long long)rg.first * per;
    const double *start = a.lv.whole
                              ? a.y0
                              : a.boundary + level_slice(a.lv, rg.first, 0) * M;
    const int mr = r < M ? (M - r + 7) / 8 : 0;        // components k = r + 8m < M
    const int i2 = 2 * lane;                           // the lane's first row
    // byte offsets within a slice block: column k starts at the wave-uniform
    // k Ms, the lane adds its (16-byte aligned) row pair; c of component
    // r + 8 lane for lanes < mr
    const unsigned row_b = unsigned(i2 < M ? i2 : Ms - 2) * 8u;
    const unsigned c_b = unsigned(Ms * M + (lane < mr ? r + 8 * lane : M - 1)) * 8u;
    // Terms past mr (components r + 8m >= M; only when KM > mr) take the state
    // value +0.0 (here, and from the broadcast of lanes >= mr, whose v stays
    // 0.0) and the table value of column M - 1; their product is then +-0.0 for
    // a finite table, and since p starts at +0.0 it is never -0.0, so adding
    // +-0.0 leaves p unchanged to the bit: no per-term condition is needed.  (A
    // non-finite value in column M - 1 makes that row non-finite in the exact
    // sum as well, in the same slice.)
    double lam[KM];
#pragma unroll
    for (int m = 0; m < KM; ++m) {
        const int k = r + 8 * m;
        lam[m] = k < M ? start[k] : 0.0;
    }
    if (a.lv.whole && tid < M) a.boundary[tid] = start[tid];
    if (tid == 0) bad_s = kNoSlice;

    double2 g[D][KM];
    double cv[D];
    // Raw buffer loads over the slice's block, every one unconditional, from a
    // clamped slice index: the column offset k Ms is a scalar operand and the
    // lane's row pair a 32-bit vector offset, so no load needs an address
    // register of its own (and the hardware checks the block's bounds).  The
    // slice index passes through readfirstlane so that the compiler keeps one
    // scalar base instead of strength-reducing every load into an address
    // register.
#define NV_LIN_FETCH(slot, s)                                                            \
    do {                                                                                 \
        const int s_ = __builtin_amdgcn_readfirstlane((s) < N ? (s) : N - 1);            \
        const __amdgpu_buffer_rsrc_t rs_ = __builtin_amdgcn_make_buffer_rsrc(            \
            (void *)(T + (long long)s_ * per), 0, per * 8, kBufferWord3);                \
        _Pragma("unroll") for (int m = 0; m < KM; ++m) {                                 \
            const int col_ = (r + 8 * m < M ? r + 8 * m : M - 1) * Ms * 8;               \
            g[slot][m] = __builtin_bit_cast(                                             \
                double2, __builtin_amdgcn_raw_buffer_load_b128(rs_, int(row_b), col_, 0)); \
        }                                                                                \
        cv[slot] = __builtin_bit_cast(double,                                            \
                                      __builtin_amdgcn_raw_buffer_load_b64(rs_, int(c_b), 0, 0)); \
    } while (0)
    // first half of a slice: the partial sums of the lane's two rows, to LDS
#define NV_LIN_PARTIAL(slot, j)                                                          \
    do {                                                                                 \
        double p0 = 0.0, p1 = 0.0;                                                       \
        _Pragma("unroll") for (int m = 0; m < KM; ++m) {                                 \
            p0 = p0 + g[slot][m].x * lam[m];                                             \
            p1 = p1 + g[slot][m].y * lam[m];                                             \
        }                                                                                \
        if (i2 < M) part[(j) & 1][r][i2] = p0;                                           \
        if (i2 + 1 < M) part[(j) & 1][r][i2 + 1] = p1;                                   \
    } while (0)
    // second half: after the barrier, the new components r + 8m and their
    // broadcast; nothing is stored for the slices past N
#define NV_LIN_COMBINE(c_now, j)                                                         \
    do {                                                                                 \
        __syncthreads();                                                                 \
        double v = 0.0;                                                                  \
        if (lane < mr) {                                                                 \
            const int k = r + 8 * lane;                                                  \
            const double *q = &part[(j) & 1][0][k];                                      \
            const double s = ((q[0] + q[kRow]) + (q[2 * kRow] + q[3 * kRow])) +          \
                             ((q[4 * kRow] + q[5 * kRow]) + (q[6 * kRow] + q[7 * kRow])); \
            v = (c_now) + s;                                                             \
            if ((j) < N) {                                                               \
                a.boundary[level_slice(a.lv, rg.first, (j) + 1) * M + k] = v;            \
                if (!(fabs(v) <= a.lv.largest)) atomicMin(&bad_s, (j));                  \
            }                                                                            \
        }                                                                                \
        _Pragma("unroll") for (int m = 0; m < KM; ++m) lam[m] = lin_readlane(v, m);      \
    } while (0)

#pragma unroll
    for (int d = 0; d < D; ++d) NV_LIN_FETCH(d, d);
    // whole groups of D slices: the up to D - 1 slices past N of the last group
    // repeat the clamped table of slice N - 1 and store nothing, which keeps
    // the loop free of a tail (a tail's extra copy of the body doubles the
    // register demand)
    for (int j0 = 0; j0 < N; j0 += D) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            NV_LIN_PARTIAL(d, j0 + d);
            const double c_now = cv[d];
            // slot d is consumed: refill it while the other waves reach the
            // barrier (not hoisted above the products, which would hold old and
            // new values of the slot at once)
            __builtin_amdgcn_sched_barrier(0);
            NV_LIN_FETCH(d, j0 + d + D);
            NV_LIN_COMBINE(c_now, j0 + d);
        }
    }
#undef NV_LIN_FETCH
#undef NV_LIN_PARTIAL
#undef NV_LIN_COMBINE
    __syncthreads();
    if (tid == 0) {
        if (a.lv.whole)
            *a.bad = bad_s == kNoSlice ? -1 : bad_s;
        else if (bad_s != kNoSlice)
            *a.bad = 0;
    }
}

// prefetch depth for KM loads per slice: a ring of about 72 doubles per lane
// (120 for the largest tables, KM >= 10, where a deeper ring measured faster),
// at least 2 and at most 8 slices ahead
constexpr int lin_depth(int KM) {
    const int ring = KM >= 10 ? 120 : 72, d = ring / (2 * KM + 1);
    return d < 2 ? 2 : (d > 8 ? 8 : d);
}

template <int KM>
void lin_launch_chain(const ComposeArgs &a, hipStream_t st) {
    const int blocks = a.lv.whole ? 1 : (a.lv.maps + kBlock - 1) / kBlock;
    hipLaunchKernelGGL((lin_chain_kernel<KM, lin_depth(KM)>), dim3(unsigned(blocks)), dim3(512), 0,
                       st, a);
}

using LinLaunch = void (*)(const ComposeArgs &, hipStream_t);
template <int... K>
constexpr void lin_fill(LinLaunch *t, std::integer_sequence<int, K...>) {
    ((t[K] = &lin_launch_chain<K + 1>), ...);
}

// lin_chain[KM - 1] launches the chain for ceil(M/8) = KM
struct LinChainTable {
    LinLaunch f[16];
    LinChainTable() { lin_fill(f, std::make_integer_sequence<int, 16>{}); }
};
const LinChainTable lin_chain;

// ---- many initial values: the chain as FP64 matrix products -------------
//
// Q chains lambda^q_{j+1} = c_j + G_j lambda^q_j are independent, so workgroup
// b carries the 16 CB chains q = 16 CB b .. 16 CB b + 16 CB - 1 through every
// slice alone (no synchronisation between workgroups): per slice the product
// G_j Lambda_j of the M x M table with the M x 16 CB block of states, on the
// matrix cores (v_mfma_f64_16x16x4f64: wave w forms rows 16 w .. 16 w + 15 of
// the product, k = 0 .. 4 KP - 1 in steps of four, each A fragment of G
// multiplied with the CB 16-column blocks of states), then c_j added.
// Lambda_j lives in LDS, double buffered (rows k >= M are zero), one barrier
// per slice; every wave holds the A fragments of its rows of G_j in registers
// and reloads them with those of G_{j+1} as it uses them.  Every workgroup reads all N tables, so
// the tables' traffic from the caches is (Q / 16 CB) x N x M (M + 1) doubles:
// CB = 2 halves it for large Q.
//
// The same kernel multiplies the maps of a block together (`product`): the
// M + 1 columns of the block's first map (c last) are the chains, run through
// the block's other maps, c_j added to the last column only.
struct ManyArgs {
    LevelArgs lv;
    const double *y0;           // [Q][M]
    double *yT;                 // [Q][M]
    double *boundary;           // [Q][N+1][M] or null
    double *product;            // [blocks][Ms (M + 1)]: the blocks' maps, or null
    int *bad;                   // first map whose state is beyond the limit (atomic min)
    long long Q;
    int groups;                 // workgroups of one block of maps
    int blocks;                 // blocks of maps
    int spread;                 // many_spread
};

typedef double v4d __attribute__((ext_vector_type(4)));

template <int KP, int CB>
__global__ __launch_bounds__(512) void lin_many_kernel(ManyArgs a) {
#pragma clang fp contract(off)
    constexpr int K = 4 * KP;                    // rows of Lambda in LDS (M <= K)
    constexpr int C = 16 * CB;                   // chains of the workgroup
    __shared__ double lam[2][K][C];
    const int tid = int(threadIdx.x), lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int M = a.lv.M, Ms = lin_stride(M), per = Ms * (M + 1);
    const unsigned spread = unsigned(a.spread), turn = blockIdx.x / spread;
    const int block = int(turn / unsigned(a.groups) * spread + blockIdx.x % spread);
    const int group = int(turn % unsigned(a.groups));
    if (block >= a.blocks) return;
    const LevelRange rg(a.lv, block);
    const bool product = a.product != nullptr;
    // the maps run through: all of a whole level; of a product all but the
    // first (whose columns it starts from); of a block all but the last (the
    // state after it is the next block's first)
    const int N = a.lv.whole && !product ? rg.count : rg.count - 1;
    const double *T0 = a.lv.T + (long long)rg.first * per;      // the block's first map
    const double *T = product ? T0 + per : T0;
    const int col = lane & 15, kq = lane >> 4;
    const long long Q = product ? M + 1 : a.Q;
    const long long q0 = (long long)group * C;
    const bool from_boundary = !product && !a.lv.whole;
    const long long span = (long long)(a.lv.N + 1) * M;         // one chain's boundary states
    int bad = kNoSlice;
    if (product && blockIdx.x == 0 && tid == 0) *a.bad = kNoSlice;
    for (int e = tid; e < 2 * K * C; e += 512) {
        const int buf = e / (K * C), k = (e / C) % K, c = e % C;
        const long long qq = q0 + c < Q ? q0 + c : Q - 1;
        double v = 0.0;
        if (buf == 0 && k < M) {
            v = product ? T0[qq * Ms + k]
                        : (from_boundary
                               ? a.boundary[qq * span + level_slice(a.lv, rg.first, 0) * M + k]
                               : a.y0[qq * M + k]);
            if (!product && a.lv.whole && a.boundary && q0 + c < Q)
                a.boundary[qq * span + k] = v;
            if (a.lv.largest < 1e301 && !(fabs(v) <= a.lv.largest)) bad = 0;
        }
        lam[buf][k][c] = v;
    }
    // the lane's A operand: row 16 w + col of G, columns 4 kk + kq (A[i][k] in
    // lane i + 16 k), B[k][j] in lane j + 16 k; the FP64 16 x 16 accumulator
    // interleaves its rows: lane l holds D[4 i + l/16][l % 16] (i = 0..3,
    // measured on the device), so the lane's outputs are rows 16 w + 4 i + kq
    // of chain column col of each column block
    const int arow = 16 * w + col;
    const bool active = 16 * w < M;
    bool live[CB], with_c[CB];
    double *states[CB];                         // the chain's boundary states, or null
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
        const long long q = q0 + 16 * cb + col;
        live[cb] = q < Q;
        with_c[cb] = !product || q == M;
        states[cb] = live[cb] && a.boundary ? a.boundary + q * span : nullptr;
    }
    // The A fragments and the c values of a slice, loaded unconditionally from
    // clamped (in-block) addresses, with no select after the load (which would
    // wait for it): a column k >= M meets the zero row k of Lambda, a row
    // >= M of the product is never stored.  (A non-finite table value in column
    // M - 1 thus also reaches the padded terms; it makes its row non-finite in
    // the exact sum as well.)  Each fragment is loaded for the next slice as soon
    // as its product is issued, into the same registers: the loads go out between
    // the products instead of ahead of them, and two workgroups fit a CU (at most
    // 128 registers instead of 224).  1024 maps of 99 points: products of the
    // first level 91 -> 71 us, 4096 chains 199 -> 169 us.  A slice takes 6,700
    // clocks of which the matrix cores are busy for 3,200 (two waves per SIMD);
    // the rest is the sums' way through LDS and the barrier.
    double g[KP], cv[4];
    const int ar = arow < M ? arow : M - 1;
    // byte offsets, so that a load takes a scalar base and one register
    const unsigned at = 8 * unsigned(kq * Ms + ar);
    const int k_last = 4 * (KP - 1) + kq;
    const unsigned at_last = 8 * unsigned((k_last < M ? k_last : M - 1) * Ms + ar);
    unsigned at_c[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int r = 16 * w + 4 * i + kq;
        at_c[i] = 8 * unsigned(Ms * M + (r < M ? r : M - 1));
    }
    const auto from = [](const double *base, unsigned bytes) {
        return *reinterpret_cast<const double *>(reinterpret_cast<const char *>(base) + bytes);
    };
    const auto load = [&](const double *Tj, int kk) {
        return kk < KP - 1 ? from(Tj + 4 * kk * Ms, at) : from(Tj, at_last);
    };
    if (active && N > 0) {
#pragma unroll
        for (int kk = 0; kk < KP; ++kk) g[kk] = load(T, kk);
#pragma unroll
        for (int i = 0; i < 4; ++i) cv[i] = from(T, at_c[i]);
    }
    int cur = 0;
    __syncthreads();
    for (int j = 0; j < N; ++j) {
        if (active) {
            const double *next = T + (long long)(j + 1 < N ? j + 1 : N - 1) * per;
            // the product on the matrix cores (even and odd k-steps in two
            // accumulators per column block), c added, the new states to LDS (and
            // the boundary), barrier
            v4d acc[CB], acc1[CB];
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) acc[cb] = acc1[cb] = v4d{0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int kk = 0; kk < KP; ++kk) {
#pragma unroll
                for (int cb = 0; cb < CB; ++cb) {
                    const double b = lam[cur][4 * kk + kq][16 * cb + col];
                    v4d &sum = kk % 2 == 0 ? acc[cb] : acc1[cb];
                    sum = __builtin_amdgcn_mfma_f64_16x16x4f64(g[kk], b, sum, 0, 0, 0);
                }
                g[kk] = load(next, kk);
            }
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) {
                const v4d s = acc[cb] + acc1[cb];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int r = 16 * w + 4 * i + kq;
                    const double v = (with_c[cb] ? cv[i] : 0.0) + s[i];
                    if (r < M) {
                        lam[cur ^ 1][r][16 * cb + col] = v;
                        if (states[cb])
                            states[cb][level_slice(a.lv, rg.first, j + 1) * M + r] = v;
                        if (live[cb] && !(fabs(v) <= a.lv.largest) && j < bad) bad = j;
                    }
                }
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) cv[i] = from(next, at_c[i]);
        }
        __syncthreads();
        cur ^= 1;
    }
    if (product) {
        // a column beyond the limit becomes NaN, so that a state formed with it
        // is reported
        __shared__ int beyond;
        if (tid == 0) beyond = 0;
        __syncthreads();
        if (bad != kNoSlice) beyond = 1;
        __syncthreads();
        double *U = a.product + (long long)block * per;
        for (int e = tid; e < Ms * C; e += 512) {
            const int k = e % Ms, c = e / Ms;
            if (q0 + c < Q)
                U[(q0 + c) * Ms + k] =
                    k < M ? (beyond ? __longlong_as_double(0x7ff8000000000000LL) : lam[cur][k][c])
                          : 0.0;
        }
        return;
    }
    if (a.yT && a.lv.whole)
        for (int e = tid; e < M * C; e += 512) {
            const int k = e / C, c = e % C;
            if (q0 + c < Q) a.yT[(q0 + c) * M + k] = lam[cur][k][c];
        }
    if (bad != kNoSlice) atomicMin(a.bad, bad);
}

template <int KP>
void lin_launch_many(ManyArgs a, long long pair_from, hipStream_t st) {
    using namespace nv::lin;
    const long long Q = a.product ? a.lv.M + 1 : a.Q;
    const long long blocks = a.lv.whole ? 1 : (a.lv.maps + kBlock - 1) / kBlock;
    const bool paired = !a.product && many_paired(a.lv.M, Q, blocks, pair_from);
    a.blocks = int(blocks);
    a.groups = int(many_groups(Q, paired));
    a.spread = many_spread(blocks, a.product != nullptr);
    const dim3 grid(unsigned(a.groups * many_rows(blocks, a.product != nullptr)));
    if constexpr (KP <= kManyPairMaxKP) {
        if (paired) {
            hipLaunchKernelGGL((lin_many_kernel<KP, 2>), grid, dim3(kThreads), 0, st, a);
            return;
        }
    }
    hipLaunchKernelGGL((lin_many_kernel<KP, 1>), grid, dim3(kThreads), 0, st, a);
}

using ManyLaunch = void (*)(ManyArgs, long long, hipStream_t);
template <int... K>
constexpr void many_fill(ManyLaunch *t, std::integer_sequence<int, K...>) {
    ((t[K] = &lin_launch_many<K + 1>), ...);
}

// lin_many[KP - 1] launches the product chain for ceil(M/4) = KP
struct LinManyTable {
    ManyLaunch f[32];
    LinManyTable() { many_fill(f, std::make_integer_sequence<int, 32>{}); }
};
const LinManyTable lin_many;

}  // namespace

constexpr int kMaxLevels = 12;          // 8^12 exceeds any number of slices

struct nv_lin {
    hipStream_t stream = nullptr;
    char *mem = nullptr;
    size_t mem_bytes = 0;
    // layout of the last build
    double *step = nullptr, *w = nullptr, *c = nullptr, *s = nullptr, *T = nullptr,
           *y0 = nullptr, *boundary = nullptr;
    double *product[kMaxLevels] = {};   // the maps of level 1, 2, ...
    int levels = 0;                     // of products, each of kBlock maps of the one below
    int *bad = nullptr;
    int M = 0, N = 0, S_tot = 0;
    bool built = false;
    bool fixed_order = false;           // one chain slice by slice, to the bit
    hipEvent_t e0 = nullptr, e1 = nullptr, e2 = nullptr, e3 = nullptr;
    float build_ms = 0.f, compose_ms = 0.f;
    // pinned staging of the step scalars and of a composition's results; none
    // when the last build needed more than kHostMost or it could not be had
    char *host = nullptr;
    size_t host_bytes = 0;
};

namespace {

size_t al(size_t x) { return (x + 255) & ~size_t(255); }

// Through pinned memory a copy is one transfer that the host does not wait for;
// from and to pageable memory the runtime stages it and waits, once per copy.
// M = 99, 1024 slices of 20
// steps: scalars up 22 -> 5 us of the host's time,
// results down (811 KB) 97 -> 45 us.  Larger transfers are left to the runtime,
// which stages them piece by piece without holding as much pinned memory.
constexpr size_t kHostMost = size_t(8) << 20;

// Room for `bytes` in l->host, or none at all.
void ensure_host(nv_lin *l, size_t bytes) {
    if (bytes <= l->host_bytes) return;
    if (l->host) {
        (void)hipStreamSynchronize(l->stream);
        (void)hipHostFree(l->host);
    }
    l->host = nullptr;
    l->host_bytes = 0;
    if (bytes > kHostMost) return;
    if (hipHostMalloc(reinterpret_cast<void **>(&l->host), bytes, hipHostMallocDefault) !=
        hipSuccess) {
        (void)hipGetLastError();
        l->host = nullptr;
        return;
    }
    l->host_bytes = bytes;
}

// FP64 host evaluations with one rounding per operation.
// a(t) = a0 + a1 sin t and beta(t) = ((pi pi) a(t)) cos t - sin t from one
// evaluation of sin t and cos t (the same values as evaluating them anew)
struct StepCoef {
    double a, beta;
};

StepCoef coef_at(const nv_heat &p, double t) {
#pragma clang fp contract(off)
    const double sn = std::sin(t), cs = std::cos(t);
    const double a = p.a0 + p.a1 * sn;
    return {a, ((M_PI * M_PI) * a) * cs - sn};
}

// The per-step scalars r = (h a(t_end)) / (dx dx) and h beta(t_end) of slices
// [j0, j1); returns the first step (global index) whose a(t) is not positive,
// or -1, with its time in *bad_t.
long long step_scalars(const nv_heat &p, double t0, double L, double dt, int S, double rem,
                       int S_tot, double dx, int j0, int j1, double *step, double *bad_t) {
#pragma clang fp contract(off)
    for (int j = j0; j < j1; ++j) {
        const double Tj = t0 + double(j) * L;
        for (int st = 0; st < S_tot; ++st) {
            const bool last = st == S;
            const double h = last ? rem : dt;
            const double te = last ? (Tj + double(S) * dt) + rem : Tj + double(st + 1) * dt;
            const StepCoef k = coef_at(p, te);
            const long long q = (long long)j * S_tot + st;
            if (!(k.a > 0.0)) {
                *bad_t = te;
                return q;
            }
            step[2 * q] = (h * k.a) / (dx * dx);
            step[2 * q + 1] = p.forcing ? h * k.beta : 0.0;
        }
    }
    return -1;
}

// step_scalars of every slice, in pieces that a few host threads take in turn.
// A thread takes about 12 us to create and the pieces of 20,480 steps 250 us to
// work through, so there is one thread per 4096 steps, eight at most (equal
// shares for eight threads took 165 us, this takes 110).
long long all_step_scalars(const nv_heat &p, double t0, double L, double dt, int S, double rem,
                           int S_tot, double dx, int n_slices, double *step, double *bad_t) {
    const long long nq = (long long)n_slices * S_tot;
    const unsigned hc = std::thread::hardware_concurrency();
    const int nth = int(std::min<long long>(std::max<long long>(nq / 4096, 1),
                                            std::min(std::max(int(hc), 1), 8)));
    const int piece = int(std::max<long long>(1, 1024 / S_tot));
    std::atomic<int> next{0};
    struct Found {
        long long q = -1;
        double t = 0.0;
    };
    std::vector<Found> found(std::max(nth, 1));
    const auto work = [&](int k) {
        for (;;) {
            const int i = next.fetch_add(1, std::memory_order_relaxed);
            if ((long long)i * piece >= n_slices) return;
            const int j0 = i * piece, j1 = int(std::min<long long>(n_slices, (long long)j0 + piece));
            double t;
            const long long q = step_scalars(p, t0, L, dt, S, rem, S_tot, dx, j0, j1, step, &t);
            // a thread's pieces come in order, so the first found is its smallest
            if (q >= 0 && found[size_t(k)].q < 0) found[size_t(k)] = {q, t};
        }
    };
    std::vector<std::thread> pool;
    pool.reserve(size_t(nth));
    for (int k = 1; k < nth; ++k) {
        try {
            pool.emplace_back(work, k);
        } catch (const std::system_error &) {
            break;                           // go on with the threads there are
        }
    }
    work(0);
    for (std::thread &t : pool) t.join();
    long long first = -1;
    for (const Found &f : found)
        if (f.q >= 0 && (first < 0 || f.q < first)) {
            first = f.q;
            *bad_t = f.t;
        }
    return first;
}

// The maps of level v: the slices' (0), or the products of blocks of level v - 1.
LevelArgs level_args(const nv_lin *l, int v, bool blocked, bool whole) {
    LevelArgs a{};
    a.T = v == 0 ? l->T : l->product[v - 1];
    a.M = l->M;
    a.N = l->N;
    a.maps = l->N;
    a.stride = 1;
    for (int u = 0; u < v; ++u) {
        a.maps = (a.maps + kBlock - 1) / kBlock;
        a.stride *= kBlock;
    }
    a.whole = whole ? 1 : 0;
    a.largest = blocked ? kLargest : 1.7976931348623157e308;
    return a;
}

// The products of every level (the first launch also clears l->bad).
hipError_t launch_products(nv_lin *l) {
    for (int v = 0; v < l->levels; ++v) {
        ManyArgs a{};
        a.lv = level_args(l, v, true, false);
        a.product = l->product[v];
        a.bad = l->bad;
        lin_many.f[(l->M + 3) / 4 - 1](a, 0, l->stream);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// One chain through level v: all of it from y0, or every block of it from the
// state at its start.
hipError_t launch_chain(nv_lin *l, int v, bool whole) {
    ComposeArgs a{level_args(l, v, v > 0 || !whole, whole), l->y0, l->boundary, l->bad};
    lin_chain.f[(l->M + 7) / 8 - 1](a, l->stream);
    return hipGetLastError();
}

}  // namespace

extern "C" {

NV_API nv_status nv_lin_create(void *stream, nv_lin **out) try {
    if (!out) return fail(NV_ERR_INVALID_ARG, "NULL argument");
    *out = nullptr;
    nv_lin *l = new (std::nothrow) nv_lin();
    if (!l) return fail(NV_ERR_OOM, "out of host memory");
    l->stream = static_cast<hipStream_t>(stream);
    hipError_t e = hipEventCreate(&l->e0);
    if (e == hipSuccess) e = hipEventCreate(&l->e1);
    if (e == hipSuccess) e = hipEventCreate(&l->e2);
    if (e == hipSuccess) e = hipEventCreate(&l->e3);
    if (e != hipSuccess) {
        nv_lin_destroy(l);
        return fail(NV_ERR_HIP, "event creation failed: %s", hipGetErrorString(e));
    }
    *out = l;
    return NV_OK;
} catch (const std::bad_alloc &) {
    return fail(NV_ERR_OOM, "nv_lin_create: host allocation failed");
}

NV_API nv_status nv_lin_destroy(nv_lin *l) {
    if (!l) return NV_OK;
    if (l->mem) {
        (void)hipStreamSynchronize(l->stream);
        (void)hipFree(l->mem);
    }
    if (l->host) (void)hipHostFree(l->host);
    for (hipEvent_t ev : {l->e0, l->e1, l->e2, l->e3})
        if (ev) (void)hipEventDestroy(ev);
    delete l;
    return NV_OK;
}

NV_API nv_status nv_lin_build(nv_lin *l, const nv_heat *p, double t0, double T, int n_slices,
                              double dt) try {
#pragma clang fp contract(off)
    if (!l || !p) return fail(NV_ERR_INVALID_ARG, "NULL argument");
    l->built = false;                        // a failed build leaves nothing to compose
    if (p->M < 1 || p->M > kMaxM)
        return fail(NV_ERR_INVALID_ARG, "M = %d: need 1..%d interior points", p->M, kMaxM);
    if (n_slices < 1) return fail(NV_ERR_INVALID_ARG, "n_slices = %d", n_slices);
    if (!std::isfinite(t0) || !std::isfinite(T) || !(T > t0))
        return fail(NV_ERR_INVALID_ARG, "need finite t0 < T");
    if (!(dt > 0.0) || !std::isfinite(dt)) return fail(NV_ERR_INVALID_ARG, "dt must be > 0");
    if (!std::isfinite(p->a0) || !std::isfinite(p->a1))
        return fail(NV_ERR_INVALID_ARG, "a0, a1 must be finite");
    const int M = p->M;
    const double L = (T - t0) / double(n_slices);
    const double Sd = std::floor(L / dt + 1e-9);
    if (Sd > 1e7) return fail(NV_ERR_INVALID_ARG, "more than 1e7 steps per slice");
    const int S = int(Sd);
    double rem = L - double(S) * dt;
    if (!(rem > 1e-12 * L)) rem = 0.0;
    const int S_tot = S + (rem > 0.0 ? 1 : 0);
    if (S_tot < 1) return fail(NV_ERR_INVALID_ARG, "a slice takes no step");
    const long long nq = (long long)n_slices * S_tot;
    // per-step scalars on the host: r = (h a(t_end)) / (dx dx), h beta(t_end)
    const double dx = 1.0 / double(M + 1);
    // [step scalars][s], laid out as in device memory
    const size_t s_at = al(size_t(nq) * 2 * 8), up = s_at + size_t(M) * 8;
    const size_t results = (size_t(n_slices) + 1) * M * 8 + sizeof(double);
    ensure_host(l, std::max(up, results));
    std::vector<double> pageable;
    if (!l->host) pageable.resize(up / 8);
    double *step = l->host ? reinterpret_cast<double *>(l->host) : pageable.data();
    double *sv = step + s_at / 8;
    double bad_t = 0.0;
    if (all_step_scalars(*p, t0, L, dt, S, rem, S_tot, dx, n_slices, step, &bad_t) >= 0)
        return fail(NV_ERR_INVALID_ARG, "a(t) = %g is not positive at t = %g",
                    coef_at(*p, bad_t).a, bad_t);
    for (int i = 0; i < M; ++i) sv[i] = std::sin(M_PI * (double(i + 1) * dx));

    // device layout
    size_t off = 0;
    const size_t o_step = off; off = al(off + size_t(nq) * 2 * 8);
    const size_t o_s = off;    off = al(off + size_t(M) * 8);
    const size_t o_w = off;    off = al(off + size_t(nq) * M * 8);
    const size_t o_c = off;    off = al(off + size_t(nq) * M * 8);
    const size_t o_T = off;    off = al(off + size_t(n_slices) * lin_stride(M) * (M + 1) * 8);
    const size_t o_y0 = off;   off = al(off + size_t(M) * 8);
    // the boundary states and the report, next to each other: one copy back
    const size_t o_b = off;    off = off + (size_t(n_slices) + 1) * M * 8;
    const size_t o_bad = off;  off = al(off + sizeof(double));
    // the products of blocks of slices, level by level, where one launch can form
    // them and there is room for them (a seventh of the tables)
    const size_t without = off;
    size_t o_prod[kMaxLevels] = {};
    int levels = 0;
    if (n_slices >= kBlockedFrom && nv::lin::products_fit(M, n_slices))
        for (int maps = n_slices; maps > kTopMaps && levels < kMaxLevels; ++levels) {
            maps = (maps + kBlock - 1) / kBlock;
            o_prod[levels] = off;
            off = al(off + size_t(maps) * lin_stride(M) * (M + 1) * 8);
        }
    if (off > l->mem_bytes) {
        if (l->mem) {
            NV_HIP(hipStreamSynchronize(l->stream));
            NV_HIP(hipFree(l->mem));
            l->mem = nullptr;
            l->mem_bytes = 0;
        }
        hipError_t e = hipMalloc(reinterpret_cast<void **>(&l->mem), off);
        if (e != hipSuccess && levels > 0) {
            (void)hipGetLastError();
            levels = 0;
            off = without;
            e = hipMalloc(reinterpret_cast<void **>(&l->mem), off);
        }
        if (e != hipSuccess) {
            (void)hipGetLastError();
            l->mem = nullptr;
            l->built = false;
            return fail(NV_ERR_OOM, "device allocation of %zu bytes failed", off);
        }
        l->mem_bytes = off;
    }
    l->step = reinterpret_cast<double *>(l->mem + o_step);
    l->w = reinterpret_cast<double *>(l->mem + o_w);
    l->c = reinterpret_cast<double *>(l->mem + o_c);
    l->s = reinterpret_cast<double *>(l->mem + o_s);
    l->T = reinterpret_cast<double *>(l->mem + o_T);
    l->y0 = reinterpret_cast<double *>(l->mem + o_y0);
    l->boundary = reinterpret_cast<double *>(l->mem + o_b);
    l->bad = reinterpret_cast<int *>(l->mem + o_bad);
    l->levels = levels;
    for (int v = 0; v < levels; ++v) l->product[v] = reinterpret_cast<double *>(l->mem + o_prod[v]);
    l->M = M;
    l->N = n_slices;
    l->S_tot = S_tot;
    l->built = false;

    NV_HIP(hipMemcpyAsync(l->step, step, up, hipMemcpyHostToDevice, l->stream));
    NV_HIP(hipEventRecord(l->e0, l->stream));
    CoefArgs ca{l->step, l->w, l->c, nq, M};
    hipLaunchKernelGGL(lin_coef_kernel, dim3(unsigned((nq + 63) / 64)), dim3(64), 0,
                       l->stream, ca);
    NV_HIP(hipGetLastError());
    BuildArgs ba{l->step, l->w, l->c, l->s, l->T, M, S_tot, p->forcing ? 1 : 0};
    lin_build.f[(M + 7) / 8 - 1](ba, n_slices, l->stream);
    NV_HIP(hipGetLastError());
    NV_HIP(hipEventRecord(l->e1, l->stream));
    // the host's scalars must outlive the copy
    NV_HIP(hipStreamSynchronize(l->stream));
    NV_HIP(hipEventElapsedTime(&l->build_ms, l->e0, l->e1));
    l->built = true;
    return NV_OK;
} catch (const std::bad_alloc &) {
    return fail(NV_ERR_OOM, "nv_lin_build: host allocation failed");
}

NV_API nv_status nv_lin_compose(nv_lin *l, const double *y0, double *yT, double *boundary) {
    if (!l || !y0 || !yT) return fail(NV_ERR_INVALID_ARG, "NULL argument");
    if (!l->built) return fail(NV_ERR_NOT_BUILT, "no successful nv_lin_build");
    const int M = l->M, N = l->N;
    NV_HIP(hipMemcpyAsync(l->y0, y0, size_t(M) * 8, hipMemcpyHostToDevice, l->stream));
    NV_HIP(hipEventRecord(l->e2, l->stream));
    int bad = -1;
    // the states asked for and the report behind them, in one copy
    const bool staged = l->host != nullptr;
    const size_t first = boundary ? 0 : size_t(N) * M;
    const size_t results = ((size_t(N) + 1) * M - first) * 8 + sizeof(double);
    // by blocks; then, should a state be beyond what that serves, slice by slice
    for (int levels = l->fixed_order ? 0 : l->levels;; levels = 0) {
        if (levels > 0) NV_HIP(launch_products(l));
        NV_HIP(launch_chain(l, levels, true));
        for (int v = levels - 1; v >= 0; --v) NV_HIP(launch_chain(l, v, false));
        NV_HIP(hipEventRecord(l->e3, l->stream));
        if (staged) {
            NV_HIP(hipMemcpyAsync(l->host, l->boundary + first, results, hipMemcpyDeviceToHost,
                                  l->stream));
            NV_HIP(hipStreamSynchronize(l->stream));
            std::memcpy(&bad, l->host + results - sizeof(double), sizeof(int));
        } else {
            NV_HIP(hipMemcpyAsync(&bad, l->bad, sizeof(int), hipMemcpyDeviceToHost, l->stream));
            NV_HIP(hipMemcpyAsync(yT, l->boundary + size_t(N) * M, size_t(M) * 8,
                                  hipMemcpyDeviceToHost, l->stream));
            if (boundary)
                NV_HIP(hipMemcpyAsync(boundary, l->boundary, (size_t(N) + 1) * M * 8,
                                      hipMemcpyDeviceToHost, l->stream));
            NV_HIP(hipStreamSynchronize(l->stream));
        }
        if (levels == 0 || bad < 0) break;
    }
    if (staged) {
        if (boundary) std::memcpy(boundary, l->host, results - sizeof(double));
        std::memcpy(yT, l->host + results - sizeof(double) - size_t(M) * 8, size_t(M) * 8);
    }
    NV_HIP(hipEventElapsedTime(&l->compose_ms, l->e2, l->e3));
    if (bad >= 0) return fail(NV_ERR_NONFINITE, "the state became non-finite in slice %d", bad);
    return NV_OK;
}

NV_API nv_status nv_lin_compose_many(nv_lin *l, const double *y0_dev, long long count,
                                     double *yT_dev, double *boundary_dev) {
    if (!l || !y0_dev || !yT_dev) return fail(NV_ERR_INVALID_ARG, "NULL argument");
    if (count < 1) return fail(NV_ERR_INVALID_ARG, "count = %lld", count);
    if ((count + 15) / 16 > 0x7fffffffLL) return fail(NV_ERR_INVALID_ARG, "too many chains");
    if (!l->built) return fail(NV_ERR_NOT_BUILT, "no successful nv_lin_build");
    const int init = kNoSlice;
    int dev = 0, n_cu = 256;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        n_cu < 1)
        n_cu = 256;
    const long long pair_from = 2LL * n_cu * 32;
    const ManyLaunch run = lin_many.f[(l->M + 3) / 4 - 1];
    ManyArgs a{};
    a.y0 = y0_dev;
    a.yT = yT_dev;
    a.boundary = boundary_dev;
    a.bad = l->bad;
    a.Q = count;
    int bad = init;
    // by blocks (with states: while the chains are few, and if one launch can hold the
    // states inside the blocks); then, should a
    // state be beyond what that serves, slice by slice.  The final states may
    // overwrite the initial ones (a workgroup reads its chains before it writes
    // them), but a second pass would then start from the first one's results: such
    // a call takes the slices at once.
    const size_t bytes = size_t(count) * l->M * sizeof(double);
    const uintptr_t from = reinterpret_cast<uintptr_t>(y0_dev),
                    to = reinterpret_cast<uintptr_t>(yT_dev);
    const bool in_place = from < to + bytes && to < from + bytes;
    const bool by_blocks = !boundary_dev ||
                           (nv::lin::states_by_blocks(l->N, count, n_cu) &&
                            nv::lin::states_fit(l->M, l->N, count, pair_from));
    const int first = in_place || !by_blocks ? 0 : l->levels;
    for (int levels = first;; levels = 0) {
        // (the products' first launch clears the report itself)
        if (levels == 0)
            NV_HIP(hipMemcpyAsync(l->bad, &init, sizeof(int), hipMemcpyHostToDevice, l->stream));
        if (levels == first) NV_HIP(hipEventRecord(l->e2, l->stream));
        if (levels > 0) NV_HIP(launch_products(l));
        a.lv = level_args(l, levels, levels > 0, true);
        run(a, pair_from, l->stream);
        NV_HIP(hipGetLastError());
        if (boundary_dev)
            for (int v = levels - 1; v >= 0; --v) {
                a.lv = level_args(l, v, true, false);
                run(a, pair_from, l->stream);
                NV_HIP(hipGetLastError());
            }
        NV_HIP(hipEventRecord(l->e3, l->stream));
        NV_HIP(hipMemcpyAsync(&bad, l->bad, sizeof(int), hipMemcpyDeviceToHost, l->stream));
        NV_HIP(hipStreamSynchronize(l->stream));
        if (levels == 0 || bad == init) break;
    }
    NV_HIP(hipEventElapsedTime(&l->compose_ms, l->e2, l->e3));
    if (bad != init)
        return fail(NV_ERR_NONFINITE, "a state became non-finite in slice %d", bad);
    return NV_OK;
}

NV_API nv_status nv_lin_set_fixed_order(nv_lin *l, int on) {
    if (!l) return fail(NV_ERR_INVALID_ARG, "NULL argument");
    l->fixed_order = on != 0;
    return NV_OK;
}

NV_API nv_status nv_lin_get_tables(nv_lin *l, double *G, double *c) {
    if (!l) return fail(NV_ERR_INVALID_ARG, "NULL argument");
    if (!l->built) return fail(NV_ERR_NOT_BUILT, "no successful nv_lin_build");
    const size_t M = size_t(l->M), N = size_t(l->N), Ms = size_t(lin_stride(l->M)),
                 per = Ms * (M + 1);
    std::vector<double> t(N * per);
    NV_HIP(hipMemcpyAsync(t.data(), l->T, t.size() * 8, hipMemcpyDeviceToHost, l->stream));
    NV_HIP(hipStreamSynchronize(l->stream));
    for (size_t j = 0; j < N; ++j) {
        const double *b = t.data() + j * per;
        if (G)
            for (size_t k = 0; k < M; ++k)
                for (size_t i = 0; i < M; ++i) G[(j * M + i) * M + k] = b[k * Ms + i];
        if (c)
            for (size_t i = 0; i < M; ++i) c[j * M + i] = b[Ms * M + i];
    }
    return NV_OK;
}

NV_API nv_status nv_lin_last_timing(nv_lin *l, float *build_ms, float *compose_ms) {
    if (!l) return fail(NV_ERR_INVALID_ARG, "NULL argument");
    if (build_ms) *build_ms = l->build_ms;
    if (compose_ms) *compose_ms = l->compose_ms;
    return NV_OK;
}

}  // extern "C"
