// gemm_f64.hip -- step a2 (the contraction C = X * Y of TCUDB Section 3.3)
// and the two products of the adjoint, in FP64 on the CDNA4 matrix cores.
//
// C (m x n) = op(A) (m x k) * op(B) (k x n), all FP64; C overwritten, or
// (accumulate) C += op(A) op(B).
//
// Design (gfx950):
//  * v_mfma_f64_16x16x4_f64: one wave multiplies a 16x4 by a 4x16 block;
//    A lane holds A[lane%16][lane/16], B lane holds B[lane/16][lane%16], the
//    accumulator lane holds D[lane/16 + 4*i][lane%16], i = 0..3 (measured on
//    gfx950: rows interleave with stride 4 across the lane groups).
//  * Workgroup tile 128 x 128, 4 waves in a 2 x 2 grid, each wave owning a
//    64 x 64 block (4 x 4 MFMA blocks, 64 FP64 accumulators per lane).
//  * K advances in stages of 16 through double-buffered LDS, one barrier per
//    stage.  Everything but the MFMAs is issued between them, one item after
//    each (64 cycles): the next k-step's fragments, stage s + 1's global loads
//    (k-step 0) and their LDS stores (k-step 2); see full_stage.  With the loads
//    and each k-step's fragment reads in front of its MFMAs instead, 4096^3 took
//    1940 us (70.8 TFLOP/s) and 2048^3 309; now 1867 (73.6, NT and TN 74.2) and
//    278.  The kernel stays within 128 VGPRs + 128 AGPRs, so two workgroups (two
//    waves per SIMD) share a CU and cover each other's barriers.
//  * Inside a stage, lane group j = lane/16 at k-step t (0..3) contracts
//    k = 4t + j (any bijection of the 16 k values is a valid contraction
//    order as long as A and B use the same one).
//  * Operands whose contraction index is contiguous in memory are staged as
//    [outer][16 + 2] in LDS, the others as [16][128 + 16]: with these pads the
//    32 lanes that LDS serves together read 64 different banks.  Global loads
//    are 16-byte vectors at any 8-byte alignment.
//  * Tiles are numbered so that each of the 8 XCDs (workgroup w runs on XCD
//    w mod 8) owns a contiguous run of tiles, grouped 8 tile-rows deep, so
//    the A and B panels a run needs stay in that XCD's L2.
//  * The tile kernel runs products of at least one tile (m, n >= 128, k >=
//    16); edge tiles are moved back inside the matrix, and the last k % 16
//    terms come straight from memory.  Its main loop's address arithmetic is
//    all scalar (see the tile path below): busy matrix cores leave vector-ALU
//    instructions few issue slots.
//  * Products whose output has too few 128 x 128 tiles to fill the chip, or
//    edges that waste much of one, run on the direct kernel (below), whose
//    tiles are an eighth or a sixteenth of that; pick_kernel holds the rule.
//  * Where such an output's contraction is long it is split into chunks over
//    workgroups, on either kernel, and the partial products are added up in
//    chunk order; pick_split holds the rule.  No chain of additions is longer
//    than a chunk of the 128 x 128 tiles' split.
#include <math.h>

#include <algorithm>
#include <type_traits>

#include "internal.h"

namespace tcu {
namespace {

typedef double d4 __attribute__((ext_vector_type(4)));

constexpr int BM = 128, BN = 128, BK = 16;
constexpr int THREADS = 256;
constexpr int WM = 64, WN = 64;
constexpr int FM = WM / 16, FN = WN / 16;
constexpr int KPAD = BK + 2;    // row stride of a contraction-contiguous tile
constexpr int OPAD = 128 + 16;  // row stride of an outer-contiguous tile
constexpr int GROUP_M = 8;
constexpr int NUM_XCD = 8;

template <bool KC>
struct Tile {
    static constexpr int elems = KC ? 128 * KPAD : BK * OPAD;
};

// Chunk i of a thread (2 doubles) to its place in an LDS tile.
template <bool KC>
__device__ __forceinline__ void store_chunk(double *__restrict__ L, int i, double2 v) {
    const int c = threadIdx.x + THREADS * i;
    const int off = KC ? (c >> 3) * KPAD + (c & 7) * 2 : (c >> 6) * OPAD + (c & 63) * 2;
    *reinterpret_cast<double2 *>(L + off) = v;
}

// The lane's element of MFMA block b in k-step t of a stage: row or column
// wbase + 16 b + lane % 16, k = 4 t + lane / 16.
template <bool KC>
__device__ __forceinline__ double read_frag(const double *__restrict__ L, int wbase, int t, int b) {
    const int lane = threadIdx.x & 63;
    const int o = wbase + b * 16 + (lane & 15), k = 4 * t + (lane >> 4);
    return KC ? L[o * KPAD + k] : L[k * OPAD + o];
}

// ----- tile path: no vector-ALU work in the main loop.  While the matrix
// cores are busy, VALU instructions of every wave on the SIMD get few issue
// slots, so the loop keeps its address arithmetic scalar: each panel load is a
// uniform SGPR base (advanced by scalar arithmetic) plus the lane's fixed 32-bit
// byte offset, and the loop is unrolled over the two LDS buffers so every LDS
// access is a fixed register plus an immediate.

typedef __attribute__((address_space(1))) const char gchar;
// 16-byte loads at 8-byte alignment (global memory takes them): leading
// dimensions, base addresses and moved tiles may be odd
typedef double d2v __attribute__((ext_vector_type(2), aligned(8)));
typedef __attribute__((address_space(1))) const d2v gd2v;
typedef __attribute__((address_space(1))) const double gdbl;

// A uniform global address computed on the vector ALU moved to scalar
// registers (kept in the global address space, so loads stay global loads).
__device__ __forceinline__ gchar *to_sgpr(const double *p) {
    const uint64_t u = (uint64_t)(uintptr_t)p;
    // the builtin returns int: widen through uint32_t (zero-extend)
    const uint64_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((unsigned)u);
    const uint64_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((unsigned)(u >> 32));
    return (gchar *)(uintptr_t)(lo | (hi << 32));
}

// One operand's panel loads: stage kt's chunk i of this lane is at byte
// base + kt * step + i * istep + off.  Chunk i of a thread is chunk 0 moved
// by 32 tile rows (KC) or 4 k rows (!KC), a uniform stride, so one 32-bit
// lane offset serves all four.
struct Panel {
    gchar *base;
    int64_t step, istep;
    unsigned off;
};

template <bool KC>
__device__ __forceinline__ Panel make_panel(const double *P, int64_t ld, int o0) {
    Panel q;
    const unsigned tid = threadIdx.x;
    q.base = to_sgpr(KC ? P + (int64_t)o0 * ld : P + o0);
    q.step = KC ? (int64_t)BK * 8 : (int64_t)BK * ld * 8;
    q.istep = KC ? (int64_t)(THREADS / 8) * ld * 8 : (int64_t)(THREADS / 64) * ld * 8;
    // chunk 0: KC (o, kk) = (tid / 8, 2 (tid % 8)); !KC (kk, o) = (tid / 64, 2 (tid % 64))
    const unsigned ldu = (unsigned)ld;
    q.off = KC ? ((tid >> 3) * ldu + (tid & 7) * 2u) * 8u : ((tid >> 6) * ldu + (tid & 63) * 2u) * 8u;
    return q;
}

// Chunk i of stage kt.
__device__ __forceinline__ double2 load_chunk(const Panel &q, int kt, int i) {
    gchar *bi = q.base + (int64_t)kt * q.step + i * q.istep;
    asm volatile("" : "+s"(bi));  // keep the chunk's base a scalar operand
    // Redefine the offset here so its zero extension is not hoisted out of
    // the loop: the SGPR-base + 32-bit-offset load form needs to see it.
    unsigned off = q.off;
    asm volatile("" : "+v"(off));
    // a native vector load (a HIP double2 copied from the global address
    // space would go through private memory)
    const d2v v = *reinterpret_cast<gd2v *>(bi + off);
    return make_double2(v.x, v.y);
}

struct Frags {
    double a[FM], b[FN];
};

// One stage of the tile loop on LDS buffer CUR, whose k-step 0 is in f0
// already: while the 16 MFMAs of a k-step run, one after the other, the next
// k-step's fragments are read, stage kt + 1's chunks are loaded (k-step 0) and
// stored to buffer CUR ^ 1 (k-step 2); the workgroup meets before the last
// k-step, which then reads stage kt + 1's k-step 0.  No wave reads buffer
// CUR ^ 1 between the previous stage's meeting and this one's.  (The last stage
// loads itself again, into a buffer that is not multiplied any more.)
template <bool A_KC, bool B_KC, int CUR>
__device__ __forceinline__ void full_stage(int kt, int nk, const Panel &pa, const Panel &pb,
                                           double (*lds_a)[Tile<A_KC>::elems],
                                           double (*lds_b)[Tile<B_KC>::elems], int wm, int wn,
                                           Frags &f0, d4 (&acc)[FM][FN]) {
    static_assert(FM * FN >= FM + FN && FM * FN >= 8, "one read or load per MFMA");
    double2 r[8];
    const int knext = kt + 1 < nk ? kt + 1 : kt;
    Frags f = f0;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        if (t == 3) __syncthreads();
        const double *la = lds_a[t == 3 ? CUR ^ 1 : CUR], *lb = lds_b[t == 3 ? CUR ^ 1 : CUR];
        Frags g;
#pragma unroll
        for (int i = 0; i < FM * FN; ++i) {
            acc[i / FN][i % FN] = __builtin_amdgcn_mfma_f64_16x16x4f64(
                f.a[i / FN], f.b[i % FN], acc[i / FN][i % FN], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            if (i < FM) g.a[i] = read_frag<A_KC>(la, wm * WM, (t + 1) % 4, i);
            else if (i < FM + FN) g.b[i - FM] = read_frag<B_KC>(lb, wn * WN, (t + 1) % 4, i - FM);
            if (t == 0 && i < 8) r[i] = i < 4 ? load_chunk(pa, knext, i) : load_chunk(pb, knext, i - 4);
            if (t == 2 && i < 4) store_chunk<A_KC>(lds_a[CUR ^ 1], i, r[i]);
            else if (t == 2 && i < 8) store_chunk<B_KC>(lds_b[CUR ^ 1], i - 4, r[i]);
            __builtin_amdgcn_sched_barrier(0);
        }
        f = g;
    }
    f0 = f;
}

template <int TILE_M, int TILE_N>
__device__ inline void tile_coords(int m, int n, int &tm, int &tn) {
    const int tiles_m = (m + TILE_M - 1) / TILE_M, tiles_n = (n + TILE_N - 1) / TILE_N;
    const int nt = tiles_m * tiles_n;
    const int wg = blockIdx.x;
    const int per = nt / NUM_XCD;
    const int full = per * NUM_XCD;
    const int logical = wg < full ? (wg % NUM_XCD) * per + wg / NUM_XCD : wg;
    const int group = GROUP_M * tiles_n;
    const int first_m = (logical / group) * GROUP_M;
    const int gm = min(tiles_m - first_m, GROUP_M);
    const int in_group = logical % group;
    tm = first_m + in_group % gm;
    tn = in_group / gm;
}

// A_KC: op(A)'s contraction index is contiguous (trans_a == 0).
// B_KC: op(B)'s contraction index is contiguous (trans_b == 1).
// Every tile is whole: edge tiles are moved back to end at m (or n), and the
// stores skip the cells a moved tile shares with its neighbour.
// kc > 0: split contraction, workgroup row y of the grid multiplies the chunk
// [y kc, (y + 1) kc) of k (at least BK of it) into its own partial product at C +
// y cstride.
template <bool A_KC, bool B_KC>
__global__ void __launch_bounds__(THREADS) __attribute__((amdgpu_waves_per_eu(2, 2)))
gemm_f64_kernel(int m, int n, int k, const double *__restrict__ A, int64_t lda,
                const double *__restrict__ B, int64_t ldb, double *__restrict__ C, int64_t ldc,
                int accumulate, int kc, int64_t cstride, const uint32_t *only_if) {
    if (only_if != nullptr && *only_if == 0u) return;
    __shared__ __attribute__((aligned(16))) double lds_a[2][Tile<A_KC>::elems];
    __shared__ __attribute__((aligned(16))) double lds_b[2][Tile<B_KC>::elems];
    if (kc > 0) {
        const int c0 = (int)blockIdx.y * kc;
        A += A_KC ? (int64_t)c0 : (int64_t)c0 * lda;
        B += B_KC ? (int64_t)c0 : (int64_t)c0 * ldb;
        C += (int64_t)blockIdx.y * cstride;
        k = min(kc, k - c0);
    }

    int tm, tn;
    tile_coords<BM, BN>(m, n, tm, tn);
    // the cells this tile owns start at (rlo, clo)
    const int rlo = tm * BM, clo = tn * BN;
    const int m0 = min(rlo, m - BM), n0 = min(clo, n - BN);

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave & 1, wn = wave >> 1;
    const int lane = threadIdx.x & 63;
    const int j = lane >> 4, l16 = lane & 15;

    d4 acc[FM][FN];
#pragma unroll
    for (int a = 0; a < FM; ++a)
#pragma unroll
        for (int b = 0; b < FN; ++b) acc[a][b] = d4{0.0, 0.0, 0.0, 0.0};

    const int nk = k / BK;  // at least 1
    const Panel pa = make_panel<A_KC>(A, lda, m0);
    const Panel pb = make_panel<B_KC>(B, ldb, n0);
    {
        double2 r[8];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            r[i] = load_chunk(pa, 0, i);
            r[i + 4] = load_chunk(pb, 0, i);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            store_chunk<A_KC>(lds_a[0], i, r[i]);
            store_chunk<B_KC>(lds_b[0], i, r[i + 4]);
        }
    }
    __syncthreads();
    Frags f0;
#pragma unroll
    for (int i = 0; i < FM; ++i) f0.a[i] = read_frag<A_KC>(lds_a[0], wm * WM, 0, i);
#pragma unroll
    for (int i = 0; i < FN; ++i) f0.b[i] = read_frag<B_KC>(lds_b[0], wn * WN, 0, i);
    for (int kt = 0; kt < nk; kt += 2) {
        full_stage<A_KC, B_KC, 0>(kt, nk, pa, pb, lds_a, lds_b, wm, wn, f0, acc);
        if (kt + 1 < nk)
            full_stage<A_KC, B_KC, 1>(kt + 1, nk, pa, pb, lds_a, lds_b, wm, wn, f0, acc);
    }
    // the last k % 16 terms, lane group j's term of step t at k = 4 t + j
    for (int kk = nk * BK; kk < k; kk += 4) {
        const int gk = kk + j;
        double fa[FM], fb[FN];
#pragma unroll
        for (int a = 0; a < FM; ++a) {
            const int64_t o = m0 + wm * WM + a * 16 + l16;
            fa[a] = gk < k ? A[A_KC ? o * lda + gk : (int64_t)gk * lda + o] : 0.0;
        }
#pragma unroll
        for (int b = 0; b < FN; ++b) {
            const int64_t o = n0 + wn * WN + b * 16 + l16;
            fb[b] = gk < k ? B[B_KC ? o * ldb + gk : (int64_t)gk * ldb + o] : 0.0;
        }
#pragma unroll
        for (int a = 0; a < FM; ++a)
#pragma unroll
            for (int b = 0; b < FN; ++b)
                acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[a], fb[b], acc[a][b], 0, 0, 0);
    }

#pragma unroll
    for (int a = 0; a < FM; ++a) {
#pragma unroll
        for (int b = 0; b < FN; ++b) {
            const int col = n0 + wn * WN + b * 16 + l16;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int row = m0 + wm * WM + a * 16 + j + 4 * i;
                if (row >= rlo && col >= clo) {
                    double *dst = C + (int64_t)row * ldc + col;
                    *dst = accumulate ? *dst + acc[a][b][i] : acc[a][b][i];
                }
            }
        }
    }
}

// ----- direct path: small tiles, fragments straight from memory.  A
// workgroup's four waves share one tile of 16 TM x 16 TN cells and split the
// contraction, so a wave needs neither LDS nor barriers until the four partial
// tiles are added at the end (in wave order: the same result on every run).
// What bounds it is the latency of its loads: three stages of 16 k are in
// registers, each stage's loads issued one after every MFMA (64 cycles), since
// loads issued in one run leave the matrix pipe idle (2048^3 products 262 us
// against 299 with the loads first).  Any edge and alignment is taken: rows
// past the end are clamped to the last one and not stored.
//
// k within a stage: lane group j's element t is k = 8 (t / 2) + 2 j + t % 2,
// so a lane of an operand with contiguous k reads 16 bytes and four lanes 64
// contiguous ones.  An operand with contiguous outer index is read in pairs
// of blocks: lane l's elements are columns 2 l and 2 l + 1 of the pair's 32,
// one 16-byte load (tiles at an edge: one 8-byte load per block).
// WIDE: lane offsets beyond 32 bits (huge leading dimensions).
template <bool KC, int F, bool WIDE>
struct DirectOp {
    gchar *base;  // the tile's first outer index, the wave's first k
    int64_t ldb;  // bytes between consecutive values of the strided index
    typename std::conditional<WIDE, uint64_t, uint32_t>::type off[F];
};

template <bool KC, int F, bool WIDE>
__device__ __forceinline__ DirectOp<KC, F, WIDE> direct_op(const double *P, int64_t ld, int o0,
                                                           int ext, int k0) {
    typedef typename std::conditional<WIDE, uint64_t, uint32_t>::type off_t;
    const int j = (threadIdx.x & 63) >> 4, l16 = threadIdx.x & 15;
    DirectOp<KC, F, WIDE> q;
    q.base = to_sgpr(KC ? P + (int64_t)o0 * ld + k0 : P + (int64_t)k0 * ld + o0);
    q.ldb = ld * 8;
#pragma unroll
    for (int b = 0; b < F; ++b) {
        const int o = min(KC ? 16 * b + l16 : 32 * (b >> 1) + 2 * l16 + (b & 1), ext - 1 - o0);
        q.off[b] = KC ? ((off_t)o * (off_t)ld + 2u * j) * 8u : (2u * j * (off_t)ld + (off_t)o) * 8u;
    }
    return q;
}

// Loads per stage of one operand.
template <bool KC, int F, bool EDGE>
constexpr int direct_items() { return KC ? 2 * F : (EDGE ? 4 * F : 2 * F); }

// Load I of the stage whose first k is at byte address b.
template <bool KC, int F, bool EDGE, bool WIDE>
__device__ __forceinline__ void direct_load(const DirectOp<KC, F, WIDE> &o, gchar *b, int I,
                                            double (&f)[F][4]) {
    const int blk = KC ? I >> 1 : (EDGE ? I >> 2 : (I >> 2) * 2);
    const int t = KC ? 2 * (I & 1) : I & 3;
    gchar *bi = KC ? b + 32 * t : b + (8 * (t >> 1) + (t & 1)) * o.ldb;
    auto off = o.off[blk];
    // a scalar base and a lane offset, as load_chunk
    asm volatile("" : "+s"(bi));
    asm volatile("" : "+v"(off));
    if (KC || !EDGE) {
        const d2v v = *reinterpret_cast<gd2v *>(bi + off);
        f[blk][t] = v.x;
        if (KC) f[blk][t + 1] = v.y;
        else f[blk + 1][t] = v.y;
    } else {
        f[blk][t] = *reinterpret_cast<gdbl *>(bi + off);
    }
}

// Adds the wave's accumulators to its own place in LDS (`first`: sets it), item e
// of this lane at run[64 e], and clears them.
template <int TM, int TN>
__device__ __forceinline__ void fold_run(d4 (&acc)[TM][TN], double *run, bool first) {
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                double *p = run + ((a * TN + b) * 4 + i) * 64;
                *p = first ? acc[a][b][i] : *p + acc[a][b][i];
                acc[a][b][i] = 0.0;
            }
}

// The stages 0 .. S - 1 of 16 k, S >= 1, of `total` (one more where a remainder
// of k follows them).  An accumulator takes at most `stages` of them before its
// run is folded away: the error of a sum grows with the length of its chain of
// additions, and where these kernels stand in for the split contraction of 128 x
// 128 tiles, runs are no longer than its chunks (kOneRun elsewhere).  Relative
// RMS error of uniform values with that split, with one chain per wave, and with
// runs: 1024 x 1024 x 4096 2.3e-16, 4.1e-16 and 2.0e-16; 1408 x 1408 x 8192
// 5.0e-16, 5.8e-16 and 3.0e-16.  A fold costs 1 to 2 us of LDS traffic,
// which all waves have at the same time (1024 x 1024 x 2048, two folds: 67.5 and
// 71.2 us; x 4096 127.1 and 130.7); with the folds between two loops over stages
// instead of in one it took the same.
// Returns whether a run has been folded.  RUNS: a wave has more stages than one
// run takes; without the folds' code 1024^3 takes 37.4 us, with it 38.1.
template <bool A_KC, bool B_KC, int TM, int TN, bool EDGE, bool WIDE, bool RUNS>
__device__ __forceinline__ bool direct_stages(const DirectOp<A_KC, TM, WIDE> &oa,
                                              const DirectOp<B_KC, TN, WIDE> &ob, int S,
                                              int total, int stages, d4 (&acc)[TM][TN],
                                              double *run) {
    constexpr int NB = TM * TN > 4 ? 3 : 2;  // stages in registers
    constexpr int IA = direct_items<A_KC, TM, EDGE>(), IB = direct_items<B_KC, TN, EDGE>();
    constexpr int MF = 4 * TM * TN;
    static_assert(IA + IB <= 2 * MF, "at most two loads per MFMA");
    constexpr int R = (IA + IB + MF - 1) / MF;
    const int64_t sa = A_KC ? 128 : 16 * oa.ldb, sb = B_KC ? 128 : 16 * ob.ldb;
    double fa[NB][TM][4], fb[NB][TN][4];
#pragma unroll
    for (int u = 0; u < NB - 1; ++u) {
        gchar *ba = oa.base + min(u, S - 1) * sa, *bb = ob.base + min(u, S - 1) * sb;
#pragma unroll
        for (int i = 0; i < IA; ++i) direct_load<A_KC, TM, EDGE, WIDE>(oa, ba, i, fa[u]);
#pragma unroll
        for (int i = 0; i < IB; ++i) direct_load<B_KC, TN, EDGE, WIDE>(ob, bb, i, fb[u]);
    }
    // runs of equal length, in whole rounds of NB stages
    int fold = 0, next = 0;
    if constexpr (RUNS) {
        const int runs = (total + stages - 1) / stages;
        fold = next = min((total + runs * NB - 1) / (runs * NB), stages / NB) * NB;
    }
    for (int s = 0; s < S; s += NB) {
#pragma unroll
        for (int u = 0; u < NB; ++u) {
            if (s + u >= S) continue;
            // the last stages load stage S - 1 again
            const int nx = min(s + u + NB - 1, S - 1);
            gchar *ba = oa.base + nx * sa, *bb = ob.base + nx * sb;
            asm volatile("" : "+s"(ba), "+s"(bb));
#pragma unroll
            for (int i = 0; i < MF; ++i) {
                const int t = i / (TM * TN), a = i % (TM * TN) / TN, b = i % TN;
                acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[u][a][t], fb[u][b][t],
                                                                 acc[a][b], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const int q = i * R + r;
                    if (q < IA)
                        direct_load<A_KC, TM, EDGE, WIDE>(oa, ba, q, fa[(u + NB - 1) % NB]);
                    else if (q < IA + IB)
                        direct_load<B_KC, TN, EDGE, WIDE>(ob, bb, q - IA, fb[(u + NB - 1) % NB]);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if constexpr (RUNS)
            if (s + NB == next && total - next > stages - fold) {
                fold_run<TM, TN>(acc, run, next == fold);
                next += fold;
            }
    }
    return next > fold;
}

// The last `left` (1 .. 15) values of k, past them zeros on both sides.
template <bool KC, int F, bool WIDE>
__device__ __forceinline__ void direct_tail(const DirectOp<KC, F, WIDE> &o, int S, int left,
                                            double (&f)[F][4]) {
    const int j = (threadIdx.x & 63) >> 4;
    gchar *b = o.base + S * (KC ? (int64_t)128 : 16 * o.ldb);
#pragma unroll
    for (int q = 0; q < F; ++q)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int kk = 8 * (t >> 1) + (t & 1);  // plus 2 j, already in the lane's offset
            double v = 0.0;
            if (2 * j + kk < left)
                v = *reinterpret_cast<gdbl *>(b + (KC ? (int64_t)8 * kk : kk * o.ldb) + o.off[q]);
            f[q][t] = v;
        }
}

// kc > 0: split contraction, as gemm_f64_kernel.  stages: of a run, at least 16;
// RUNS: a wave has more (direct_stages).
template <bool A_KC, bool B_KC, int TM, int TN, bool WIDE, bool RUNS>
__global__ void __launch_bounds__(THREADS)
gemm_direct_kernel(int m, int n, int k, const double *__restrict__ A, int64_t lda,
                   const double *__restrict__ B, int64_t ldb, double *__restrict__ C,
                   int64_t ldc, int accumulate, int kc, int64_t cstride, int stages,
                   const uint32_t *only_if) {
    if (only_if != nullptr && *only_if == 0u) return;
    constexpr int TILE_M = 16 * TM, TILE_N = 16 * TN, W = THREADS / 64, E = 4 * TM * TN;
    static_assert((A_KC || TM % 2 == 0) && (B_KC || TN % 2 == 0), "pairs of blocks");
    __shared__ double red[W * E * 64];
    if (kc > 0) {
        const int c0 = (int)blockIdx.y * kc;
        A += A_KC ? (int64_t)c0 : (int64_t)c0 * lda;
        B += B_KC ? (int64_t)c0 : (int64_t)c0 * ldb;
        C += (int64_t)blockIdx.y * cstride;
        k = min(kc, k - c0);
    }
    int tm, tn;
    tile_coords<TILE_M, TILE_N>(m, n, tm, tn);
    const int m0 = tm * TILE_M, n0 = tn * TILE_N;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63, j = lane >> 4, l16 = lane & 15;
    // the wave's share of k: whole stages, the remainder in the last share
    const int64_t kw = ((int64_t)k + W * BK - 1) / (W * BK) * BK;
    const int k0 = (int)min((int64_t)k, wave * kw), k1 = (int)min((int64_t)k, k0 + kw);
    const auto oa = direct_op<A_KC, TM, WIDE>(A, lda, m0, m, k0);
    const auto ob = direct_op<B_KC, TN, WIDE>(B, ldb, n0, n, k0);

    d4 acc[TM][TN];
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b) acc[a][b] = d4{0.0, 0.0, 0.0, 0.0};
    const int S = (k1 - k0) / BK, left = (k1 - k0) % BK;
    const int total = S + (left > 0 ? 1 : 0);
    double *run = red + wave * E * 64 + lane;
    bool folded = false;
    if (S > 0) {
        if ((A_KC || m0 + TILE_M <= m) && (B_KC || n0 + TILE_N <= n))
            folded = direct_stages<A_KC, B_KC, TM, TN, false, WIDE, RUNS>(oa, ob, S, total, stages,
                                                                          acc, run);
        else
            folded = direct_stages<A_KC, B_KC, TM, TN, true, WIDE, RUNS>(oa, ob, S, total, stages,
                                                                         acc, run);
    }
    if (left > 0) {
        double fa[TM][4], fb[TN][4];
        direct_tail<A_KC, TM, WIDE>(oa, S, left, fa);
        direct_tail<B_KC, TN, WIDE>(ob, S, left, fb);
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int a = 0; a < TM; ++a)
#pragma unroll
                for (int b = 0; b < TN; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[a][t], fb[b][t], acc[a][b],
                                                                     0, 0, 0);
    }
    // the waves' partial tiles, added in wave order
    fold_run<TM, TN>(acc, run, !folded);
    __syncthreads();
#pragma unroll
    for (int e0 = 0; e0 < E; e0 += W) {
        const int e = e0 + wave;
        double s = red[e * 64 + lane];
#pragma unroll
        for (int w = 1; w < W; ++w) s += red[(w * E + e) * 64 + lane];
        const int a = e / (4 * TN), b = e / 4 % TN, q = j + 4 * (e & 3);
        const int row = m0 + (A_KC ? 16 * a + q : 32 * (a >> 1) + 2 * q + (a & 1));
        const int col = n0 + (B_KC ? 16 * b + l16 : 32 * (b >> 1) + 2 * l16 + (b & 1));
        if (row < m && col < n) {
            double *dst = C + (int64_t)row * ldc + col;
            *dst = accumulate ? *dst + s : s;
        }
    }
}

// ------------------------------------------------------------- host side

constexpr int kOneRun = 0x7fffffff / 64;  // stages: no run is folded

// The kernels a product can run on.
enum Kernel { kTile, kDirectWide, kDirectSmall };  // 128 x 128; 32 x 64; 32 x 32

// Microseconds of an m x n x k product: full rounds of resident workgroups
// (two per CU of the first two, four of the last), then the rest with w
// workgroups per CU, at a share of the CU's 0.307 TFLOP/s that grows with w,
// plus the launch with its first loads and last stores.  The shares are fits
// to measured products (us, many in a row; tile, 32 x 64, 32 x 32): 512^3 -, 13,
// 8.4; 1024^3 126, 43, 45; 2048^3 278, 306, 332; 4096^3 1867, 1998, -; 1500 x
// 2777 x 2051 (264 tiles) 478, 336, 342; 3000^3 1030, 846, -.  The direct kernels
// read both operands of A B^T in 64-byte pieces of many rows, which costs them
// more (2048^3: 368, the tile kernel 265), and more yet where few tiles of a long
// contraction leave the reads their latency (1024 x 1024 x 8192 365 and 266 TN, 512
// x 512 x 16384 226 and 143).
// parts: that many such products, of k each, in one launch; 0: one product, of an
// output without room for partial products.
double kernel_us(Kernel which, bool nt, int m, int n, int k, int cus, int parts = 0) {
    struct Shape {
        int bm, bn, per_cu;
        double one, full, fixed;
    };
    Shape sh =
        which == kTile         ? Shape{BM, BN, 2, 0.84, 0.94, 8.0}
        : which == kDirectWide ? Shape{32, 64, 2, 0.65, nt ? 0.66 : 0.80, 6.0}
                               : Shape{32, 32, 4, 0.50, nt ? 0.58 : 0.68, 4.0};
    if (nt && parts > 0 && which == kDirectWide) sh.one = sh.full = 0.62;
    if (nt && parts > 0 && which == kDirectSmall) sh.full = sh.one;
    const double tiles =
        ceil((double)m / sh.bm) * ceil((double)n / sh.bn) * std::max(parts, 1);
    const double one_us = 2.0 * sh.bm * sh.bn * (double)k / 0.307e6;
    const double rounds = floor(tiles / (sh.per_cu * cus));
    const double left = tiles - rounds * sh.per_cu * cus;
    // (chunks of 128 x 128 tiles do not spread one to a CU beyond a few)
    const double w = which == kTile && parts > 1 && left > cus / 4 ? 2.0 : ceil(left / cus);
    double us = sh.fixed + rounds * sh.per_cu * one_us / sh.full;
    if (w > 0) us += w * one_us / (sh.one + (sh.full - sh.one) * (w - 1) / (sh.per_cu - 1));
    return us;
}

int device_cus() {
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        return 0;
    return cus;
}

// Whether every lane's byte offset inside a stage of `outer` rows or columns
// stays below 2^32.
bool offsets_fit(bool kc, int outer, int64_t ld) {
    return (kc ? outer * ld + BK : (int64_t)BK * ld + outer) * 8 < ((int64_t)1 << 32);
}

Kernel pick_kernel(bool a_kc, bool b_kc, int m, int n, int k, int64_t lda, int64_t ldb) {
    const int cus = std::max(1, device_cus());
    const bool nt = a_kc && b_kc;
    const double wide = kernel_us(kDirectWide, nt, m, n, k, cus);
    const double small = kernel_us(kDirectSmall, nt, m, n, k, cus);
    const bool tile_ok = m >= BM && n >= BN && k >= BK && offsets_fit(a_kc, BM, lda) &&
                         offsets_fit(b_kc, BN, ldb);
    if (tile_ok && kernel_us(kTile, nt, m, n, k, cus) <= std::min(wide, small)) return kTile;
    return wide < small ? kDirectWide : kDirectSmall;
}

template <bool A_KC, bool B_KC, int TM, int TN>
void launch_direct(int m, int n, int k, const double *A, int64_t lda, const double *B,
                   int64_t ldb, double *C, int64_t ldc, int accumulate, int kc, int parts,
                   int stages, const uint32_t *only_if, hipStream_t s) {
    const int64_t cstride = (int64_t)m * n;
    const bool narrow = offsets_fit(A_KC, std::min(m, 16 * TM), lda) &&
                        offsets_fit(B_KC, std::min(n, 16 * TN), ldb);
    // stages of a wave's share of the contraction
    constexpr int per_wave = THREADS / 64 * BK;
    const bool runs = ((int64_t)(kc > 0 ? kc : k) + per_wave - 1) / per_wave > stages;
    auto *kernel = narrow ? (runs ? gemm_direct_kernel<A_KC, B_KC, TM, TN, false, true>
                                  : gemm_direct_kernel<A_KC, B_KC, TM, TN, false, false>)
                          : (runs ? gemm_direct_kernel<A_KC, B_KC, TM, TN, true, true>
                                  : gemm_direct_kernel<A_KC, B_KC, TM, TN, true, false>);
    // as many tiles per launch as it may have workgroups (a C of 2^29 cells and
    // more in a line, or of 137 GB, takes several)
    const int64_t down = ((int64_t)m + 16 * TM - 1) / (16 * TM);
    const int64_t across = ((int64_t)n + 16 * TN - 1) / (16 * TN);
    const int64_t most = max_workgroups(THREADS);
    const int64_t step_n = std::min(across, most), step_m = std::min(down, most / step_n);
    for (int64_t tm = 0; tm < down; tm += step_m)
        for (int64_t tn = 0; tn < across; tn += step_n) {
            const int64_t r0 = tm * 16 * TM, c0 = tn * 16 * TN;
            const int mm = (int)std::min<int64_t>(m - r0, step_m * 16 * TM);
            const int nn = (int)std::min<int64_t>(n - c0, step_n * 16 * TN);
            const dim3 grid((unsigned)(std::min(down - tm, step_m) * std::min(across - tn, step_n)),
                            (unsigned)parts);
            kernel<<<grid, THREADS, 0, s>>>(mm, nn, k, A + (A_KC ? r0 * lda : r0), lda,
                                            B + (B_KC ? c0 * ldb : c0), ldb, C + r0 * ldc + c0,
                                            ldc, accumulate, kc, cstride, stages, only_if);
        }
}

// The product on kernel `which`; parts > 1: in chunks of kc of k, their partial
// products one after the other at C (ldc = n).  stages: of the direct kernels' runs.
template <bool A_KC, bool B_KC>
void launch_on(Kernel which, int m, int n, int k, const double *A, int64_t lda, const double *B,
               int64_t ldb, double *C, int64_t ldc, int accumulate, int kc, int parts,
               int stages, const uint32_t *only_if, hipStream_t s) {
    switch (which) {
        case kTile: {
            const dim3 grid((unsigned)(((m + BM - 1) / BM) * ((n + BN - 1) / BN)),
                            (unsigned)parts);
            gemm_f64_kernel<A_KC, B_KC><<<grid, THREADS, 0, s>>>(
                m, n, k, A, lda, B, ldb, C, ldc, accumulate, kc, (int64_t)m * n, only_if);
            break;
        }
        case kDirectWide:
            launch_direct<A_KC, B_KC, 2, 4>(m, n, k, A, lda, B, ldb, C, ldc, accumulate, kc, parts,
                                            stages, only_if, s);
            break;
        case kDirectSmall:
            launch_direct<A_KC, B_KC, 2, 2>(m, n, k, A, lda, B, ldb, C, ldc, accumulate, kc, parts,
                                            stages, only_if, s);
            break;
    }
}

template <bool A_KC, bool B_KC>
hipError_t launch(int m, int n, int k, const double *A, int64_t lda, const double *B,
                  int64_t ldb, double *C, int64_t ldc, int accumulate, const uint32_t *only_if,
                  hipStream_t s) {
    TraceScope ts(TCU_KERNEL_GEMM_F64, m, n, k, 1, 2.0 * m * n * (double)k, s);
    launch_on<A_KC, B_KC>(pick_kernel(A_KC, B_KC, m, n, k, lda, ldb), m, n, k, A, lda, B, ldb, C,
                          ldc, accumulate, 0, 1, kOneRun, only_if, s);
    return hipGetLastError();
}

// The split contraction's partial products summed in chunk order:
// C[i, j] = sum_p part[p][i * n + j], the same order on every run.
__global__ void __launch_bounds__(THREADS)
sum_partials_kernel(int m, int n, int parts, const double *__restrict__ part,
                    double *__restrict__ C, int64_t ldc) {
    const int64_t i = (int64_t)blockIdx.x * THREADS + threadIdx.x;
    const int64_t mn = (int64_t)m * n;
    if (i >= mn) return;
    double s = 0.0;
    for (int p = 0; p < parts; ++p) s += part[p * mn + i];
    C[(i / n) * ldc + i % n] = s;
}

// Partial products the workspace has room for, one per chunk of k: outputs of
// fewer than 128 tiles of 128 x 128, k at least 1024; two workgroups per CU,
// chunks of at least 256.  0: none.
int split_room(int m, int n, int k) {
    const int64_t tiles = (int64_t)((m + BM - 1) / BM) * ((n + BN - 1) / BN);
    if (tiles >= 128 || k < 1024) return 0;
    int64_t parts = (512 + tiles - 1) / tiles;
    parts = std::min<int64_t>(parts, k / 256);
    return parts >= 2 ? (int)parts : 0;
}

int split_chunk(int k, int parts) { return ((k + parts - 1) / parts + BK - 1) / BK * BK; }

// How a product with room for partial products runs: on the direct kernels in
// one piece or in as many chunks as give each CU one, two or four workgroups, or
// on the tile kernel in as many as there is room for (fewer would lengthen its
// chains of additions; the direct kernels' do not follow the chunks).  Few 32 x 32
// tiles take one workgroup per CU (64 x 64 x 4096 in 16 chunks 10.5 us, in one
// piece 40); elsewhere the estimate above decides, with a margin for its errors,
// which for chunks on the direct kernels reach a quarter.  us in one piece, on the
// tile kernel, on the direct kernels split, * taken: 1024^3 43* 52 -; 1024 x 1024 x
// 8192 NT 365 267* -; 512 x 512 x 65536 810 490* 540; 1024 x 128 x 65536 834 294*
// 442; 300 x 500 x 20000 267 134* 147; 100 x 1500 x 30000 411 - 218*; 768 x 768 x
// 8192 218 193* 190; 1408 x 1408 x 8192 510* 748 -.
struct SplitPlan {
    Kernel which;
    int parts;
};

SplitPlan pick_split(bool a_kc, bool b_kc, int m, int n, int k, int64_t lda, int64_t ldb) {
    const int room = split_room(m, n, k);
    const int tiles = ((m + 31) / 32) * ((n + 31) / 32);
    // few tiles: one workgroup per CU
    const int few = tiles <= 128 ? std::min((256 + tiles - 1) / tiles, room) : 1;
    const int kt = split_chunk(k, room);
    const bool tile_ok = m >= BM && n >= BN && (k % kt == 0 || k % kt >= BK) &&
                         offsets_fit(a_kc, BM, lda) && offsets_fit(b_kc, BN, ldb);
    SplitPlan best{kDirectSmall, few};
    if (tiles <= 128 && !tile_ok) return best;
    const int cus = std::max(1, device_cus());
    const bool nt = a_kc && b_kc;
    auto estimate = [&](Kernel which, int parts) {
        const int kc = parts > 1 ? split_chunk(k, parts) : k;
        const int used = (k + kc - 1) / kc;
        double us = kernel_us(which, nt, m, n, kc, cus, used);
        // the sum of the partial products: a launch, and one cell's loads one
        // after the other or all cells' bytes
        if (used > 1) us += 4.0 + std::max(0.22 * used, (used + 1) * (8.0 * m * n / 4.0e6));
        return us;
    };
    double best_us = estimate(kDirectSmall, few);
    // taken where the estimate is `margin` of the others' or less
    auto consider = [&](Kernel which, int parts, double margin) {
        parts = std::min(parts, room);
        if (parts < 2 && margin < 1.0) return;
        const double us = estimate(which, parts) / margin;
        if (us >= best_us) return;
        best_us = us;
        best = SplitPlan{which, parts};
    };
    if (tiles > 128) {
        const int wide = ((m + 31) / 32) * ((n + 63) / 64);
        consider(kDirectWide, 1, 1.0);
        consider(kDirectWide, 2 * cus / wide, 0.75);
        for (int w = 1; w <= 4; w *= 2) {
            consider(kDirectSmall, w * cus / tiles, 0.75);
            consider(kDirectSmall, (w * cus + tiles - 1) / tiles, 0.75);
        }
    }
    // (a few tiles' estimate errs more: 300 x 300 x 9000 A B^T 68 us for 88)
    if (tile_ok) consider(kTile, room, tiles <= 128 ? 0.85 : 0.93);
    return best;
}

template <bool A_KC, bool B_KC>
hipError_t launch_split(int m, int n, int k, const double *A, int64_t lda, const double *B,
                        int64_t ldb, double *C, int64_t ldc, double *part, hipStream_t s) {
    const SplitPlan p = pick_split(A_KC, B_KC, m, n, k, lda, ldb);
    const int kc = p.parts > 1 ? split_chunk(k, p.parts) : 0;
    const int used = kc > 0 ? (k + kc - 1) / kc : 1;  // chunks that hold part of k
    {
        TraceScope ts(TCU_KERNEL_GEMM_F64, m, n, k, used, 2.0 * m * n * (double)k, s);
        const int stages = split_chunk(k, split_room(m, n, k)) / BK;
        if (used == 1)
            launch_on<A_KC, B_KC>(p.which, m, n, k, A, lda, B, ldb, C, ldc, 0, 0, 1, stages,
                                  nullptr, s);
        else
            launch_on<A_KC, B_KC>(p.which, m, n, k, A, lda, B, ldb, part, n, 0, kc, used, stages,
                                  nullptr, s);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || used == 1) return e;
    const int64_t mn = (int64_t)m * n;
    sum_partials_kernel<<<(unsigned)((mn + THREADS - 1) / THREADS), THREADS, 0, s>>>(
        m, n, used, part, C, ldc);
    return hipGetLastError();
}

}  // namespace

size_t gemm_f64_split_bytes(int m, int n, int k) {
    const int parts = split_room(m, n, k);
    return parts == 0 ? 0 : (size_t)parts * (size_t)m * (size_t)n * sizeof(double);
}

hipError_t launch_gemm_f64_split(int trans_a, int trans_b, int m, int n, int k, const double *A,
                                 int64_t lda, const double *B, int64_t ldb, double *C,
                                 int64_t ldc, double *part, hipStream_t s) {
    if (split_room(m, n, k) == 0 || part == nullptr)
        return launch_gemm_f64(trans_a, trans_b, m, n, k, A, lda, B, ldb, C, ldc, s);
    if (!trans_a && !trans_b)
        return launch_split<true, false>(m, n, k, A, lda, B, ldb, C, ldc, part, s);
    if (!trans_a && trans_b)
        return launch_split<true, true>(m, n, k, A, lda, B, ldb, C, ldc, part, s);
    if (trans_a && !trans_b)
        return launch_split<false, false>(m, n, k, A, lda, B, ldb, C, ldc, part, s);
    return launch_split<false, true>(m, n, k, A, lda, B, ldb, C, ldc, part, s);
}

int gemm_f64_row_cut(int m, int n, int k) {
    const int cus = device_cus();
    if (cus <= 0) return 0;
    // two workgroups per CU: each is 4 waves, and the kernel runs 2 waves per SIMD
    const int64_t resident = 2 * (int64_t)cus;
    const int64_t rt = (m + BM - 1) / BM, ct = (n + BN - 1) / BN;
    auto rounds = [&](int64_t tiles) { return (tiles + resident - 1) / resident; };
    const int64_t whole = rounds(rt * ct);
    if (whole < 2) return 0;
    // the most even cut among those that add no round
    auto skew = [&](int64_t r) { return 2 * r > rt ? 2 * r - rt : rt - 2 * r; };
    int64_t best = 0;
    for (int64_t r = 1; r < rt; ++r) {
        if (rounds(r * ct) + rounds((rt - r) * ct) != whole) continue;
        if (best == 0 || skew(r) < skew(best)) best = r;
    }
    // the whole and both parts on one kernel, so that the cut changes no bit
    const int m1 = (int)(best * BM);
    auto tile = [&](int rows) { return pick_kernel(false, false, rows, n, k, m, n) == kTile; };
    return m1 > 0 && tile(m) && tile(m1) && tile(m - m1) ? m1 : 0;
}

hipError_t launch_gemm_f64(int trans_a, int trans_b, int m, int n, int k, const double *A,
                           int64_t lda, const double *B, int64_t ldb, double *C, int64_t ldc,
                           hipStream_t s, int accumulate, const uint32_t *only_if) {
    if (m == 0 || n == 0) return hipSuccess;
    if (!trans_a && !trans_b)
        return launch<true, false>(m, n, k, A, lda, B, ldb, C, ldc, accumulate, only_if, s);
    if (!trans_a && trans_b)
        return launch<true, true>(m, n, k, A, lda, B, ldb, C, ldc, accumulate, only_if, s);
    if (trans_a && !trans_b)
        return launch<false, false>(m, n, k, A, lda, B, ldb, C, ldc, accumulate, only_if, s);
    return launch<false, true>(m, n, k, A, lda, B, ldb, C, ldc, accumulate, only_if, s);
}

}  // namespace tcu
