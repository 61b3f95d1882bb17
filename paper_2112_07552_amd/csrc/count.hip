// count.hip -- products of 0/1 encodings (Section 3.1 of TCUDB): exact pair
// counts on the int8 matrix cores.
//
// A relation with unique cells and no values encodes to a 0/1 matrix, so the
// operator's result is an exact integer below 2^31: the contraction runs on
// int8 planes with int32 sums, and C gets the same doubles that an FP64
// product of the 0/1 matrices gives, at an eighth of the operand bytes and on
// matrix cores 64 times as fast.  The exact pair counts that a forward with
// values may ask for are the same product stored as int32.
#include "internal.h"

namespace tcu {
namespace {

typedef int i4 __attribute__((ext_vector_type(4)));
typedef double d2 __attribute__((ext_vector_type(2)));
typedef int i16v __attribute__((ext_vector_type(16)));

constexpr int kThreads = 256;
constexpr int BM = 128, BN = 128;  // 4 waves of 64 x 64
constexpr size_t kLastLevelCache = (size_t)256 << 20;

// plane[t / 32][(t % 32) / 16][line][t % 16]: the 16 bytes one lane feeds the
// matrix core are contiguous, and so are those of neighbouring lines
__device__ inline int64_t plane_offset(int line, int t, int lines_pad) {
    return (((int64_t)(t >> 5) * 2 + ((t >> 4) & 1)) * lines_pad + line) * 16 + (t & 15);
}

// A 1 at (line = group, position = key) of every in-range record, A's into
// plane qa and B's into qb (zeroed before); plain byte stores, as the cells
// are unique.  Records outside the shape are counted in the status block (st
// may be NULL: counted by another pass).
__global__ void __launch_bounds__(kThreads)
count_planes_kernel(int64_t na, const int32_t *__restrict__ ga, const int32_t *__restrict__ ka,
                    int64_t nb, const int32_t *__restrict__ gb, const int32_t *__restrict__ kb,
                    int M, int N, int K, int8_t *__restrict__ qa, int alp,
                    int8_t *__restrict__ qb, int blp, StatusBlock *st) {
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    const bool of_a = i < na;
    const int64_t j = of_a ? i : i - na;
    bool bad = false;
    if (i < na + nb) {
        const int g = of_a ? ga[j] : gb[j], k = of_a ? ka[j] : kb[j];
        bad = (unsigned)g >= (unsigned)(of_a ? M : N) || (unsigned)k >= (unsigned)K;
        if (!bad) {
            if (of_a) qa[plane_offset(g, k, alp)] = 1;
            else qb[plane_offset(g, k, blp)] = 1;
        }
    }
    if (st == nullptr) return;
    const unsigned long long all = __ballot(bad), of = __ballot(bad && of_a);
    if (all != 0ull && (threadIdx.x & 63) == 0) {
        atomicOr(&st->flags, kFlagKeyRange);
        if (of) atomicAdd(&st->skipped_a, (unsigned long long)__popcll(of));
        if (all != of) atomicAdd(&st->skipped_b, (unsigned long long)__popcll(all ^ of));
    }
}

// C[g, h] = sum over k of qa[g, k] qb[h, k] as doubles and / or int32.  The
// result's 8 bytes per cell bound it at the contraction lengths of a
// dictionary with few values (16384 x 16384 cells over 32 keys: 2.1 GB
// written, 1.7e10 integer operations), so what matters is many workgroups
// per CU whose stores overlap the others' loads: no LDS, each lane loads its
// matrix-core operands straight from the planes (two runs of 512 bytes per
// wave), one k-step ahead.  Workgroups take the tiles in row-major order, so
// that those in flight write long runs of the same rows: 377 us (5.7 TB/s; a
// plain fill reaches 6.7) against 438 us in the GEMMs' order of eight
// tile rows per XCD, and 504 us for the FP64 product (these with 8-byte
// stores).  A result larger than the last-level cache goes past the caches
// (NT), which then keep the planes:
// 33024 x 4096 cells over 512 keys 217 us against 334 us, FP64 2067 us; at
// 4096 x 4096 cells, which a next kernel may still find cached, it would gain
// nothing (127 and 130 us over 4096 keys, FP64 1959 us).
// A lane's two columns of a wave's 64 are neighbours (column block b holds the
// columns 2 l + b), so that a wave stores 512 bytes of a row per instruction
// (PAIR: an even n and aligned outputs; 8 bytes per store otherwise):
// 16384 x 16384 cells over 32 keys 360 us instead of 368, 33024 x 4096 over 512
// 175 instead of 194.  Stores of 8 bytes always go through the caches, which
// join them: 5001 x 7003 cells 73 us, past the caches 191.
template <bool NT, bool PAIR>
__global__ void __launch_bounds__(kThreads)
count_product_kernel(int m, int n, int nblk, int tiles_n,
                     const int8_t *__restrict__ xs, int xlp, const int8_t *__restrict__ ys,
                     int ylp, double *__restrict__ C, int64_t ldc, int32_t *__restrict__ cnt,
                     int64_t ldcnt) {
    const int m0 = (int)(blockIdx.x / (unsigned)tiles_n) * BM;
    const int n0 = (int)(blockIdx.x % (unsigned)tiles_n) * BN;

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int l32 = lane & 31, half = lane >> 5;
    const int r0 = m0 + (wave & 1) * 64, c0 = n0 + (wave >> 1) * 64;
    const int8_t *xp = xs + ((int64_t)half * xlp + r0 + l32) * 16;
    const int8_t *yp = ys + ((int64_t)half * ylp + c0 + 2 * l32) * 16;
    const int64_t xstep = (int64_t)xlp * 32, ystep = (int64_t)ylp * 32;

    i16v acc[2][2];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) acc[a][b] = i16v{};
    i4 xa[2], yb[2];
#pragma unroll
    for (int a = 0; a < 2; ++a) {
        xa[a] = *reinterpret_cast<const i4 *>(xp + a * 512);
        yb[a] = *reinterpret_cast<const i4 *>(yp + a * 16);
    }
    for (int kb = 0; kb < nblk; ++kb) {
        // the last k-step loads itself again
        if (kb + 1 < nblk) {
            xp += xstep;
            yp += ystep;
        }
        i4 xn[2], yn[2];
#pragma unroll
        for (int a = 0; a < 2; ++a) {
            xn[a] = *reinterpret_cast<const i4 *>(xp + a * 512);
            yn[a] = *reinterpret_cast<const i4 *>(yp + a * 16);
        }
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b)
                acc[a][b] =
                    __builtin_amdgcn_mfma_i32_32x32x32_i8(xa[a], yb[b], acc[a][b], 0, 0, 0);
#pragma unroll
        for (int a = 0; a < 2; ++a) {
            xa[a] = xn[a];
            yb[a] = yn[a];
        }
    }
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int row = r0 + a * 32 + 8 * (i >> 2) + 4 * half + (i & 3);
            const int col = c0 + 2 * l32;
            if (row >= m || col >= n) continue;
            const int v0 = acc[a][0][i], v1 = acc[a][1][i];
            if (C != nullptr) {
                double *dst = C + (int64_t)row * ldc + col;
                if (PAIR) {
                    if (NT) __builtin_nontemporal_store(d2{(double)v0, (double)v1},
                                                        reinterpret_cast<d2 *>(dst));
                    else *reinterpret_cast<d2 *>(dst) = d2{(double)v0, (double)v1};
                } else {
                    dst[0] = (double)v0;
                    if (col + 1 < n) dst[1] = (double)v1;
                }
            }
            if (cnt != nullptr) {
                int32_t *dst = cnt + (int64_t)row * ldcnt + col;
                if (PAIR) {
                    *reinterpret_cast<int2 *>(dst) = make_int2(v0, v1);
                } else {
                    *dst = v0;
                    if (col + 1 < n) dst[1] = v1;
                }
            }
        }
}

}  // namespace

int64_t count_lines_pad(int64_t lines) { return (lines + BM - 1) / BM * BM; }

size_t count_plane_bytes(int64_t lines, int64_t len) {
    return (size_t)count_lines_pad(lines) * (size_t)((len + 31) / 32 * 32);
}

hipError_t launch_count(const tcu_relation &A, const tcu_relation &B, int M, int K, int N,
                        int8_t *qa, int8_t *qb, StatusBlock *st, double *C, int32_t *cnt,
                        hipStream_t s) {
    const size_t ba = count_plane_bytes(M, K), bb = count_plane_bytes(N, K);
    // zeroed by a kernel, not a memset node (the call may be captured); the
    // sizes are multiples of 128 * 32
    hipError_t e = launch_zero_f64(reinterpret_cast<double *>(qa), ba / 8, s);
    if (e == hipSuccess) e = launch_zero_f64(reinterpret_cast<double *>(qb), bb / 8, s);
    if (e != hipSuccess) return e;
    const int alp = (int)count_lines_pad(M), blp = (int)count_lines_pad(N);
    auto place = [&](int64_t na, int64_t nb) {
        if (na + nb > 0)
            count_planes_kernel<<<(unsigned)((na + nb + kThreads - 1) / kThreads), kThreads, 0,
                                  s>>>(na, A.group, A.key, nb, B.group, B.key, M, N, K, qa, alp,
                                       qb, blp, st);
    };
    if (A.n + B.n <= max_workgroups(kThreads) * kThreads) {
        place(A.n, B.n);
    } else {  // too many records for one launch
        place(A.n, 0);
        place(0, B.n);
    }
    if ((e = hipGetLastError()) != hipSuccess) return e;
    return launch_count_planes_product(M, K, N, qa, qb, C, cnt, s);
}

hipError_t launch_count_planes_product(int M, int K, int N, const int8_t *qa, const int8_t *qb,
                                       double *C, int32_t *cnt, hipStream_t s) {
    const int alp = (int)count_lines_pad(M), blp = (int)count_lines_pad(N);
    TraceScope ts(TCU_KERNEL_COUNT, M, N, K, 1, 2.0 * M * N * (double)K, s);
    const int tiles_n = blp / BN, nblk = (K + 31) / 32;
    const unsigned grid = (unsigned)((int64_t)(alp / BM) * tiles_n);
    const bool pair = N % 2 == 0 && ((uintptr_t)C & 15) == 0 && ((uintptr_t)cnt & 7) == 0;
    const bool nt = pair && (size_t)M * (size_t)N * sizeof(double) > kLastLevelCache;
    auto *kernel = nt     ? count_product_kernel<true, true>
                   : pair ? count_product_kernel<false, true>
                          : count_product_kernel<false, false>;
    kernel<<<grid, kThreads, 0, s>>>(M, N, nblk, tiles_n, qa, alp, qb, blp, C, N, cnt, N);
    return hipGetLastError();
}

}  // namespace tcu
