// compact.hip -- nonzero(): the matrix-to-table conversion between the
// joins of a multi-way join (TCUDB Section 3.2, query Q2).
//
// After the first join, the n x m result matrix is turned back into the
// list of its nonzero cells, (i, j) with M[i,j] != 0, in row-major order, so
// that the next join can re-encode the surviving tuple pairs.  This is an
// HBM-bound stream compaction over the whole matrix (8 bytes read per
// cell), done in three passes:
//   1. every workgroup turns its chunk of 4096 cells into 64 words of one bit
//      per cell (wave ballots) and counts them;
//   2. one workgroup turns the chunk counts into exclusive offsets;
//   3. one wave per chunk reads its bits back and writes the (row, col) pairs
//      of its nonzeros at their offsets.
// The bits are a 64th of the matrix: reading the cells themselves again took
// 145 us beside the first pass's 84 us at 8192 x 8192 cells (6.4 TB/s, the
// rate a plain read reaches).
// Row-major order makes the output deterministic and identical to the
// order a sequential scan would give.  An optional column map replaces the
// column by map[col] in a third output (the key of the next join).
#include "internal.h"

namespace tcu {
namespace {

constexpr int kThreads = 256;
constexpr int kPerThread = 16;
constexpr int kChunk = kThreads * kPerThread;  // cells per workgroup
constexpr int kWords = kChunk / 64;

// Row and column of flat cell index i, cols >= 1: the quotient from a
// multiply by the reciprocal, then corrected by one either way.  i < 2^43
// (the launch covers at most 2^31 chunks of 4096 cells), so i is exact in a
// double and the product is within 2^-8 of i / cols.
__device__ inline void row_col(int64_t i, int64_t cols, double inv_cols, int64_t &r, int64_t &c) {
    r = (int64_t)((double)i * inv_cols);
    c = i - r * cols;
    if (c < 0) { --r; c += cols; }
    if (c >= cols) { ++r; c -= cols; }
}

// The kPerThread cells of this thread, read before any is used: cell j is
// b * kChunk + j * kThreads + t.  Every lane loads (cell 0 stands in past the
// end, total > 0), so the loads are in flight together; contiguous matrices
// (ld == cols, a uniform branch) need no row/column split.  The cells are read
// once, past the caches: 8192 x 8192 of them 139 us per call, 128 so.
__device__ inline void load_cells(const double *__restrict__ M, int64_t total, int64_t cols,
                                  int64_t ld, double (&v)[kPerThread]) {
    const int64_t base = (int64_t)blockIdx.x * kChunk + threadIdx.x;
    if (ld == cols) {
#pragma unroll
        for (int j = 0; j < kPerThread; ++j) {
            const int64_t i = base + (int64_t)j * kThreads;
            const bool in = i < total;
            const double x = __builtin_nontemporal_load(M + (in ? i : 0));
            v[j] = in ? x : 0.0;
        }
    } else {
        const double inv = 1.0 / (double)cols;
#pragma unroll
        for (int j = 0; j < kPerThread; ++j) {
            const int64_t i = base + (int64_t)j * kThreads;
            const bool in = i < total;
            int64_t r, c;
            row_col(in ? i : 0, cols, inv, r, c);
            const double x = M[r * ld + c];
            v[j] = in ? x : 0.0;
        }
    }
}

// Pass 1: one bit per cell and the nonzeros per chunk (coalesced across the
// workgroup).  Word 4 j + w of a chunk holds the 64 cells that wave w reads in
// step j, so the words are in row-major order.
__global__ void __launch_bounds__(kThreads)
nz_bits_kernel(const double *__restrict__ M, int64_t total, int64_t cols, int64_t ld,
               unsigned long long *__restrict__ bits, unsigned *__restrict__ counts) {
    __shared__ unsigned wave_sum[kThreads / 64];
    double v[kPerThread];
    load_cells(M, total, cols, ld, v);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    unsigned c = 0;
    unsigned long long mine = 0;
#pragma unroll
    for (int j = 0; j < kPerThread; ++j) {
        const unsigned long long word = __ballot(v[j] != 0.0);  // cells past the end read as 0
        c += (unsigned)__popcll(word);
        if (lane == j) mine = word;
    }
    if (lane < kPerThread) bits[(size_t)blockIdx.x * kWords + lane * (kThreads / 64) + wave] = mine;
    if (lane == 0) wave_sum[wave] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned s = 0;
        for (int w = 0; w < kThreads / 64; ++w) s += wave_sum[w];
        counts[blockIdx.x] = s;
    }
}

// Exclusive prefix sum of n counts into offsets (int64), total into
// offsets[n]; one workgroup, kScanThreads * kScanPer counts per round (16384
// counts 7 us; with 256 per round and an LDS scan, 74 us).
constexpr int kScanThreads = 1024;
constexpr int kScanPer = 8;

__global__ void __launch_bounds__(kScanThreads)
nz_scan_kernel(const unsigned *__restrict__ counts, int64_t n,
               unsigned long long *__restrict__ offsets) {
    __shared__ unsigned wave_sum[2][kScanThreads / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    unsigned long long carry = 0;
    int buf = 0;
    for (int64_t t0 = 0; t0 < n; t0 += kScanThreads * kScanPer, buf ^= 1) {
        const int64_t i0 = t0 + (int64_t)threadIdx.x * kScanPer;
        // a round's counts sum to at most 2^13 * 2^12: 32 bits hold them
        unsigned v[kScanPer], mine = 0;
        const bool whole = i0 + kScanPer <= n;  // counts are 256-byte aligned
        if (whole) {
#pragma unroll
            for (int j = 0; j < kScanPer; j += 4) {
                const uint4 x = *reinterpret_cast<const uint4 *>(counts + i0 + j);
                v[j] = x.x; v[j + 1] = x.y; v[j + 2] = x.z; v[j + 3] = x.w;
            }
        } else {
#pragma unroll
            for (int j = 0; j < kScanPer; ++j) v[j] = i0 + j < n ? counts[i0 + j] : 0u;
        }
#pragma unroll
        for (int j = 0; j < kScanPer; ++j) mine += v[j];
        unsigned incl = mine;
        for (int d = 1; d < 64; d <<= 1) {
            const unsigned up = (unsigned)__shfl_up((int)incl, d);
            if (lane >= d) incl += up;
        }
        if (lane == 63) wave_sum[buf][wave] = incl;
        __syncthreads();  // the other buffer is rewritten only after the next one
        unsigned before = 0, all = 0;
        for (int w = 0; w < kScanThreads / 64; ++w) {
            const unsigned s = wave_sum[buf][w];
            before += w < wave ? s : 0u;
            all += s;
        }
        unsigned long long at = carry + before + (incl - mine);
        if (whole) {
#pragma unroll
            for (int j = 0; j < kScanPer; j += 2) {
                const unsigned long long next = at + v[j];
                *reinterpret_cast<ulonglong2 *>(offsets + i0 + j) = make_ulonglong2(at, next);
                at = next + v[j + 1];
            }
        } else {
#pragma unroll
            for (int j = 0; j < kScanPer; ++j) {
                if (i0 + j < n) offsets[i0 + j] = at;
                at += v[j];
            }
        }
        carry += all;
    }
    if (threadIdx.x == 0) offsets[n] = carry;
}

// Pass 3, one wave per chunk: lane l holds word l.  In a sparse chunk each
// lane writes the cells of its own word; in a dense one (more than a quarter
// of the cells) the wave takes the words one after the other, a lane per
// cell, so that the stores stay contiguous.
struct NzOut {
    int32_t *row, *col;
    const int32_t *map;
    int32_t *key;
    int64_t capacity;
};

__device__ inline void write_cell(const NzOut &o, int64_t p, int64_t cell, int64_t cols,
                                  double inv_cols) {
    if (p >= o.capacity) return;
    int64_t r, c;
    row_col(cell, cols, inv_cols, r, c);
    o.row[p] = (int32_t)r;
    o.col[p] = (int32_t)c;
    if (o.key != nullptr) o.key[p] = o.map[c];
}

__global__ void __launch_bounds__(kThreads)
nz_write_kernel(const unsigned long long *__restrict__ bits, int64_t chunks, int64_t cols,
                const unsigned long long *__restrict__ offsets, NzOut o) {
    const int64_t chunk = (int64_t)blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);
    if (chunk >= chunks) return;
    const int lane = threadIdx.x & 63;
    const int64_t pos = (int64_t)offsets[chunk];
    unsigned long long word = bits[(size_t)chunk * kWords + lane];
    const unsigned mine = (unsigned)__popcll(word);
    unsigned incl = mine;
    for (int d = 1; d < 64; d <<= 1) {
        const unsigned up = (unsigned)__shfl_up((int)incl, d);
        if (lane >= d) incl += up;
    }
    const unsigned all = (unsigned)__shfl((int)incl, 63);
    const double inv_cols = 1.0 / (double)cols;
    const int64_t cell0 = chunk * kChunk;
    if (all <= kChunk / 4) {
        int64_t p = pos + (incl - mine);
        while (word) {
            write_cell(o, p++, cell0 + lane * 64 + __builtin_ctzll(word), cols, inv_cols);
            word &= word - 1;
        }
        return;
    }
    const unsigned lo = (unsigned)word, hi = (unsigned)(word >> 32);
    int64_t p = pos;
    for (int w = 0; w < kWords; ++w) {
        const unsigned long long x = (unsigned)__builtin_amdgcn_readlane((int)lo, w) |
                                     (unsigned long long)(unsigned)__builtin_amdgcn_readlane(
                                         (int)hi, w) << 32;
        const unsigned below =
            __builtin_amdgcn_mbcnt_hi((unsigned)(x >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)x, 0u));
        if (x >> lane & 1ull) write_cell(o, p + below, cell0 + w * 64 + lane, cols, inv_cols);
        p += __popcll(x);
    }
}

inline size_t chunks_of(int64_t total) { return (size_t)((total + kChunk - 1) / kChunk); }

}  // namespace

size_t nonzero_workspace_bytes(int64_t rows, int64_t cols) {
    const size_t nb = chunks_of(rows * cols);
    // bits, counts, offsets
    return align_up(nb * kWords * 8) + align_up(nb * 4) + align_up((nb + 1) * 8);
}

hipError_t run_nonzero(const double *M, int64_t rows, int64_t cols, int64_t ld, int32_t *out_row,
                       int32_t *out_col, const int32_t *col_map, int32_t *out_key,
                       int64_t capacity, int64_t *count, void *ws, hipStream_t s) {
    const int64_t total = rows * cols;
    const size_t nb = chunks_of(total);
    char *p = static_cast<char *>(ws);
    auto *bits = reinterpret_cast<unsigned long long *>(p);
    p += align_up(nb * kWords * 8);
    unsigned *counts = reinterpret_cast<unsigned *>(p);
    unsigned long long *offsets = reinterpret_cast<unsigned long long *>(p + align_up(nb * 4));
    if (nb > 0x7fffffffull) return hipErrorInvalidValue;
    if (nb > 0) {
        nz_bits_kernel<<<(unsigned)nb, kThreads, 0, s>>>(M, total, cols, ld, bits, counts);
        nz_scan_kernel<<<1, kScanThreads, 0, s>>>(counts, (int64_t)nb, offsets);
        nz_write_kernel<<<(unsigned)((nb + kThreads / 64 - 1) / (kThreads / 64)), kThreads, 0, s>>>(
            bits, (int64_t)nb, cols, offsets, NzOut{out_row, out_col, col_map, out_key, capacity});
    } else {
        // no cells: offsets[0] = 0
        hipError_t e = launch_zero_f64(reinterpret_cast<double *>(offsets), 1, s);
        if (e != hipSuccess) return e;
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    unsigned long long host = 0;
    e = hipMemcpyAsync(&host, offsets + nb, sizeof(host), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return e;
    *count = (int64_t)host;
    return hipSuccess;
}

}  // namespace tcu
