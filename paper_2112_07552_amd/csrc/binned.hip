// binned.hip -- encodings of relations with repeated (group, key) cells
// (Sections 3.1 and 3.3 of TCUDB): the records are sorted into tiles of the
// matrix first, and each tile is then summed in LDS and written once.
//
// Placing such records one by one takes a device-scope FP64 atomic per record
// at a random address, 23 G records/s (2 M records 87 us, and again for the
// pair counts' multiplicities), after a pass that zeroes the matrix.  Here,
// for both relations of a join in the same launches:
//   1. the records per tile are counted (LDS histograms, one global atomic
//      per workgroup and tile);
//   2. one workgroup turns the counts into offsets;
//   3. each workgroup stages 8192 records in LDS in tile order and writes them
//      to the tiles' places in runs: 2 bytes of cell, 8 of value;
//   4. one workgroup per tile adds its records up in LDS and writes the tile's
//      cells, zeros included, and, for the pair counts, the multiplicities as
//      int8 in the layout the count product reads.
// Every record is read twice and its 10 staged bytes are written and read
// once; no pass zeroes the matrices.  SUM and COUNT of 2 M records each, 1500 x
// 2051 x 2777 cells: 996 us record by record, 442 through tiles.
//
// One workgroup sums a tile however many records it has, which bounds small
// domains and skewed keys; the atomics that it replaces meet on the same few
// addresses there and take longer still.  The whole forward, 2^24 records each, us
// record by record and through tiles: 16^3 cells 12620 and 8299, 128^3 1767 and
// 454, 1000^3 with all records in 1/50 of the groups and keys 12342 and 8354, in
// one cell 402800 and 21970; 2^19 records in 1/50 556 and 235.  The histogram over
// 10^5 keys, 2^24 records on 100 of them 13226 and 6550, on one 202257 and 34987.
#include <algorithm>

#include "internal.h"

namespace tcu {
namespace {

constexpr int kThreads = 1024;
constexpr int kPer = 8;
constexpr int kChunk = kThreads * kPer;  // records per workgroup of the partition
constexpr int kHistChunk = 2 * kChunk;   // and of the count
constexpr int kMaxTiles = 4096;          // tiles per relation (LDS histograms)
constexpr int kMaxCells = 8192;          // cells per tile

// One relation and its matrix (A: rows = groups, columns = keys; B: rows =
// keys, columns = groups), cut into tiles of 2^lr x 2^lc cells, `across` of
// them side by side.
struct Side {
    int64_t n;
    const int32_t *row, *col;  // row NULL: one row, number 0
    const void *val;
    int f32;
    int rows, cols;
    int lr, lc, across, tiles, first;  // first: number of the first tile
    double *out;
    // the multiplicities' plane (NULL: none): line = row (A) or column (B)
    int8_t *plane;
    int lines_are_cols, lines_pad, len_pad;
};

struct Both {
    Side a, b;
};

// The side a block of a launch over `per`-record chunks of both relations works on.
__device__ inline const Side &side_of(const Both &p, int64_t per, int &chunk) {
    const int na = (int)((p.a.n + per - 1) / per);
    const bool of_a = (int)blockIdx.x < na;
    chunk = of_a ? (int)blockIdx.x : (int)blockIdx.x - na;
    return of_a ? p.a : p.b;
}

__device__ inline bool tile_of(const Side &s, int64_t i, int &tile, unsigned &cell) {
    const int r = s.row != nullptr ? s.row[i] : 0, c = s.col[i];
    if ((unsigned)r >= (unsigned)s.rows || (unsigned)c >= (unsigned)s.cols) return false;
    tile = (r >> s.lr) * s.across + (c >> s.lc);
    cell = ((unsigned)(r & ((1 << s.lr) - 1)) << s.lc) | (unsigned)(c & ((1 << s.lc) - 1));
    return true;
}

// Step 1.  totals zeroed beforehand; records outside the shape are counted as
// skipped here, once.
__global__ void __launch_bounds__(kThreads)
bin_count_kernel(Both p, uint32_t *__restrict__ totals, StatusBlock *st) {
    __shared__ unsigned int hist[kMaxTiles];
    int chunk;
    const Side &s = side_of(p, kHistChunk, chunk);
    for (int b = threadIdx.x; b < s.tiles; b += kThreads) hist[b] = 0u;
    __syncthreads();
    unsigned bad = 0;
#pragma unroll
    for (int j = 0; j < kHistChunk / kThreads; ++j) {
        const int64_t i = (int64_t)chunk * kHistChunk + j * kThreads + threadIdx.x;
        if (i >= s.n) continue;
        int tile;
        unsigned cell;
        if (tile_of(s, i, tile, cell)) atomicAdd(&hist[tile], 1u);
        else ++bad;
    }
    if (bad != 0u) {
        atomicOr(&st->flags, kFlagKeyRange);
        atomicAdd(s.first == 0 ? &st->skipped_a : &st->skipped_b, (unsigned long long)bad);
    }
    __syncthreads();
    for (int b = threadIdx.x; b < s.tiles; b += kThreads)
        if (hist[b] != 0u) atomicAdd(&totals[s.first + b], hist[b]);
}

// v[0 .. n) (n <= 8 kThreads) becomes its exclusive prefix sums; returns the
// total.  `tmp`: one word per wave.
__device__ inline unsigned lds_exclusive(unsigned *v, int n, unsigned *tmp) {
    constexpr int per = 8;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    unsigned x[per], sum = 0;
#pragma unroll
    for (int j = 0; j < per; ++j) {
        const int i = (int)threadIdx.x * per + j;
        x[j] = i < n ? v[i] : 0u;
        sum += x[j];
    }
    unsigned incl = sum;
    for (int d = 1; d < 64; d <<= 1) {
        const unsigned up = (unsigned)__shfl_up((int)incl, d);
        if (lane >= d) incl += up;
    }
    if (lane == 63) tmp[wave] = incl;
    __syncthreads();
    unsigned before = 0, all = 0;
    for (int w = 0; w < kThreads / 64; ++w) {
        if (w < wave) before += tmp[w];
        all += tmp[w];
    }
    unsigned at = before + incl - sum;
#pragma unroll
    for (int j = 0; j < per; ++j) {
        const int i = (int)threadIdx.x * per + j;
        if (i < n) v[i] = at;
        at += x[j];
    }
    __syncthreads();
    return all;
}

// Step 2: offsets[t] = records of the tiles before t, offsets[tiles] = all;
// cursor starts as a copy.
__global__ void __launch_bounds__(kThreads)
bin_offsets_kernel(const uint32_t *__restrict__ totals, uint32_t *__restrict__ offsets,
                   uint32_t *__restrict__ cursor, int tiles) {
    static_assert(2 * kMaxTiles <= 8 * kThreads, "one scan covers both relations' tiles");
    __shared__ unsigned v[2 * kMaxTiles];
    __shared__ unsigned tmp[kThreads / 64];
    for (int t = threadIdx.x; t < tiles; t += kThreads) v[t] = totals[t];
    __syncthreads();
    const unsigned all = lds_exclusive(v, tiles, tmp);
    for (int t = threadIdx.x; t < tiles; t += kThreads) offsets[t] = cursor[t] = v[t];
    if (threadIdx.x == 0) offsets[tiles] = all;
}

// Step 3.
__global__ void __launch_bounds__(kThreads)
bin_partition_kernel(Both p, uint32_t *__restrict__ cursor, uint16_t *__restrict__ out_cell,
                     double *__restrict__ out_val) {
    __shared__ unsigned int cnt[kMaxTiles], first[kMaxTiles], tmp[kThreads / 64];
    __shared__ double s_val[kChunk];
    __shared__ uint16_t s_cell[kChunk], s_tile[kChunk];
    int chunk;
    const Side &s = side_of(p, kChunk, chunk);
    const int t = threadIdx.x;
    for (int b = t; b < s.tiles; b += kThreads) cnt[b] = 0u;
    __syncthreads();
    int tile[kPer];
    unsigned cell[kPer], rank[kPer];
    double v[kPer];
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const int64_t i = (int64_t)chunk * kChunk + j * kThreads + t;
        tile[j] = -1;
        cell[j] = rank[j] = 0u;
        v[j] = 1.0;
        int b;
        if (i < s.n && tile_of(s, i, b, cell[j])) {
            tile[j] = b;
            if (s.val != nullptr)
                v[j] = s.f32 ? (double)static_cast<const float *>(s.val)[i]
                             : static_cast<const double *>(s.val)[i];
            rank[j] = atomicAdd(&cnt[b], 1u);
        }
    }
    __syncthreads();
    for (int b = t; b < s.tiles; b += kThreads) first[b] = cnt[b];
    __syncthreads();
    const unsigned total = lds_exclusive(first, s.tiles, tmp);
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        if (tile[j] < 0) continue;
        const unsigned q = first[tile[j]] + rank[j];
        s_val[q] = v[j];
        s_cell[q] = (uint16_t)cell[j];
        s_tile[q] = (uint16_t)tile[j];
    }
    // cnt[b] becomes the place of the run's first record, less its place here
    for (int b = t; b < s.tiles; b += kThreads)
        if (cnt[b] != 0u) cnt[b] = atomicAdd(&cursor[s.first + b], cnt[b]) - first[b];
    __syncthreads();
    for (unsigned q = t; q < total; q += kThreads) {
        const unsigned at = cnt[s_tile[q]] + q;
        out_cell[at] = s_cell[q];
        out_val[at] = s_val[q];
    }
}

// What step 4 leaves: the sums; the sums and the multiplicities' planes; or
// the multiplicities as doubles.
constexpr int kSums = 0, kSumsAndPlanes = 1, kMultiplicities = 2;

// Step 4.  A multiplicity beyond int8 raises st->wide_counts.  only_if: leave
// at once unless *only_if is set (NULL: run).
template <int MODE>
__global__ void __launch_bounds__(kThreads)
bin_fill_kernel(Both p, const uint32_t *__restrict__ offsets, const uint16_t *__restrict__ cell,
                const double *__restrict__ val, StatusBlock *st, const uint32_t *only_if) {
    constexpr bool kPlanes = MODE == kSumsAndPlanes;
    __shared__ double v[kMaxCells];
    // a gap after every 16 words spreads the plane's 16-cell groups over the banks
    __shared__ unsigned c[kPlanes ? kMaxCells / 16 * 17 : 1];
    if (only_if != nullptr && *only_if == 0u) return;
    const Side &s = (int)blockIdx.x < p.b.first ? p.a : p.b;
    const int tile = (int)blockIdx.x - s.first, t = threadIdx.x;
    const int cells = 1 << (s.lr + s.lc), cmask = (1 << s.lc) - 1;
    const int r0 = (tile / s.across) << s.lr, c0 = (tile % s.across) << s.lc;
    for (int i = t; i < cells; i += kThreads) {
        v[i] = 0.0;
        if (kPlanes) c[i + (i >> 4)] = 0u;
    }
    __syncthreads();
    const uint32_t lo = offsets[blockIdx.x], hi = offsets[blockIdx.x + 1];
    for (uint32_t q = lo + t; q < hi; q += kThreads) {
        const unsigned i = cell[q];
        atomicAdd(&v[i], MODE == kMultiplicities ? 1.0 : val[q]);
        if (kPlanes) atomicAdd(&c[i + (i >> 4)], 1u);
    }
    __syncthreads();
    for (int i = t; i < cells; i += kThreads) {
        const int r = r0 + (i >> s.lc), col = c0 + (i & cmask);
        if (r < s.rows && col < s.cols) s.out[(int64_t)r * s.cols + col] = v[i];
    }
    if (kPlanes) {
        // 16 cells along the contraction of one line per thread and step
        bool wide = false;
        const int lines = s.lines_are_cols ? 1 << s.lc : 1 << s.lr;
        const int groups = cells / lines / 16;
        for (int u = t; u < lines * groups; u += kThreads) {
            const int line = s.lines_are_cols ? u % lines : u / groups;
            const int g = s.lines_are_cols ? u / lines : u % groups;
            uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int i = s.lines_are_cols ? ((g * 16 + e) << s.lc) | line
                                               : (line << s.lc) | (g * 16 + e);
                const unsigned m = c[i + (i >> 4)];
                wide |= m > 127u;
                w[e >> 2] |= min(m, 127u) << (8 * (e & 3));
            }
            const int L = (s.lines_are_cols ? c0 : r0) + line;
            const int T = (s.lines_are_cols ? r0 : c0) + g * 16;
            if (L < s.lines_pad && T < s.len_pad)
                *reinterpret_cast<uint4 *>(s.plane + ((int64_t)(T >> 4) * s.lines_pad + L) * 16) =
                    make_uint4(w[0], w[1], w[2], w[3]);
        }
        if (__ballot(wide) != 0ull && (t & 63) == 0) atomicOr(&st->wide_counts, 1u);
    }
}

// Step 4 of a histogram over keys (one row of cells): sums and numbers of
// records.
__global__ void __launch_bounds__(kThreads)
bin_hist_kernel(Side s, const uint32_t *__restrict__ offsets, const uint16_t *__restrict__ cell,
                const double *__restrict__ val, unsigned long long *__restrict__ counts) {
    __shared__ double v[kMaxCells];
    __shared__ unsigned c[kMaxCells];
    const int cells = 1 << s.lc, t = threadIdx.x;
    const int64_t c0 = (int64_t)blockIdx.x << s.lc;
    for (int i = t; i < cells; i += kThreads) {
        v[i] = 0.0;
        c[i] = 0u;
    }
    __syncthreads();
    const uint32_t lo = offsets[blockIdx.x], hi = offsets[blockIdx.x + 1];
    for (uint32_t q = lo + t; q < hi; q += kThreads) {
        const unsigned i = cell[q];
        atomicAdd(&v[i], val[q]);
        atomicAdd(&c[i], 1u);
    }
    __syncthreads();
    for (int i = t; i < cells; i += kThreads)
        if (c0 + i < s.cols) {
            s.out[c0 + i] = v[i];
            counts[c0 + i] = c[i];
        }
}

struct TilePlan {
    int lr = 5, lc = 8, across = 0, tiles = 0;
};

// Tiles of 32 x 256 cells (rows of 2 KB), smaller ones for small matrices so
// that a few hundred workgroups share the records; never below 16 x 16, the
// planes' groups.  tiles = 0: more than kMaxTiles.
TilePlan tile_plan(int64_t rows, int64_t cols) {
    TilePlan p;
    for (;;) {
        const int64_t down = (rows + (1 << p.lr) - 1) >> p.lr;
        const int64_t across = (cols + (1 << p.lc) - 1) >> p.lc;
        if (down * across > kMaxTiles) return TilePlan{};
        p.across = (int)across;
        p.tiles = (int)(down * across);
        if (p.tiles >= 512 || (p.lr == 4 && p.lc == 4)) return p;
        TilePlan q = p;
        if (q.lc > 4) --q.lc;
        else --q.lr;
        const int64_t d2 = (rows + (1 << q.lr) - 1) >> q.lr;
        const int64_t a2 = (cols + (1 << q.lc) - 1) >> q.lc;
        if (d2 * a2 > kMaxTiles) return p;
        p.lr = q.lr;
        p.lc = q.lc;
    }
}

// Records of both relations from which the tiles pay, as they take four
// launches more (us of the whole forward, record by record and through tiles;
// n records per relation): sums alone, 500^3: n = 2^17 33 and 41, 2^18 45 and
// 47, 2^19 66 and 48; 1500 x 2051 x 2777: 2^18 352 and 349, 2^21 506 and 378.
// With pair counts: 500^3: 2^17 64 and 66, 2^18 86 and 71; and for products
// of kCountWork and more at any length, since the counts then leave the FP64
// matrix cores: 4000^3, n = 2^15: 3862 and 2139.
constexpr int64_t kMinRecords = (int64_t)1 << 19, kMinRecordsCount = (int64_t)1 << 18;
constexpr double kCountWork = 0x1p30;
// contraction length up to which int32 sums of 127 * 127 stay exact
constexpr int kMaxCountKeys = 131072;

// The matrices' extents in tiles: with planes, padded as they are.
struct Plan {
    TilePlan a, b;
    int alp = 0, blp = 0, len = 0;  // planes: padded lines and length (0: none)
    size_t qa = 0, qb = 0;
};

bool make_plan(const tcu_relation &A, const tcu_relation &B, int M, int K, int N, bool planes,
               Plan *p) {
    if ((A.flags | B.flags) & TCU_REL_UNIQUE_CELLS) return false;
    const int64_t n = A.n + B.n;
    if (A.n < 1 || B.n < 1 || n > 0x7fffffffLL) return false;
    if (n < (planes ? kMinRecordsCount : kMinRecords) &&
        !(planes && (double)M * K * N >= kCountWork))
        return false;
    if (M > (1 << 30) || K > (1 << 30) || N > (1 << 30)) return false;
    if (planes) {
        if (K > kMaxCountKeys) return false;
        p->alp = (int)count_lines_pad(M);
        p->blp = (int)count_lines_pad(N);
        p->len = (K + 31) / 32 * 32;
        p->qa = count_plane_bytes(M, K);
        p->qb = count_plane_bytes(N, K);
    }
    p->a = tile_plan(planes ? p->alp : M, planes ? p->len : K);
    p->b = tile_plan(planes ? p->len : K, planes ? p->blp : N);
    return p->a.tiles > 0 && p->b.tiles > 0;
}

// Scratch: totals, cursors and offsets (u32 per tile), the planes, then per
// record a cell (u16) and a value.
struct Scratch {
    size_t totals = 0, cursor = 0, offsets = 0, qa = 0, qb = 0, cell = 0, val = 0, bytes = 0;
};

Scratch scratch_layout(const Plan &p, int64_t n) {
    Scratch w;
    const size_t table = align_up((size_t)(p.a.tiles + p.b.tiles + 1) * 4);
    size_t off = 0;
    w.totals = off; off += table;
    w.cursor = off; off += table;
    w.offsets = off; off += table;
    w.qa = off; off += align_up(p.qa);
    w.qb = off; off += align_up(p.qb);
    w.cell = off; off += align_up((size_t)n * 2);
    w.val = off; off += align_up((size_t)n * 8);
    w.bytes = off;
    return w;
}

// Tiles of one row of K cells: at least 512 of them where K has 16 times that.
TilePlan hist_plan(int K) {
    TilePlan p;
    p.lr = 0;
    p.lc = 4;
    while ((1 << p.lc) < kMaxCells && ((int64_t)K >> p.lc) >= 1024) ++p.lc;
    const int64_t across = ((int64_t)K + (1 << p.lc) - 1) >> p.lc;
    if (across > kMaxTiles) return TilePlan{};
    p.across = p.tiles = (int)across;
    return p;
}

// Records from which the histogram's tiles pay (us of the whole of Q3 with as
// many records on both sides, 500 groups, 3000 and 400000 keys; two global
// atomics per record against these launches): 2^18 46 and 55 against 35 and 56,
// 2^19 75 and 80 against 38 and 59, 2^24 1910 and 1679 against 333 and 479.
constexpr int64_t kMinHistRecords = (int64_t)1 << 18;

Side make_side(const tcu_relation &R, bool is_b, const TilePlan &t, int rows, int cols, int first,
               double *out, int8_t *plane, int lines_pad, int len_pad) {
    return Side{R.n, is_b ? R.key : R.group, is_b ? R.group : R.key, R.val, R.dtype == TCU_F32,
                rows, cols, t.lr, t.lc, t.across, t.tiles, first, out, plane, is_b, lines_pad,
                len_pad};
}

// Steps 1-3.
hipError_t partition(const Both &both, int tiles, const Scratch &w, char *base, StatusBlock *st,
                     hipStream_t s) {
    auto *totals = reinterpret_cast<uint32_t *>(base + w.totals);
    auto *cursor = reinterpret_cast<uint32_t *>(base + w.cursor);
    auto chunks = [&](int64_t per) {
        return (unsigned)((both.a.n + per - 1) / per + (both.b.n + per - 1) / per);
    };
    const hipError_t e = launch_zero_f64(reinterpret_cast<double *>(totals),
                                         align_up((size_t)(tiles + 1) * 4) / 8, s);
    if (e != hipSuccess) return e;
    bin_count_kernel<<<chunks(kHistChunk), kThreads, 0, s>>>(both, totals, st);
    bin_offsets_kernel<<<1, kThreads, 0, s>>>(
        totals, reinterpret_cast<uint32_t *>(base + w.offsets), cursor, tiles);
    bin_partition_kernel<<<chunks(kChunk), kThreads, 0, s>>>(
        both, cursor, reinterpret_cast<uint16_t *>(base + w.cell),
        reinterpret_cast<double *>(base + w.val));
    return hipGetLastError();
}

}  // namespace

size_t binned_hist_scratch_bytes(const tcu_relation &A, int K) {
    Plan p;
    if (A.n < kMinHistRecords || A.n > 0x7fffffffLL) return 0;
    p.a = hist_plan(K);
    return p.a.tiles > 0 ? scratch_layout(p, A.n).bytes : 0;
}

hipError_t launch_binned_hist(const tcu_relation &A, int K, double *h, unsigned long long *hc,
                              StatusBlock *st, void *scratch, hipStream_t s) {
    Plan p;
    p.a = hist_plan(K);
    if (p.a.tiles == 0 || A.n < 1) return hipErrorInvalidValue;
    const Scratch w = scratch_layout(p, A.n);
    char *base = static_cast<char *>(scratch);
    Both both{};
    both.a = Side{A.n, nullptr, A.key, A.val, A.dtype == TCU_F32, 1, K, p.a.lr, p.a.lc,
                  p.a.across, p.a.tiles, 0, h, nullptr, 0, 0, 0};
    const hipError_t e = partition(both, p.a.tiles, w, base, st, s);
    if (e != hipSuccess) return e;
    bin_hist_kernel<<<(unsigned)p.a.tiles, kThreads, 0, s>>>(
        both.a, reinterpret_cast<uint32_t *>(base + w.offsets),
        reinterpret_cast<uint16_t *>(base + w.cell), reinterpret_cast<double *>(base + w.val), hc);
    return hipGetLastError();
}

size_t binned_scratch_bytes(const tcu_relation &A, const tcu_relation &B, int M, int K, int N,
                            bool planes) {
    Plan p;
    return make_plan(A, B, M, K, N, planes, &p) ? scratch_layout(p, A.n + B.n).bytes : 0;
}

hipError_t launch_binned(const tcu_relation &A, const tcu_relation &B, int M, int K, int N,
                         double *X, double *Y, int32_t *count, double *C, StatusBlock *st,
                         void *scratch, hipStream_t s) {
    const bool planes = count != nullptr;
    Plan p;
    if (!make_plan(A, B, M, K, N, planes, &p)) return hipErrorInvalidValue;
    const Scratch w = scratch_layout(p, A.n + B.n);
    char *base = static_cast<char *>(scratch);
    auto *offsets = reinterpret_cast<uint32_t *>(base + w.offsets);
    auto *qa = reinterpret_cast<int8_t *>(base + w.qa), *qb = reinterpret_cast<int8_t *>(base + w.qb);
    auto *cell = reinterpret_cast<uint16_t *>(base + w.cell);
    auto *val = reinterpret_cast<double *>(base + w.val);
    Both both{make_side(A, false, p.a, M, K, 0, X, planes ? qa : nullptr, p.alp, p.len),
              make_side(B, true, p.b, K, N, p.a.tiles, Y, planes ? qb : nullptr, p.blp, p.len)};
    const int tiles = p.a.tiles + p.b.tiles;
    hipError_t e = partition(both, tiles, w, base, st, s);
    if (e != hipSuccess) return e;
    if (!planes) {
        bin_fill_kernel<kSums><<<(unsigned)tiles, kThreads, 0, s>>>(both, offsets, cell, val, st,
                                                                    nullptr);
        return hipGetLastError();
    }
    bin_fill_kernel<kSumsAndPlanes><<<(unsigned)tiles, kThreads, 0, s>>>(both, offsets, cell, val,
                                                                         st, nullptr);
    e = hipGetLastError();
    // exact counts: the int8 product of the multiplicities
    if (e == hipSuccess) e = launch_count_planes_product(M, K, N, qa, qb, nullptr, count, s);
    if (e != hipSuccess) return e;
    // multiplicities beyond int8 (known on the device only: these launches
    // leave at once otherwise, 9 us): the counts again, from FP64 encodings of
    // the multiplicities multiplied in FP64 (every partial sum is an integer no
    // larger than the count, so a count below 2^53 is exact), C as scratch;
    // counts beyond int32 are saturated and flagged; then the sums once more
    const uint32_t *wide = &st->wide_counts;
    bin_fill_kernel<kMultiplicities><<<(unsigned)tiles, kThreads, 0, s>>>(both, offsets, cell, val,
                                                                          st, wide);
    e = hipGetLastError();
    if (e == hipSuccess) e = launch_gemm_f64(0, 0, M, N, K, X, K, Y, N, C, N, s, 0, wide);
    if (e == hipSuccess) e = launch_f64_to_i32(C, count, (size_t)M * N, st, s, wide);
    if (e != hipSuccess) return e;
    bin_fill_kernel<kSums><<<(unsigned)tiles, kThreads, 0, s>>>(both, offsets, cell, val, st, wide);
    return hipGetLastError();
}

}  // namespace tcu
