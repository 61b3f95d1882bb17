// bsr.hip -- the join-aggregate on block-sparse encodings: the analogue of
// TCUDB's TCU-SpMM operator (Section 4.2.4, handling sparse matrices).
//
// When the key domain K is large and each group touches few keys (the
// microbenchmarks' many-distinct-values regime, Section 5.2), X (M x K) and
// Y (K x N) are almost all zeros and the dense product wastes its work on
// them.  Following the paper, both encodings are cut into 16 x 16 tiles, the
// tiles holding no record are never stored or multiplied, and the remaining
// tile pairs run on the matrix cores:
//
//   1. a bit per tile of X and Y, set for every record (rows of bits: tile
//      rows of X, tile columns of Y; bit: key tile), and counted per row;
//   2. one workgroup scans the rows' counts: the first tile of every row;
//   3. per row, the tiles' key tiles in ascending order, the index of every
//      64-bit word's first tile, and the tiles zeroed;
//   4. every record's value added into its tile (16 x 16 FP64, X tiles
//      [g%16][k%16], Y tiles [k%16][h%16]), whose index is its word's plus the
//      bits below its own;
//   5. per tile row of C and chunk of column tiles: the tiles whose lists
//      share no key tile are zeroed, the others take, for every common key
//      tile, four v_mfma_f64_16x16x4_f64 into their accumulator (see below).
// The result equals the dense operator's: the products skipped are products
// of all-zero tiles.  C is dense M x N FP64, as for tcu_join_agg_fwd.
//
// No step needs the host.  Where the bits would take more memory than the
// dictionary machinery (kMaxBitBytes), steps 1-3 take the distinct tile keys
// (outer << 32 | key tile) and their ranks from that, one to three host waits per
// side.
#include <algorithm>

#include "internal.h"

namespace tcu {
namespace {

typedef double d4 __attribute__((ext_vector_type(4)));

constexpr int kThreads = 256;
constexpr int TB = 16;                           // tile edge
constexpr long long kBadKey = 0x7fffffffffffffffll;  // record outside the shape

// ---------------------------------------------------------- tiles by bits
// One relation: A (outer = group of A, X) or B (outer = group of B, Y).
struct BitSide {
    int64_t n;
    const int32_t *outer, *key;
    const void *val;
    int f32, unique, key_rows, outer_ext, rows;  // rows: outer tiles
    unsigned long long *bits;  // rows x words
    unsigned *word_first;      // rows x words: index of the word's first tile
    int *ptr;                  // rows + 1
    long long *tkeys;
    double *tiles;
    unsigned *mask;  // per tile: the keys (mod 16) that have a record; NULL: not wanted
};

struct BitPair {
    BitSide a, b;
    int words, key_ext;
};

// The side of a launch whose workgroups [0, blocks_a) work on A; `block`
// becomes the block's number within its side.
__device__ inline const BitSide &bit_side(const BitPair &p, unsigned blocks_a, unsigned &block) {
    const bool of_a = blockIdx.x < blocks_a;
    block = of_a ? blockIdx.x : blockIdx.x - blocks_a;
    return of_a ? p.a : p.b;
}

// Step 1.  Records outside the shape are skipped and counted here.
__global__ void __launch_bounds__(kThreads)
tile_bits_kernel(BitPair p, unsigned blocks_a, StatusBlock *st) {
    unsigned block;
    const BitSide &s = bit_side(p, blocks_a, block);
    const int64_t i = (int64_t)block * kThreads + threadIdx.x;
    bool bad = false;
    if (i < s.n) {
        const int o = s.outer[i], k = s.key[i];
        bad = (unsigned)o >= (unsigned)s.outer_ext || (unsigned)k >= (unsigned)p.key_ext;
        if (!bad) {
            const int kt = k / TB;
            unsigned long long *w = s.bits + (int64_t)(o / TB) * p.words + (kt >> 6);
            const unsigned long long bit = 1ull << (kt & 63);
            // a bit already set costs no atomic (one set by another XCD may
            // still read as clear: one atomic too many)
            if (!(__hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) & bit))
                atomicOr(w, bit);
        }
    }
    const unsigned long long mask = __ballot(bad);
    if (mask != 0ull && (threadIdx.x & 63) == 0) {
        atomicOr(&st->flags, kFlagKeyRange);
        atomicAdd(s.key_rows ? &st->skipped_b : &st->skipped_a,
                  (unsigned long long)__popcll(mask));
    }
}

// Each row's number of tiles, into ptr[row + 1]: one wave per row.
__global__ void __launch_bounds__(kThreads)
tile_count_kernel(BitPair p, unsigned blocks_a) {
    unsigned block;
    const BitSide &s = bit_side(p, blocks_a, block);
    const int row = (int)block * (kThreads / 64) + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (row >= s.rows) return;
    int c = 0;
    for (int w = lane; w < p.words; w += 64) c += __popcll(s.bits[(int64_t)row * p.words + w]);
    for (int d = 32; d > 0; d >>= 1) c += __shfl_xor(c, d);
    if (lane == 0) s.ptr[row + 1] = c;
}

// Step 2: ptr[1 ..] from counts to their inclusive sums, ptr[0] = 0; one
// workgroup per side.
constexpr int kScanThreads = 1024;
__global__ void __launch_bounds__(kScanThreads)
tile_scan_kernel(BitPair p) {
    __shared__ int wave_sum[kScanThreads / 64];
    const BitSide &s = blockIdx.x == 0 ? p.a : p.b;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int before = 0;
    if (threadIdx.x == 0) s.ptr[0] = 0;
    for (int r0 = 0; r0 < s.rows; r0 += kScanThreads) {
        const int r = r0 + (int)threadIdx.x;
        int c = r < s.rows ? s.ptr[r + 1] : 0;
        for (int d = 1; d < 64; d <<= 1) {
            const int up = __shfl_up(c, d);
            if (lane >= d) c += up;
        }
        if (lane == 63) wave_sum[wave] = c;
        __syncthreads();
        int base = before;
        for (int w = 0; w < kScanThreads / 64; ++w) {
            if (w < wave) base += wave_sum[w];
            before += wave_sum[w];
        }
        if (r < s.rows) s.ptr[r + 1] = base + c;
        __syncthreads();
    }
}

// Step 3: one wave per row.
__global__ void __launch_bounds__(kThreads)
tile_list_kernel(BitPair p, unsigned blocks_a) {
    unsigned block;
    const BitSide &s = bit_side(p, blocks_a, block);
    const int row = (int)block * (kThreads / 64) + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (row >= s.rows) return;
    const int first = s.ptr[row], end = s.ptr[row + 1];
    int at = first;
    for (int w0 = 0; w0 < p.words; w0 += 64) {
        const int w = w0 + lane;
        unsigned long long bits = w < p.words ? s.bits[(int64_t)row * p.words + w] : 0ull;
        const int c = __popcll(bits);
        int incl = c;
        for (int d = 1; d < 64; d <<= 1) {
            const int up = __shfl_up(incl, d);
            if (lane >= d) incl += up;
        }
        int q = at + incl - c;
        if (w < p.words) s.word_first[(int64_t)row * p.words + w] = (unsigned)q;
        for (; bits; bits &= bits - 1)
            s.tkeys[q++] = ((long long)row << 32) | (long long)(w * 64 + __builtin_ctzll(bits));
        at += __shfl(incl, 63);
    }
    if (s.mask != nullptr)
        for (int i = first + lane; i < end; i += 64) s.mask[i] = 0u;
    double2 *z = reinterpret_cast<double2 *>(s.tiles + (int64_t)first * (TB * TB));
    const int64_t nz = (int64_t)(end - first) * (TB * TB / 2);
    for (int64_t i = lane; i < nz; i += 64) z[i] = make_double2(0.0, 0.0);
}

// Step 4.
__global__ void __launch_bounds__(kThreads)
tile_place_kernel(BitPair p, unsigned blocks_a) {
    unsigned block;
    const BitSide &s = bit_side(p, blocks_a, block);
    const int64_t i = (int64_t)block * kThreads + threadIdx.x;
    if (i >= s.n) return;
    const int o = s.outer[i], k = s.key[i];
    if ((unsigned)o >= (unsigned)s.outer_ext || (unsigned)k >= (unsigned)p.key_ext) return;
    const int kt = k / TB;
    const int64_t w = (int64_t)(o / TB) * p.words + (kt >> 6);
    const int64_t tile =
        (int64_t)s.word_first[w] + __popcll(s.bits[w] & ((1ull << (kt & 63)) - 1ull));
    double v = 1.0;
    if (s.val != nullptr)
        v = s.f32 ? (double)static_cast<const float *>(s.val)[i]
                  : static_cast<const double *>(s.val)[i];
    double *dst = s.tiles + tile * (TB * TB) +
                  (s.key_rows ? (k % TB) * TB + o % TB : (o % TB) * TB + k % TB);
    if (s.unique) *dst = v;
    else unsafeAtomicAdd(dst, v);
    if (s.mask != nullptr) atomicOr(s.mask + tile, 1u << (k % TB));
}

// ---------------------------------------------------- tiles by dictionary
template <typename T>
__global__ void __launch_bounds__(kThreads)
tile_key_kernel(int64_t n, const int32_t *__restrict__ outer, const int32_t *__restrict__ key,
                int outer_ext, int key_ext, long long *__restrict__ keys, StatusBlock *st,
                int which) {
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    bool bad = false;
    if (i < n) {
        const int o = outer[i], k = key[i];
        bad = (unsigned)o >= (unsigned)outer_ext || (unsigned)k >= (unsigned)key_ext;
        keys[i] = bad ? kBadKey : ((long long)(o / TB) << 32) | (long long)(k / TB);
    }
    const unsigned long long mask = __ballot(bad);
    if (mask != 0ull && (threadIdx.x & 63) == 0) {
        atomicOr(&st->flags, kFlagKeyRange);
        atomicAdd(which == 0 ? &st->skipped_a : &st->skipped_b,
                  (unsigned long long)__popcll(mask));
    }
}

// ptr[o] = index of the first sorted tile key whose outer tile is >= o.
__global__ void __launch_bounds__(kThreads)
tile_ptr_kernel(const long long *__restrict__ tkeys, int64_t ntiles, int outer_tiles,
                int *__restrict__ ptr) {
    const int o = blockIdx.x * kThreads + threadIdx.x;
    if (o > outer_tiles) return;
    const long long target = (long long)o << 32;
    int64_t lo = 0, hi = ntiles;
    while (lo < hi) {
        const int64_t mid = (lo + hi) / 2;
        if (tkeys[mid] < target) lo = mid + 1;
        else hi = mid;
    }
    ptr[o] = (int)lo;
}

// tiles[code][r][c] (+)= v with (r, c) = (outer % 16, key % 16) for X, or
// (key % 16, outer % 16) for Y (key_rows).
template <typename T, bool UNIQUE>
__global__ void __launch_bounds__(kThreads)
tile_scatter_kernel(int64_t n, const int32_t *__restrict__ outer, const int32_t *__restrict__ key,
                    const T *__restrict__ val, const long long *__restrict__ keys,
                    const int *__restrict__ codes, int key_rows, double *__restrict__ tiles) {
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i >= n || keys[i] == kBadKey) return;
    const int o = outer[i] % TB, k = key[i] % TB;
    const int cell = key_rows ? k * TB + o : o * TB + k;
    const double v = val ? (double)val[i] : 1.0;
    double *dst = tiles + (int64_t)codes[i] * (TB * TB) + cell;
    if (UNIQUE) *dst = v;
    else unsafeAtomicAdd(dst, v);
}

// ------------------------------------------------------------ the product
// Most tiles of a sparse product are zero, and C's 8 bytes per cell bound it:
// what costs is finding out.  One wave per tile, walking both key lists one
// scalar load after the other, took 1555 us on 1024 x 1024 tiles of which
// 256 meet (2.1 GB of zeros, 1.4 TB/s).  Here a workgroup takes one tile row
// of C and kChunk column tiles:
//   1. the row's X keys go to LDS, as a list and as a bit per key modulo
//      8192, and eight threads test one column tile: a short list of Y against
//      the bits and, where one is set, by binary search of the list (a short
//      list of X against a long one of Y by searches in the latter; lists
//      that both exceed kTestKeys keys are taken to meet);
//   2. the tiles that do not meet are zeroed row by row, past the caches when
//      C exceeds the last-level one;
//   3. the others go to the waves, one tile each: the lanes take 64 keys of
//      the shorter list, search the longer, and the tile pairs that meet run
//      on the matrix cores in ascending key order (as the serial walk did, so
//      the sums round the same).
// For pair counts (no values on either side) two tiles also have to share a
// key, by a mask of 16 keys per tile, to meet: with one record per tile, one
// pair in 16 does.  (With values a zero of one tile may meet an infinity of
// the other, so every pair of tiles counts.)
// At 16384^2 cells the operator then takes 379-424 us with 1000 to 2^20 distinct
// keys (C alone: 377 at 5.7 TB/s; without the masks and with cached stores 1992
// with 1000, 473 with 2^20); 4096 x 4096 cells where nine tiles in ten meet 285
// us against 707 by serial walks, a graph's 65536 x 64 with long lists of Y
// 324 against 2751 (both the product alone).  The whole operator, with the tiles'
// lists and zeroing by one wave per tile row, against the start with dictionaries
// and walks: a graph of 65536 nodes and 2^20 edges by 64 features 3.1 ms and 5.9;
// one tile row of 62,500 tiles (16 groups, 10^6 keys) by 16 records 2.1 and 5.4.
// Column tiles per workgroup.  At 16384^2 cells (us of the operator for 4000 and
// 2^20 distinct keys, one thread per column tile): 32 tiles 407 and 414, 64 tiles
// 416 and 430, 256 tiles 445 and 450; with cached stores 578 and 420, 494 and
// 427, 519 and 441.
constexpr int kChunk = 32;
constexpr int kTesters = kThreads / kChunk;  // threads per column tile
constexpr size_t kLastLevelCache = (size_t)256 << 20;
constexpr int kPastCaches = 2;  // 16-byte stores past the caches (1: through them; 0: 8-byte)
typedef double d2 __attribute__((ext_vector_type(2)));
constexpr int kXKeys = 1024;     // X keys of one tile row held in LDS
constexpr int kTestKeys = 64;
constexpr int kBits = 8192;      // one bit per key modulo this: set for the row's X keys
static_assert(kThreads % kChunk == 0 && 64 % kTesters == 0, "testers of a tile share a wave");

__device__ inline int key_of(int k) { return k; }
__device__ inline int key_of(long long k) { return (int)(k & 0xffffffffll); }

// Position in [0, n) of `key` in the ascending list `keys`, or -1.
template <typename P>
__device__ inline int find_key(P keys, int n, int key) {
    int lo = 0, hi = n;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (key_of(keys[mid]) < key) lo = mid + 1;
        else hi = mid;
    }
    return lo < n && key_of(keys[lo]) == key ? lo : -1;
}

// The fragments of one tile pair: A lane: X tile [r16][4t + q]; B lane: Y
// tile [4t + q][r16], t = 0..3.
struct PairFrags {
    double x[4], y[4];
};
__device__ inline void load_pair(const double *xt, const double *yt, int64_t xi, int64_t yi,
                                 int r16, int q, PairFrags &f) {
    const double *xp = xt + xi * (TB * TB) + r16 * TB + q;
    const double *yp = yt + yi * (TB * TB) + q * TB + r16;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        f.x[t] = xp[4 * t];
        f.y[t] = yp[4 * t * TB];
    }
}

// Whether X tile `at` of the row (its mask in LDS) and the list's Y tile y, or
// the X tile of mask m and Y tile `at`, share a key; at < 0: no such tile.
__device__ inline bool shares(int at, const uint16_t *xm, int y, const unsigned *ym) {
    return at >= 0 && (ym == nullptr || (xm[at] & ym[y]) != 0u);
}
__device__ inline bool shares_at(unsigned m, int at, const unsigned *ym) {
    return at >= 0 && (ym == nullptr || (m & ym[at]) != 0u);
}

// Eight waves per SIMD, which the pairs' loads need in flight (66 registers leave
// seven, and the eighth share of a launch a round of its own): 2^20 records each,
// 16384 x 16384 x 1024, 26.1 ms with seven and 23.7 with eight; 4096^3 with 2^18
// 9.6 and 8.8.
__global__ void __launch_bounds__(kThreads, 8)
bsr_product_kernel(int M, int N, int nt, const long long *__restrict__ xkeys,
                   const int *__restrict__ xptr, const double *__restrict__ xt,
                   const long long *__restrict__ ykeys, const int *__restrict__ yptr,
                   const double *__restrict__ yt, const unsigned *__restrict__ xmask,
                   const unsigned *__restrict__ ymask, double *__restrict__ C, int64_t ldc,
                   int vec) {
    __shared__ int xk[kXKeys];
    __shared__ uint16_t xm[kXKeys];
    __shared__ unsigned bits[kBits / 32];
    __shared__ unsigned char meets[kChunk];
    const int gt = blockIdx.y, h0 = blockIdx.x * kChunk;
    const int cols = min(kChunk, nt - h0);  // column tiles of this workgroup
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int xa = xptr[gt], nx = xptr[gt + 1] - xa;
    const long long *xlist = xkeys + xa;
    const bool in_lds = nx <= kXKeys;
    for (int i = t; i < kBits / 32; i += kThreads) bits[i] = 0u;
    __syncthreads();
    if (in_lds)
        for (int i = t; i < nx; i += kThreads) {
            const int key = key_of(xlist[i]);
            xk[i] = key;
            xm[i] = xmask != nullptr ? (uint16_t)xmask[xa + i] : (uint16_t)0xffff;
            atomicOr(bits + (key / 32) % (kBits / 32), 1u << (key % 32));
        }
    __syncthreads();

    {
        const int b = t / kTesters, part = t % kTesters;
        bool meet = false;
        if (b < cols) {
            const int ya = yptr[h0 + b], ny = yptr[h0 + b + 1] - ya;
            const long long *ylist = ykeys + ya;
            const unsigned *ym = ymask != nullptr ? ymask + ya : nullptr;
            meet = min(nx, ny) > kTestKeys;
            if (!meet && ny <= kTestKeys && in_lds) {
                for (int i = part; i < ny && !meet; i += kTesters) {
                    const int key = key_of(ylist[i]);
                    if (bits[(key / 32) % (kBits / 32)] >> (key % 32) & 1u)
                        meet = shares(find_key(xk, nx, key), xm, i, ym);
                }
            } else if (!meet && nx <= kTestKeys) {
                for (int i = part; i < nx && !meet; i += kTesters)
                    meet = shares_at(xm[i], find_key(ylist, ny, xk[i]), ym);
            } else if (!meet) {
                for (int i = part; i < ny && !meet; i += kTesters)
                    meet = find_key(xlist, nx, key_of(ylist[i])) >= 0;
            }
        }
        const unsigned long long any = __ballot(meet);
        const unsigned long long group = ((1ull << kTesters) - 1ull) << (lane & ~(kTesters - 1));
        if (part == 0 && b < cols) meets[b] = (any & group) != 0ull;
    }
    __syncthreads();

    // zero the tiles that do not meet
    const int c0 = h0 * TB, cend = min(N, (h0 + cols) * TB);
    const int rows = min(TB, M - gt * TB);
    double *Crow = C + (int64_t)gt * TB * ldc;
    // (row by row, so that the workgroup's stores run along each row of C)
    if (vec) {
        // two columns per thread; N is even: a pair never straddles the edge
        static_assert(kChunk * TB == 2 * kThreads, "one pair of columns per thread");
        if (c0 + 2 * t < cend && !meets[2 * t / TB]) {
            double *dst = Crow + c0 + 2 * t;
            // (two loops: as the two sides of one branch the stores are
            // merged into a cached one)
            if (vec == kPastCaches) {
                for (int r = 0; r < rows; ++r)
                    __builtin_nontemporal_store(d2{0.0, 0.0},
                                                reinterpret_cast<d2 *>(dst + r * ldc));
            } else {
                for (int r = 0; r < rows; ++r)
                    *reinterpret_cast<d2 *>(dst + r * ldc) = d2{0.0, 0.0};
            }
        }
    } else {
        for (int r = 0; r < rows; ++r)
            for (int c = c0 + t; c < cend; c += kThreads)
                if (!meets[(c - c0) / TB]) Crow[r * ldc + c] = 0.0;
    }

    const int r16 = lane & 15, q = lane >> 4;
    for (int b = wave; b < cols; b += kThreads / 64) {
        if (!meets[b]) continue;
        const int ht = h0 + b;
        const int ya = yptr[ht], ny = yptr[ht + 1] - ya;
        const long long *ylist = ykeys + ya;
        const bool by_x = nx <= ny;
        const int ns = by_x ? nx : ny;
        d4 acc = {0.0, 0.0, 0.0, 0.0};
        for (int s0 = 0; s0 < ns; s0 += 64) {
            // this lane's pair: (xi, yi), or none
            const int s = s0 + lane;
            int xi = 0, yi = 0, at = -1;
            if (s < ns) {
                if (by_x) {
                    at = find_key(ylist, ny, in_lds ? xk[s] : key_of(xlist[s]));
                    xi = s;
                    yi = at;
                } else {
                    const int key = key_of(ylist[s]);
                    at = in_lds ? find_key(xk, nx, key) : find_key(xlist, nx, key);
                    xi = at;
                    yi = s;
                }
            }
            if (at >= 0 && in_lds && ymask != nullptr && (xm[xi] & ymask[ya + yi]) == 0u) at = -1;
            unsigned long long mask = __ballot(at >= 0);
            while (mask) {
                // two pairs at a time: the second one's loads are in flight
                // while the first multiplies
                const int l0 = __builtin_ctzll(mask);
                mask &= mask - 1;
                PairFrags f0, f1;
                load_pair(xt, yt, xa + __shfl(xi, l0), ya + __shfl(yi, l0), r16, q, f0);
                const bool two = mask != 0ull;
                if (two) {
                    const int l1 = __builtin_ctzll(mask);
                    mask &= mask - 1;
                    load_pair(xt, yt, xa + __shfl(xi, l1), ya + __shfl(yi, l1), r16, q, f1);
                }
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(f0.x[u], f0.y[u], acc, 0, 0, 0);
                if (two) {
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(f1.x[u], f1.y[u], acc, 0, 0, 0);
                }
            }
        }
        // accumulator item i of lane l: row q + 4 i, column r16
        const int col = ht * TB + r16;
        if (col < N) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int row = q + 4 * i;
                if (row < rows) Crow[row * ldc + col] = acc[i];
            }
        }
    }
}

inline unsigned grid_for(int64_t n) { return (unsigned)((n + kThreads - 1) / kThreads); }

struct Side {
    long long *keys;
    int *codes;
    long long *tkeys;
    int *ptr;
    double *tiles;
};

// distinct tile keys of n records: at most n, and at most every tile of the
// grid plus the one sentinel key of skipped records
inline int64_t max_tiles(int64_t n, int outer_ext, int key_ext) {
    const int64_t grid = (int64_t)((outer_ext + TB - 1) / TB) * ((key_ext + TB - 1) / TB) + 1;
    return n < grid ? n : grid;
}

// Bytes of bits (both sides) up to which the tiles are found by them: the
// bits are cleared, set, and read twice, which at this size takes about as
// long (60 us) as the dictionary's launches and waits at any.
constexpr int64_t kMaxBitBytes = (int64_t)64 << 20;
// rows of bits per side that one workgroup scans, 1024 per round
constexpr int64_t kMaxBitRows = 65536;

int64_t outer_tiles(int ext) { return ((int64_t)ext + TB - 1) / TB; }
int64_t bit_words(int K) { return (((int64_t)K + TB - 1) / TB + 63) / 64; }
bool by_bits(int M, int K, int N) {
    return outer_tiles(M) <= kMaxBitRows && outer_tiles(N) <= kMaxBitRows &&
           (outer_tiles(M) + outer_tiles(N)) * bit_words(K) * 8 <= kMaxBitBytes;
}

struct Layout {
    size_t status, bits, bits_bytes, dict_ws, total;
    size_t keys[2], codes[2], tkeys[2], ptr[2], tiles[2], side_bits[2], word_first[2], mask[2];
};

Layout layout(int64_t na, int64_t nb, int M, int K, int N) {
    Layout L{};
    size_t off = sizeof(StatusBlock);
    L.status = 0;
    const int64_t n[2] = {na, nb};
    const int outer[2] = {M, N};
    const bool bits = by_bits(M, K, N);
    if (bits) {
        // right after the status block: both are cleared in one pass
        L.bits = off;
        for (int s = 0; s < 2; ++s) {
            L.side_bits[s] = off;
            off += (size_t)(outer_tiles(outer[s]) * bit_words(K)) * 8;
        }
        off = align_up(off);
        L.bits_bytes = off - L.bits;
        for (int s = 0; s < 2; ++s) {
            L.word_first[s] = off;
            off += align_up((size_t)(outer_tiles(outer[s]) * bit_words(K)) * 4);
        }
    }
    for (int s = 0; s < 2; ++s) {
        if (!bits) {
            L.keys[s] = off;
            off += align_up((size_t)n[s] * 8);
            L.codes[s] = off;
            off += align_up((size_t)n[s] * 4);
        } else {
            L.mask[s] = off;
            off += align_up((size_t)n[s] * 4);
        }
        L.tkeys[s] = off;
        off += align_up((size_t)(n[s] > 0 ? n[s] : 1) * 8);
        L.ptr[s] = off;
        off += align_up((size_t)(outer_tiles(outer[s]) + 1) * 4);
        L.tiles[s] = off;
        off += align_up((size_t)max_tiles(n[s], outer[s], K) * TB * TB * 8);
    }
    if (!bits) {
        L.dict_ws = off;
        const int64_t nmax = na > nb ? na : nb;
        off += align_up(dict_workspace_bytes(nmax));
    }
    L.total = off;
    return L;
}

BitSide bit_side_of(const tcu_relation &R, bool is_b, int ext, bool masks, char *base,
                    const Layout &L) {
    const int i = is_b ? 1 : 0;
    return BitSide{R.n, R.group, R.key, R.val, R.dtype == TCU_F32,
                   (R.flags & TCU_REL_UNIQUE_CELLS) != 0, is_b, ext, (int)outer_tiles(ext),
                   reinterpret_cast<unsigned long long *>(base + L.side_bits[i]),
                   reinterpret_cast<unsigned *>(base + L.word_first[i]),
                   reinterpret_cast<int *>(base + L.ptr[i]),
                   reinterpret_cast<long long *>(base + L.tkeys[i]),
                   reinterpret_cast<double *>(base + L.tiles[i]),
                   masks ? reinterpret_cast<unsigned *>(base + L.mask[i]) : nullptr};
}

// Steps 1-4 of both relations by bits, the status block cleared.
hipError_t build_by_bits(const tcu_relation &A, const tcu_relation &B, int M, int K, int N,
                         bool masks, char *base, const Layout &L, StatusBlock *st,
                         hipStream_t s) {
    const BitPair p{bit_side_of(A, false, M, masks, base, L),
                    bit_side_of(B, true, N, masks, base, L), (int)bit_words(K), K};
    hipError_t e = launch_zero_f64(reinterpret_cast<double *>(st),
                                   (L.bits + L.bits_bytes) / sizeof(double), s);
    if (e != hipSuccess) return e;
    const unsigned ga = grid_for(A.n), gb = grid_for(B.n);
    constexpr unsigned kRows = kThreads / 64;
    const unsigned ra = ((unsigned)p.a.rows + kRows - 1) / kRows;
    const unsigned rb = ((unsigned)p.b.rows + kRows - 1) / kRows;
    // both sides' records in one launch, where that may have so many
    const bool one = (int64_t)ga + gb <= max_workgroups(kThreads);
    if (one && ga + gb > 0) tile_bits_kernel<<<ga + gb, kThreads, 0, s>>>(p, ga, st);
    if (!one) tile_bits_kernel<<<ga, kThreads, 0, s>>>(p, ga, st);
    if (!one) tile_bits_kernel<<<gb, kThreads, 0, s>>>(p, 0u, st);
    tile_count_kernel<<<ra + rb, kThreads, 0, s>>>(p, ra);
    tile_scan_kernel<<<2, kScanThreads, 0, s>>>(p);
    tile_list_kernel<<<ra + rb, kThreads, 0, s>>>(p, ra);
    if (one && ga + gb > 0) tile_place_kernel<<<ga + gb, kThreads, 0, s>>>(p, ga);
    if (!one) tile_place_kernel<<<ga, kThreads, 0, s>>>(p, ga);
    if (!one) tile_place_kernel<<<gb, kThreads, 0, s>>>(p, 0u);
    return hipGetLastError();
}

template <typename T>
hipError_t scatter_t(const tcu_relation &R, const Side &sd, int key_rows, hipStream_t s) {
    const T *v = static_cast<const T *>(R.val);
    if (R.flags & TCU_REL_UNIQUE_CELLS)
        tile_scatter_kernel<T, true><<<grid_for(R.n), kThreads, 0, s>>>(
            R.n, R.group, R.key, v, sd.keys, sd.codes, key_rows, sd.tiles);
    else
        tile_scatter_kernel<T, false><<<grid_for(R.n), kThreads, 0, s>>>(
            R.n, R.group, R.key, v, sd.keys, sd.codes, key_rows, sd.tiles);
    return hipGetLastError();
}

// Steps 1-4 for one relation: outer = group column (g for A, h for B).
hipError_t build_side(const tcu_relation &R, int outer_ext, int K, int which, const Side &sd,
                      void *dict_ws, StatusBlock *st, hipStream_t s) {
    int64_t ntiles = 0;
    if (R.n > 0) {
        if (R.dtype == TCU_F32)
            tile_key_kernel<float><<<grid_for(R.n), kThreads, 0, s>>>(R.n, R.group, R.key,
                                                                      outer_ext, K, sd.keys, st,
                                                                      which);
        else
            tile_key_kernel<double><<<grid_for(R.n), kThreads, 0, s>>>(R.n, R.group, R.key,
                                                                       outer_ext, K, sd.keys, st,
                                                                       which);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        e = run_dict_encode(sd.keys, R.n, nullptr, 0, sd.codes, nullptr, sd.tkeys, &ntiles,
                            dict_ws, s);
        if (e != hipSuccess) return e;
        // the sentinel key of skipped records, if present, is the last tile
        // and lies beyond every tile row: the pointers exclude it
        e = launch_zero_f64(sd.tiles, (size_t)ntiles * TB * TB, s);
        if (e != hipSuccess) return e;
        e = R.dtype == TCU_F32 ? scatter_t<float>(R, sd, which, s)
                               : scatter_t<double>(R, sd, which, s);
        if (e != hipSuccess) return e;
    }
    const int ot = (int)outer_tiles(outer_ext);
    tile_ptr_kernel<<<grid_for(ot + 1), kThreads, 0, s>>>(sd.tkeys, ntiles, ot, sd.ptr);
    return hipGetLastError();
}

}  // namespace

size_t bsr_workspace_bytes(int64_t na, int64_t nb, int M, int K, int N) {
    return layout(na, nb, M, K, N).total;
}

hipError_t run_join_agg_bsr(const tcu_relation &A, const tcu_relation &B, int M, int K, int N,
                            double *C, void *ws, hipStream_t s) {
    const Layout L = layout(A.n, B.n, M, K, N);
    char *base = static_cast<char *>(ws);
    StatusBlock *st = reinterpret_cast<StatusBlock *>(base);
    Side sd[2];
    for (int i = 0; i < 2; ++i) {
        sd[i].keys = reinterpret_cast<long long *>(base + L.keys[i]);
        sd[i].codes = reinterpret_cast<int *>(base + L.codes[i]);
        sd[i].tkeys = reinterpret_cast<long long *>(base + L.tkeys[i]);
        sd[i].ptr = reinterpret_cast<int *>(base + L.ptr[i]);
        sd[i].tiles = reinterpret_cast<double *>(base + L.tiles[i]);
    }
    hipError_t e;
    const bool masks = L.bits_bytes > 0 && A.val == nullptr && B.val == nullptr;
    if (L.bits_bytes > 0) {
        e = build_by_bits(A, B, M, K, N, masks, base, L, st, s);
    } else {
        e = launch_clear_status(st, s);
        if (e == hipSuccess) e = build_side(A, M, K, 0, sd[0], base + L.dict_ws, st, s);
        if (e == hipSuccess) e = build_side(B, N, K, 1, sd[1], base + L.dict_ws, st, s);
    }
    if (e != hipSuccess) return e;
    const int mt = (M + TB - 1) / TB, nt = (N + TB - 1) / TB;
    const int vec = N % 2 != 0 || ((uintptr_t)C & 15) != 0 ? 0
                    : (size_t)M * (size_t)N * sizeof(double) > kLastLevelCache ? kPastCaches : 1;
    for (int g0 = 0; g0 < mt; g0 += 65535) {
        // tile rows run along the grid's y, at most 65535 per launch
        const int gn = mt - g0 < 65535 ? mt - g0 : 65535;
        bsr_product_kernel<<<dim3((unsigned)((nt + kChunk - 1) / kChunk), (unsigned)gn), kThreads, 0,
                             s>>>(M - g0 * TB, N, nt, sd[0].tkeys, sd[0].ptr + g0,
                                  sd[0].tiles, sd[1].tkeys, sd[1].ptr, sd[1].tiles,
                                  masks ? reinterpret_cast<unsigned *>(base + L.mask[0]) : nullptr,
                                  masks ? reinterpret_cast<unsigned *>(base + L.mask[1]) : nullptr,
                                  C + (int64_t)g0 * TB * N, N, vec);
    }
    return hipGetLastError();
}

}  // namespace tcu
