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
//   1. tile key per record: X: (g/16, k/16), Y: (h/16, k/16), packed as
//      outer << 32 | key tile;
//   2. the distinct tile keys, sorted, and each record's tile index (the
//      dictionary machinery of dict.hip: hash set, compaction, bitonic sort,
//      rank lookup; one host synchronisation to size the sort);
//   3. the first tile of every tile row of X and tile column of Y (binary
//      search over the sorted keys): tile lists sorted by key tile;
//   4. every record's value added into its tile (16 x 16 FP64, X tiles
//      [g%16][k%16], Y tiles [k%16][h%16]);
//   5. per tile row of C and chunk of column tiles: the tiles whose lists
//      share no key tile are zeroed, the others take, for every common key
//      tile, four v_mfma_f64_16x16x4_f64 into their accumulator (see below).
// The result equals the dense operator's: the products skipped are products
// of all-zero tiles.  C is dense M x N FP64, as for tcu_join_agg_fwd.
#include "internal.h"

namespace tcu {
namespace {

typedef double d4 __attribute__((ext_vector_type(4)));

constexpr int kThreads = 256;
constexpr int TB = 16;                           // tile edge
constexpr long long kBadKey = 0x7fffffffffffffffll;  // record outside the shape

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
// of C and up to kMaxChunk column tiles:
//   1. the row's X keys go to LDS, as a list and as a bit per key modulo
//      8192, and each thread tests one column tile: a short list of Y against
//      the bits and, where one is set, by binary search of the list (a short
//      list of X against a long one of Y by searches in the latter; lists
//      that both exceed kTestKeys keys are taken to meet);
//   2. the tiles that do not meet are zeroed row by row in long stores;
//   3. the others go to the waves, one tile each: the lanes take 64 keys of
//      the shorter list, search the longer, and the tile pairs that meet run
//      on the matrix cores in ascending key order (as the serial walk did, so
//      the sums round the same).
// The same product then takes about 450 us (4.7 TB/s of stores; a plain fill
// reaches 6.7); 4096 x 4096 cells where nine tiles in ten meet 285 us for the
// whole operator against 707, a graph's 65536 x 64 with long lists of Y 324
// against 2751.
constexpr int kMaxChunk = 256;   // column tiles per workgroup, one per thread
constexpr int kMinChunk = 32;
constexpr int kXKeys = 1024;     // X keys of one tile row held in LDS
constexpr int kTestKeys = 64;
constexpr int kBits = 8192;      // one bit per key modulo this: set for the row's X keys
static_assert(kMaxChunk == kThreads, "one thread per column tile");

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

__global__ void __launch_bounds__(kThreads)
bsr_product_kernel(int M, int N, int nt, int chunk, const long long *__restrict__ xkeys,
                   const int *__restrict__ xptr, const double *__restrict__ xt,
                   const long long *__restrict__ ykeys, const int *__restrict__ yptr,
                   const double *__restrict__ yt, double *__restrict__ C, int64_t ldc, int vec) {
    __shared__ int xk[kXKeys];
    __shared__ unsigned bits[kBits / 32];
    __shared__ unsigned char meets[kMaxChunk];
    const int gt = blockIdx.y, h0 = blockIdx.x * chunk;
    const int cols = min(chunk, nt - h0);  // column tiles of this workgroup
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
            atomicOr(bits + (key / 32) % (kBits / 32), 1u << (key % 32));
        }
    __syncthreads();

    if (t < cols) {
        const int ya = yptr[h0 + t], ny = yptr[h0 + t + 1] - ya;
        const long long *ylist = ykeys + ya;
        bool meet = min(nx, ny) > kTestKeys;
        if (!meet && ny <= kTestKeys && in_lds) {
            for (int i0 = 0; i0 < ny && !meet; i0 += 8) {
                int key[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) key[i] = key_of(ylist[min(i0 + i, ny - 1)]);
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    if (!meet && (bits[(key[i] / 32) % (kBits / 32)] >> (key[i] % 32) & 1u))
                        meet = find_key(xk, nx, key[i]) >= 0;
            }
        } else if (!meet && nx <= kTestKeys) {
            for (int i = 0; i < nx && !meet; ++i) meet = find_key(ylist, ny, xk[i]) >= 0;
        } else if (!meet) {
            for (int i = 0; i < ny && !meet; ++i)
                meet = find_key(xlist, nx, key_of(ylist[i])) >= 0;
        }
        meets[t] = meet;
    }
    __syncthreads();

    // zero the tiles that do not meet
    const int c0 = h0 * TB, cend = min(N, (h0 + cols) * TB);
    const int rows = min(TB, M - gt * TB);
    double *Crow = C + (int64_t)gt * TB * ldc;
    // (row by row, so that the workgroup's stores run along each row of C)
    if (vec) {
        // columns c0 + 2 t + 512 p; N is even: a pair never straddles the edge
        constexpr int kPasses = kMaxChunk * TB / (2 * kThreads);
        unsigned todo = 0;
        for (int p = 0; p < kPasses; ++p) {
            const int c = 2 * t + 2 * kThreads * p;
            if (c0 + c < cend && !meets[c / TB]) todo |= 1u << p;
        }
        for (int r = 0; r < rows; ++r) {
            double2 *dst = reinterpret_cast<double2 *>(Crow + r * ldc + c0) + t;
#pragma unroll
            for (int p = 0; p < kPasses; ++p)
                if (todo >> p & 1) dst[p * kThreads] = make_double2(0.0, 0.0);
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

struct Layout {
    size_t status, dict_ws, total;
    size_t keys[2], codes[2], tkeys[2], ptr[2], tiles[2];
};

Layout layout(int64_t na, int64_t nb, int M, int K, int N) {
    Layout L{};
    size_t off = sizeof(StatusBlock);
    L.status = 0;
    const int64_t n[2] = {na, nb};
    const int outer[2] = {M, N};
    for (int s = 0; s < 2; ++s) {
        L.keys[s] = off;
        off += align_up((size_t)n[s] * 8);
        L.codes[s] = off;
        off += align_up((size_t)n[s] * 4);
        L.tkeys[s] = off;
        off += align_up((size_t)(n[s] > 0 ? n[s] : 1) * 8);
        L.ptr[s] = off;
        off += align_up((size_t)((outer[s] + TB - 1) / TB + 1) * 4);
        L.tiles[s] = off;
        off += align_up((size_t)max_tiles(n[s], outer[s], K) * TB * TB * 8);
    }
    L.dict_ws = off;
    const int64_t nmax = na > nb ? na : nb;
    off += align_up(dict_workspace_bytes(nmax));
    L.total = off;
    return L;
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
    const int outer_tiles = (outer_ext + TB - 1) / TB;
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
    tile_ptr_kernel<<<grid_for(outer_tiles + 1), kThreads, 0, s>>>(sd.tkeys, ntiles, outer_tiles,
                                                                   sd.ptr);
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
    hipError_t e = launch_clear_status(st, s);
    if (e != hipSuccess) return e;
    e = build_side(A, M, K, 0, sd[0], base + L.dict_ws, st, s);
    if (e != hipSuccess) return e;
    e = build_side(B, N, K, 1, sd[1], base + L.dict_ws, st, s);
    if (e != hipSuccess) return e;
    const int mt = (M + TB - 1) / TB, nt = (N + TB - 1) / TB;
    // wide chunks share the row's keys and give long stores; fewer column
    // tiles per workgroup while the grid has fewer than 16384 of them (about
    // nine rounds): measured at 16384^2 cells, 2^20 keys, 726 us for the
    // operator with at least 4096 workgroups, 706 with 8192, 682 with 16384
    int chunk = kMaxChunk;
    while (chunk > kMinChunk && (int64_t)mt * ((nt + chunk - 1) / chunk) < 16384) chunk /= 2;
    const int vec = N % 2 == 0 && ((uintptr_t)C & 15) == 0;
    for (int g0 = 0; g0 < mt; g0 += 65535) {
        // tile rows run along the grid's y, at most 65535 per launch
        const int gn = mt - g0 < 65535 ? mt - g0 : 65535;
        bsr_product_kernel<<<dim3((unsigned)((nt + chunk - 1) / chunk), (unsigned)gn), kThreads, 0,
                             s>>>(M - g0 * TB, N, nt, chunk, sd[0].tkeys, sd[0].ptr + g0,
                                  sd[0].tiles, sd[1].tkeys, sd[1].ptr, sd[1].tiles,
                                  C + (int64_t)g0 * TB * N, N, vec);
    }
    return hipGetLastError();
}

}  // namespace tcu
