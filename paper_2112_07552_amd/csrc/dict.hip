// dict.hip -- dictionary encoding of join and group-by columns.
//
// Section 3.1 of TCUDB builds its matrices over dom(ID), the union of the
// two relations' ID domains with k distinct values v_1, ..., v_k: a value's
// matrix column is its position in that domain.  Here the domain is sorted,
// so a value's code is its rank among the distinct values of both columns:
// codes are deterministic (independent of record order and of the GPU's
// scheduling) and ORDER BY on codes is ORDER BY on values (Section 3.4).
//
// Steps (all on the caller's stream):
//  1. insert every value into an open-addressing hash set (linear probing,
//     64-bit compare-and-swap);
//  2. up to kSmallDict distinct values: each one's rank among them goes into a
//     code array parallel to the table, and every record's value is looked up;
//  3. the host waits, for the count it returns;
//  4. with more distinct values only then, and with grids of that count: the
//     occupied slots compacted into a list, the list sorted (chunks of 2048 in
//     LDS, then merges of eight runs at a time, each value finding its place
//     by binary search in the other runs), ranks and codes as above.
// So a dictionary of few values takes four launches and any other up to ten, with
// one wait.  The first attempt uses a table of at most 2^18 slots
// (3 MB with its codes, which an XCD's L2 holds), whatever the column length:
// clearing and scanning a table sized for 2^25 values with 32 distinct ones
// took 270 us, clearing this one 4 us.  When the values do not fit (a probe
// sequence of kSmallProbes slots, or more than half of the slots taken) the
// insertion is run again, with 2^21 slots and then with twice as many slots as
// values, where every probe sequence meets a free slot: four launches and a wait
// more each.  (With these attempts enqueued behind the first, to leave at once
// on the device, no call would wait twice, but every one of more than 2^17 values
// paid for their launches: 2^24 values, 32 distinct 88 us and so 112, 10^6, 500
// distinct 59 and 65, against 17 to 50 us of 800 to 5200 gained above 2^17 distinct
// ones.)
//
// INT64_MIN marks an empty slot; a column value equal to INT64_MIN is
// handled apart (it is the smallest value, so it gets code 0 when present).
#include <algorithm>

#include "internal.h"

namespace tcu {
namespace {

constexpr int kThreads = 256;
constexpr unsigned long long kEmpty = 0x8000000000000000ull;
constexpr size_t kSmallSlots[2] = {(size_t)1 << 18, (size_t)1 << 21};
constexpr unsigned long long kSmallProbes = 64;

// MurmurHash3's 64-bit finaliser (Appleby) as the slot hash.
__device__ inline unsigned long long fmix64(unsigned long long k) {
    k ^= k >> 33;
    k *= 0xff51afd7ed558ccdull;
    k ^= k >> 33;
    k *= 0xc4ceb9fe1a85ec53ull;
    k ^= k >> 33;
    return k;
}

// A cheaper hash for the LDS arrays (Fibonacci hashing of the folded value):
// two 32-bit multiplies, where fmix64 takes the time of ten.
__device__ inline unsigned lds_hash(unsigned long long k, int bits) {
    return (((unsigned)k ^ ((unsigned)(k >> 32) * 0x85ebca6bu)) * 0x9e3779b1u) >> (32 - bits);
}

struct DictState {
    unsigned long long count;  // distinct values other than INT64_MIN
    unsigned int has_min;      // INT64_MIN occurs
    unsigned int overflow;     // a probe sequence ran out: the table is too small
    unsigned int listed;       // places taken in the compacted list
};

// One attempt: the table, the most distinct values it may hold, and the
// probes allowed per value.
struct Table {
    unsigned long long *slot;
    int *code;  // rank of the slot's value
    unsigned long long mask, max_probes, max_count;
};

// Up to this many distinct values the insertion lists their slots, in LDS first
// (with a list of twice as many fewer of its workgroups would fit a CU).
constexpr int kSmallDict = 1024;

// What the sort's kernels do first: the number of distinct values, or 0 when
// this attempt failed.
__device__ inline int64_t live_count(const DictState *st, const Table &t) {
    const unsigned long long c = st->count;
    return (st->overflow || c > t.max_count) ? 0 : (int64_t)c;
}

__global__ void dict_clear_kernel(Table t, DictState *st) {
    const size_t stride = (size_t)gridDim.x * kThreads;
    for (size_t i = (size_t)blockIdx.x * kThreads + threadIdx.x; i <= t.mask; i += stride)
        t.slot[i] = kEmpty;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        st->count = 0;
        st->has_min = 0;
        st->overflow = 0;
        st->listed = 0;
    }
}

// After step (kk, j) of a bitonic sort with one pair per thread: a wave's 64
// pairs at distance j <= 64 are 128 neighbouring values, its own, so the
// workgroup meets only around wider steps (2048 values: 20 us with a barrier
// after every step).
__device__ inline void step_barrier(int kk, int j) {
    if (max(j, j > 1 ? j / 2 : kk) > 64) {
        __syncthreads();
    } else {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
}

// Both columns, value i of [0, n_a + n_b).  A workgroup remembers values it
// has seen in a direct-mapped LDS array, so a column with few distinct values
// touches the table a few times per workgroup instead of once per record:
// 2^24 values with 32 distinct took 300 us against 46 us here (2.9 TB/s of
// the column).  Columns with many distinct values mostly miss and go to the
// table.
constexpr int kInsThreads = 1024;
constexpr int kSeenBits = 12;       // LDS entries: 4096 (32 KB)
constexpr unsigned kSeen = 1u << kSeenBits;

// PER: values per thread and round, loaded together.  Columns too short to
// fill the chip that way take one per thread: a value's probes are a chain of
// memory round trips.
// `mine` lists the slots this workgroup has filled, while they are few; each
// workgroup adds its number to the count and, as long as all of them are at
// most kSmallDict, its slots to `list`.
template <int PER, int THREADS>
__global__ void __launch_bounds__(THREADS)
dict_insert_kernel(const long long *__restrict__ a, int64_t n_a, const long long *__restrict__ b,
                   int64_t n, Table t, unsigned int *__restrict__ list, DictState *st) {
    __shared__ unsigned long long seen[kSeen];
    __shared__ unsigned int mine[kSmallDict];
    __shared__ unsigned int seen_min, full, filled;
    __shared__ unsigned long long base;
    for (unsigned i = threadIdx.x; i < kSeen; i += THREADS) seen[i] = kEmpty;
    if (threadIdx.x == 0) seen_min = full = filled = 0u;
    __syncthreads();
    const int64_t step = (int64_t)gridDim.x * THREADS * PER;
    for (int64_t i0 = (int64_t)blockIdx.x * THREADS * PER; i0 < n; i0 += step) {
        // the table found full by anyone: leave (one lane asks for all)
        if (threadIdx.x == 0 &&
            __hip_atomic_load(&st->overflow, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
            __hip_atomic_store(&full, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (__hip_atomic_load(&full, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) break;
        unsigned long long v[PER];
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const int64_t i = i0 + j * THREADS + threadIdx.x;
            const int64_t c = i < n ? i : i0;  // past the end: a value again
            v[j] = (unsigned long long)(c < n_a ? a[c] : b[c - n_a]);
        }
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            if (v[j] == kEmpty) {
                if (seen_min == 0u) {
                    atomicOr(&st->has_min, 1u);
                    seen_min = 1u;
                }
                continue;
            }
            unsigned long long *slot_seen = seen + lds_hash(v[j], kSeenBits);
            // An entry holding v was put there by the thread that inserts v:
            // the exchange lets one thread of the workgroup through, so that
            // at the kernel's start not every wave goes to the same few slots
            // (2^25 + 2^24 values, 32 distinct: 139 us; with a plain store
            // after the insertion 527 us)
            if (__hip_atomic_load(slot_seen, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) ==
                    v[j] ||
                atomicExch(slot_seen, v[j]) == v[j])
                continue;
            unsigned long long h = fmix64(v[j]) & t.mask;
            unsigned long long probe = 0;
            for (; probe < t.max_probes; ++probe) {
                // a read first: a value already present costs no atomic (one
                // that another XCD has just put there may still read as a
                // free slot; the compare-and-swap then returns it)
                const unsigned long long got = __hip_atomic_load(
                    t.slot + h, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                if (got == v[j]) break;
                if (got == kEmpty) {
                    const unsigned long long prev = atomicCAS(t.slot + h, kEmpty, v[j]);
                    if (prev == kEmpty) {
                        const unsigned int q = atomicAdd(&filled, 1u);
                        if (q < (unsigned)kSmallDict) mine[q] = (unsigned int)h;
                        break;
                    }
                    if (prev == v[j]) break;
                }
                h = (h + 1) & t.mask;
            }
            if (probe == t.max_probes) atomicOr(&st->overflow, 1u);
        }
    }
    __syncthreads();
    const unsigned int got = filled;
    if (threadIdx.x == 0 && got > 0u) base = atomicAdd(&st->count, (unsigned long long)got);
    __syncthreads();
    if (got > 0u && base + got <= (unsigned long long)kSmallDict)
        for (unsigned int i = threadIdx.x; i < got; i += THREADS) list[base + i] = mine[i];
}

// A small dictionary, kRankValues values per workgroup: the listed slots' values
// written to dict at their ranks, and the ranks to the slots' codes.  A value's
// rank is counted, by kRankParts neighbouring lanes that each compare it with
// an eighth of the values: 6 us for 512 of them, where one workgroup's bitonic
// network took 11 (for runs of 2048 the network is the faster one).  (Done by
// the insertion's last workgroup to finish, this saved a launch and cost 40 us
// at 2^24 values, for a count of finished workgroups and fences.)
constexpr int kRankThreads = 512, kRankParts = 8, kRankValues = kRankThreads / kRankParts;
__global__ void __launch_bounds__(kRankThreads)
dict_small_kernel(Table t, const unsigned int *__restrict__ list, const DictState *st,
                  long long *__restrict__ dict) {
    __shared__ long long val[kSmallDict];
    const unsigned long long k = st->count;
    const int first = (int)blockIdx.x * kRankValues;
    if (st->overflow || k > (unsigned long long)kSmallDict) return;
    const int shift = st->has_min ? 1 : 0;
    if (first == 0 && threadIdx.x == 0 && shift) dict[0] = (long long)kEmpty;
    if (first >= (int)k) return;
    for (int i = threadIdx.x; i < (int)k; i += kRankThreads) val[i] = (long long)t.slot[list[i]];
    __syncthreads();
    const int i = first + (int)threadIdx.x / kRankParts, part = (int)threadIdx.x % kRankParts;
    const long long v = val[min(i, (int)k - 1)];
    int rank = 0;  // (the values differ)
    for (int j = part; j < (int)k; j += kRankParts) rank += val[j] < v;
    for (int d = 1; d < kRankParts; d <<= 1) rank += __shfl_xor(rank, d);
    if (i >= (int)k || part != 0) return;
    dict[rank + shift] = v;
    t.code[list[i]] = rank + shift;
}

// The occupied slots as a list, in no particular order.  One atomic per
// workgroup and kThreads * PER slots: atomics on one address are served one
// after the other at about 9 ns each, and one per wave cost 600 us at 2^22
// slots.
template <int PER>
__global__ void __launch_bounds__(kThreads)
dict_compact_kernel(Table t, long long *__restrict__ distinct, DictState *st) {
    __shared__ unsigned int wave_sum[kThreads / 64], base;
    if (st->overflow) return;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const size_t i0 = (size_t)blockIdx.x * kThreads * PER + threadIdx.x;
    unsigned long long v[PER];
    unsigned int mine = 0;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const size_t i = i0 + (size_t)j * kThreads;
        const unsigned long long x = t.slot[i <= t.mask ? i : 0];
        v[j] = i <= t.mask ? x : kEmpty;
    }
#pragma unroll
    for (int j = 0; j < PER; ++j) mine += v[j] != kEmpty;
    unsigned int incl = mine;
    for (int d = 1; d < 64; d <<= 1) {
        const unsigned int up = (unsigned int)__shfl_up((int)incl, d);
        if (lane >= d) incl += up;
    }
    if (lane == 63) wave_sum[wave] = incl;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned int all = 0;
        for (int w = 0; w < kThreads / 64; ++w) {
            const unsigned int c = wave_sum[w];
            wave_sum[w] = all;
            all += c;
        }
        base = all ? atomicAdd(&st->listed, all) : 0u;
    }
    __syncthreads();
    unsigned int at = base + wave_sum[wave] + (incl - mine);
#pragma unroll
    for (int j = 0; j < PER; ++j)
        if (v[j] != kEmpty && at < t.max_count) distinct[at++] = (long long)v[j];
}

// ------------------------------------------------------------------- sort
// Runs of kRunLen sorted in LDS, then passes that merge kFan neighbouring
// runs.  k values take merge_passes(k) passes; each pass moves the list from
// one buffer to the other, and the first kernel picks its target so that the
// last one leaves the result in `sorted`.
constexpr int kRunLen = 2048;
constexpr int kFan = 8;
constexpr int kSortThreads = 1024;

__host__ __device__ inline int merge_passes(int64_t k) {
    int p = 0;
    for (int64_t run = kRunLen; run < k; run *= kFan) ++p;
    return p;
}

// Bitonic sort of one run in LDS (in place, or into `other` when the number
// of merge passes is odd).
__global__ void __launch_bounds__(kSortThreads)
dict_sort_runs_kernel(long long *__restrict__ sorted, long long *__restrict__ other, Table t,
                      const DictState *st) {
    __shared__ long long v[kRunLen];
    const int64_t k = live_count(st, t);
    const int64_t r0 = (int64_t)blockIdx.x * kRunLen;
    if (r0 >= k) return;
    const int len = (int)min((int64_t)kRunLen, k - r0);
    int P = 2;
    while (P < len) P *= 2;
    for (int i = threadIdx.x; i < P; i += kSortThreads)
        v[i] = i < len ? sorted[r0 + i] : 0x7fffffffffffffffll;
    __syncthreads();
    for (int kk = 2; kk <= P; kk *= 2)
        for (int j = kk / 2; j > 0; j /= 2) {
            const int p = threadIdx.x;
            if (p < P / 2) {
                const int i = ((p & ~(j - 1)) << 1) | (p & (j - 1)), l = i + j;
                const long long x = v[i], y = v[l];
                if ((x > y) == ((i & kk) == 0)) {
                    v[i] = y;
                    v[l] = x;
                }
            }
            step_barrier(kk, j);
        }
    __syncthreads();
    long long *dst = (merge_passes(k) & 1) ? other : sorted;
    for (int i = threadIdx.x; i < len; i += kSortThreads) dst[r0 + i] = v[i];
}

// Pass `pass` over runs of `run` values: a value's place in the merged group
// of kFan runs is its own index in its run plus the number of smaller values
// in each other run (all values differ).  The searches of one thread advance
// together, so their loads overlap: a pass takes one search's latency (about
// 6 us at 2^17 values, where the passes of a bitonic network took 300 us).
__global__ void __launch_bounds__(kThreads)
dict_merge_kernel(long long *__restrict__ sorted, long long *__restrict__ other, int64_t run,
                  int pass, Table t, const DictState *st) {
    const int64_t k = live_count(st, t);
    if (k <= run) return;  // one run: merged already
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i >= k) return;
    const bool flip = ((merge_passes(k) - pass) & 1) != 0;
    const long long *src = flip ? other : sorted;
    long long *dst = flip ? sorted : other;
    const long long v = src[i];
    const int64_t own = i / run, g0 = own / kFan * kFan;
    int64_t lo[kFan], end[kFan];
#pragma unroll
    for (int q = 0; q < kFan; ++q) {
        lo[q] = min((g0 + q) * run, k);
        end[q] = (g0 + q == own) ? lo[q] : min(lo[q] + run, k);
    }
    for (int64_t s = run; s > 0; s >>= 1) {
        long long x[kFan];
#pragma unroll
        for (int q = 0; q < kFan; ++q) x[q] = src[min(lo[q] + s - 1, k - 1)];
#pragma unroll
        for (int q = 0; q < kFan; ++q)
            if (lo[q] + s <= end[q] && x[q] < v) lo[q] += s;
    }
    int64_t pos = g0 * run + (i - own * run);
#pragma unroll
    for (int q = 0; q < kFan; ++q)
        if (g0 + q != own) pos += lo[q] - min((g0 + q) * run, k);
    dst[pos] = v;
}

// ----------------------------------------------------------------- lookup
__device__ inline int64_t find_slot(const Table &t, unsigned long long v) {
    unsigned long long h = fmix64(v) & t.mask;
    for (unsigned long long probe = 0; probe <= t.mask; ++probe) {
        const unsigned long long x = t.slot[h];
        if (x == v) return (int64_t)h;
        if (x == kEmpty) return -1;
        h = (h + 1) & t.mask;
    }
    return -1;
}

__global__ void __launch_bounds__(kThreads)
dict_rank_kernel(const long long *__restrict__ sorted, Table t, const DictState *st,
                 long long *__restrict__ dict) {
    if (st->overflow || st->count > t.max_count) return;
    const int64_t k = (int64_t)st->count;
    const int64_t r = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    const int shift = st->has_min ? 1 : 0;
    if (r == 0 && shift) dict[0] = (long long)kEmpty;
    if (r >= k) return;
    const long long v = sorted[r];
    dict[r + shift] = v;
    const int64_t s = find_slot(t, (unsigned long long)v);
    if (s >= 0) t.code[s] = (int)(r + shift);
}

// Codes of both columns, if the dictionary has at most `limit` values.  A
// dictionary of at most kLdsDict values is put into an LDS hash table by each
// workgroup when the columns are long enough to repay it (kLdsMinN): 2^24 records
// with 32 distinct values 38 us (5.3 TB/s) against 72 us through the table in
// memory.
constexpr int kLookThreads = 512;
constexpr int kLdsDict = 2048;
constexpr int kLdsBits = 12;
constexpr unsigned kLdsSlots = 1u << kLdsBits;  // 32 KB of values, 8 KB of codes
constexpr int64_t kLdsMinN = (int64_t)1 << 19;

template <int PER>
__global__ void __launch_bounds__(kLookThreads)
dict_lookup_kernel(const long long *__restrict__ a, int64_t n_a, const long long *__restrict__ b,
                   int64_t n, const long long *__restrict__ dict, Table t,
                   unsigned long long limit, const DictState *st, int *__restrict__ codes_a,
                   int *__restrict__ codes_b) {
    __shared__ unsigned long long lv[kLdsSlots];
    __shared__ uint16_t lc[kLdsSlots];
    if (st->overflow || st->count > limit) return;
    const int64_t k = (int64_t)st->count;
    const int shift = st->has_min ? 1 : 0;
    const bool lds = k <= kLdsDict && n >= kLdsMinN;
    if (lds) {
        for (unsigned i = threadIdx.x; i < kLdsSlots; i += kLookThreads) lv[i] = kEmpty;
        __syncthreads();
        for (int r = threadIdx.x; r < (int)k; r += kLookThreads) {
            const unsigned long long v = (unsigned long long)dict[r + shift];
            // at most half of the slots are taken, so a free one is met
            unsigned h = lds_hash(v, kLdsBits);
            while (atomicCAS(lv + h, kEmpty, v) != kEmpty) h = (h + 1) & (kLdsSlots - 1);
            lc[h] = (uint16_t)(r + shift);
        }
        __syncthreads();
    }
    // from the columns' end: what the insertion read last is still in the
    // last-level cache
    constexpr int64_t kPart = (int64_t)kLookThreads * PER;
    const int64_t parts = (n + kPart - 1) / kPart;
    for (int64_t q = blockIdx.x; q < parts; q += gridDim.x) {
        const int64_t i0 = (parts - 1 - q) * kPart;
        unsigned long long v[PER];
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const int64_t i = i0 + j * kLookThreads + threadIdx.x;
            const int64_t c = i < n ? i : i0;
            v[j] = (unsigned long long)(c < n_a ? a[c] : b[c - n_a]);
        }
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const int64_t i = i0 + j * kLookThreads + threadIdx.x;
            if (i >= n) continue;
            int code;
            if (v[j] == kEmpty) {
                code = 0;
            } else if (lds) {
                unsigned h = lds_hash(v[j], kLdsBits);
                unsigned long long x;
                while ((x = lv[h]) != v[j] && x != kEmpty) h = (h + 1) & (kLdsSlots - 1);
                code = x == v[j] ? (int)lc[h] : -1;
            } else {
                const int64_t s = find_slot(t, v[j]);
                code = s >= 0 ? t.code[s] : -1;
            }
            if (i < n_a) codes_a[i] = code;
            else codes_b[i - n_a] = code;
        }
    }
}

inline unsigned grid_for(int64_t n) { return (unsigned)((n + kThreads - 1) / kThreads); }

// Workgroups of a kernel over the columns: `per` records each, at most `most`
// (more records then take more rounds).
inline unsigned stream_grid(int64_t n, int per, int64_t most) {
    return (unsigned)std::min<int64_t>(most, (n + per - 1) / per);
}

// Columns by length: one value per thread while that takes one round of 256
// workgroups of 1024 threads (of 512 up to kTiny values: a value's probes are a
// chain of memory round trips, so they go to more CUs); then those 256 with four
// values per thread; from 2^21 values 512 workgroups with eight.  Fewer and larger
// workgroups meet less often on the same few slots at the start: us per call with
// 512 threads and twice the workgroups, and now: 2^24 + 2^24 values, 32 distinct
// 182 and 167; 2^24 110 and 97; 10^6, 500 distinct 78 and 72; 10^5 + 10^5, 200
// distinct 63 and 55; (eight values at a time against four: 211 and 242).
constexpr int64_t kTiny = 65536, kShort = (int64_t)256 * kInsThreads, kMiddle = (int64_t)1 << 21;

struct Columns {
    const long long *a, *b;
    int64_t n_a, n;
};

// Steps 1-2 on one table, codes apart.
void enqueue_insert(const Columns &c, const Table &t, unsigned int *list, DictState *st,
                    long long *dict, hipStream_t s) {
    const size_t clear_blocks = ((size_t)t.mask + kThreads) / kThreads;
    dict_clear_kernel<<<(unsigned)std::min<size_t>(clear_blocks, 65536), kThreads, 0, s>>>(t, st);
    if (c.n == 0) return;
    if (c.n <= kTiny)
        dict_insert_kernel<1, 512><<<stream_grid(c.n, 512, 128), 512, 0, s>>>(c.a, c.n_a, c.b, c.n,
                                                                              t, list, st);
    else if (c.n <= kShort)
        dict_insert_kernel<1, kInsThreads><<<stream_grid(c.n, kInsThreads, 256), kInsThreads, 0,
                                             s>>>(c.a, c.n_a, c.b, c.n, t, list, st);
    else if (c.n <= kMiddle)
        dict_insert_kernel<4, kInsThreads><<<stream_grid(c.n, kInsThreads * 4, 256), kInsThreads,
                                             0, s>>>(c.a, c.n_a, c.b, c.n, t, list, st);
    else
        dict_insert_kernel<8, kInsThreads><<<stream_grid(c.n, kInsThreads * 8, 512), kInsThreads,
                                             0, s>>>(c.a, c.n_a, c.b, c.n, t, list, st);
    dict_small_kernel<<<kSmallDict / kRankValues, kRankThreads, 0, s>>>(t, list, st, dict);
}

void enqueue_lookup(const Columns &c, const Table &t, unsigned long long limit,
                    const DictState *st, const long long *dict, int *codes_a, int *codes_b,
                    hipStream_t s) {
    if (c.n == 0) return;
    if (c.n <= kMiddle)
        dict_lookup_kernel<1><<<stream_grid(c.n, kLookThreads, 1024), kLookThreads, 0, s>>>(
            c.a, c.n_a, c.b, c.n, dict, t, limit, st, codes_a, codes_b);
    else
        dict_lookup_kernel<8><<<stream_grid(c.n, kLookThreads * 8, 1024), kLookThreads, 0, s>>>(
            c.a, c.n_a, c.b, c.n, dict, t, limit, st, codes_a, codes_b);
}

// Step 4 for k distinct values.
void enqueue_codes(const Columns &c, const Table &t, int64_t k, long long *sorted, DictState *st,
                   long long *dict, int *codes_a, int *codes_b, hipStream_t s) {
    // slots per thread: few enough workgroups that their atomics are not the
    // time, enough of them to fill the chip
    const size_t slots = (size_t)t.mask + 1;
    if (slots <= ((size_t)1 << 20))
        dict_compact_kernel<4><<<(unsigned)((slots + kThreads * 4 - 1) / (kThreads * 4)), kThreads,
                                 0, s>>>(t, sorted, st);
    else
        dict_compact_kernel<32><<<(unsigned)((slots + kThreads * 32 - 1) / (kThreads * 32)),
                                  kThreads, 0, s>>>(t, sorted, st);
    long long *other = reinterpret_cast<long long *>(t.code);  // free until the ranks
    dict_sort_runs_kernel<<<(unsigned)((k + kRunLen - 1) / kRunLen), kSortThreads, 0, s>>>(
        sorted, other, t, st);
    int64_t run = kRunLen;
    for (int p = 0; p < merge_passes(k); ++p, run *= kFan)
        dict_merge_kernel<<<grid_for(k), kThreads, 0, s>>>(sorted, other, run, p, t, st);
    dict_rank_kernel<<<grid_for(k), kThreads, 0, s>>>(sorted, t, st, dict);
    enqueue_lookup(c, t, t.max_count, st, dict, codes_a, codes_b, s);
}

hipError_t read_state(const DictState *st, DictState *host, hipStream_t s) {
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = hipMemcpyAsync(host, st, sizeof(*host), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    return e;
}

}  // namespace

size_t dict_table_slots(int64_t n) {
    size_t slots = 1024;
    while (slots < (size_t)(2 * n)) slots *= 2;
    return slots;
}

size_t dict_workspace_bytes(int64_t n) {
    const size_t slots = dict_table_slots(n);
    // state, table (8 B/slot), slot codes (4 B/slot; also the sort's second
    // buffer), sort buffer (8 B per slot / 2: at most slots / 2 values)
    return align_up(sizeof(DictState)) + align_up(slots * 8) + align_up(slots * 4) +
           align_up(slots / 2 * 8);
}

hipError_t run_dict_encode(const long long *a, int64_t n_a, const long long *b, int64_t n_b,
                           int *codes_a, int *codes_b, long long *dict, int64_t *k_out,
                           void *ws, hipStream_t s) {
    const Columns c{a, b, n_a, n_a + n_b};
    const size_t full = dict_table_slots(c.n);
    char *p = static_cast<char *>(ws);
    DictState *st = reinterpret_cast<DictState *>(p);
    p += align_up(sizeof(DictState));
    auto *table = reinterpret_cast<unsigned long long *>(p);
    p += align_up(full * 8);
    int *slot_code = reinterpret_cast<int *>(p);
    p += align_up(full * 4);
    long long *sorted = reinterpret_cast<long long *>(p);

    DictState host;
    for (int attempt = 0;; ++attempt) {
        const size_t slots = attempt < 2 ? std::min(full, kSmallSlots[attempt]) : full;
        const Table t{table, slot_code, slots - 1,
                      slots == full ? (unsigned long long)full : kSmallProbes, slots / 2};
        // (the list of a small dictionary takes half of the sort buffer's place)
        enqueue_insert(c, t, reinterpret_cast<unsigned int *>(sorted), st, dict, s);
        enqueue_lookup(c, t, kSmallDict, st, dict, codes_a, codes_b, s);
        hipError_t e = read_state(st, &host, s);
        if (e != hipSuccess) return e;
        if (!host.overflow && host.count <= t.max_count && host.count > kSmallDict)
            enqueue_codes(c, t, (int64_t)host.count, sorted, st, dict, codes_a, codes_b, s);
        if (!host.overflow && host.count <= t.max_count) break;
        if (slots == full) return hipErrorUnknown;  // cannot happen by sizing
    }
    *k_out = (int64_t)host.count + (host.has_min ? 1 : 0);
    return hipGetLastError();
}

}  // namespace tcu
