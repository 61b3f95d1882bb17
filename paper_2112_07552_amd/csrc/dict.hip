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
//  2. compact the occupied slots into a list of the distinct values;
//  3. sort that list: chunks of 2048 in LDS, then merges of eight runs at a
//     time, each value finding its place by binary search in the other runs;
//  4. write each distinct value's rank into a code array parallel to the
//     table, then look every record's value up.
// Every kernel reads the number of distinct values from device memory, so
// the whole sequence is enqueued at once and the host waits only at the end,
// for the count it returns.  The first attempt uses a table of at most 2^18
// slots (3 MB with its codes, which an XCD's L2 holds), whatever the column
// length: clearing and scanning a table sized for 2^25 values with 32
// distinct ones took 270 us, with this one 8 us.  When the values do not fit
// (a probe sequence of kSmallProbes slots, or more than half of the slots
// taken) the remaining kernels of the attempt leave at once and the sequence
// runs again, with 2^21 slots and then with twice as many slots as values,
// where every probe sequence meets a free slot.
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
};

// One attempt: the table, the most distinct values it may hold, and the
// probes allowed per value.
struct Table {
    unsigned long long *slot;
    int *code;  // rank of the slot's value
    unsigned long long mask, max_probes, max_count;
};

// What every kernel after the insertion does first: the number of distinct
// values, or 0 when this attempt failed.
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
    }
}

// Both columns, value i of [0, n_a + n_b).  A workgroup remembers values it
// has seen in a direct-mapped LDS array, so a column with few distinct values
// touches the table a few times per workgroup instead of once per record:
// 2^24 values with 32 distinct took 300 us against 46 us here (2.9 TB/s of
// the column).  Columns with many distinct values mostly miss and go to the
// table: 2^25 values with 5000 distinct 584 us for the whole encoding, with
// 32 distinct 222 us (before 1008 and 884 us).
constexpr int kInsThreads = 512;
constexpr int kSeenBits = 12;       // LDS entries: 4096 (32 KB)
constexpr unsigned kSeen = 1u << kSeenBits;

// PER: values per thread and round, loaded together.  Columns too short to
// fill the chip that way take one per thread: a value's probes are a chain of
// memory round trips.
template <int PER>
__global__ void __launch_bounds__(kInsThreads)
dict_insert_kernel(const long long *__restrict__ a, int64_t n_a, const long long *__restrict__ b,
                   int64_t n, Table t, DictState *st) {
    __shared__ unsigned long long seen[kSeen];
    __shared__ unsigned int seen_min, full;
    for (unsigned i = threadIdx.x; i < kSeen; i += kInsThreads) seen[i] = kEmpty;
    if (threadIdx.x == 0) seen_min = full = 0u;
    __syncthreads();
    const int64_t step = (int64_t)gridDim.x * kInsThreads * PER;
    for (int64_t i0 = (int64_t)blockIdx.x * kInsThreads * PER; i0 < n; i0 += step) {
        // the table found full by anyone: leave (one lane asks for all)
        if (threadIdx.x == 0 &&
            __hip_atomic_load(&st->overflow, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
            __hip_atomic_store(&full, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (__hip_atomic_load(&full, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) return;
        unsigned long long v[PER];
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const int64_t i = i0 + j * kInsThreads + threadIdx.x;
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
            unsigned long long *mine = seen + lds_hash(v[j], kSeenBits);
            // An entry holding v was put there by the thread that inserts v:
            // the exchange lets one thread of the workgroup through, so that
            // at the kernel's start not every wave goes to the same few slots
            // (2^25 + 2^24 values, 32 distinct: 139 us; with a plain store
            // after the insertion 527 us)
            if (__hip_atomic_load(mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) == v[j] ||
                atomicExch(mine, v[j]) == v[j])
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
                    if (prev == kEmpty || prev == v[j]) break;
                }
                h = (h + 1) & t.mask;
            }
            if (probe == t.max_probes) atomicOr(&st->overflow, 1u);
        }
    }
}

// The occupied slots as a list, in no particular order.  One atomic per
// workgroup and kThreads * PER slots: atomics on one address are served one
// after the other at about 9 ns each, and one per wave cost 600 us at 2^22
// slots.
template <int PER>
__global__ void __launch_bounds__(kThreads)
dict_compact_kernel(Table t, long long *__restrict__ distinct, DictState *st) {
    __shared__ unsigned int wave_sum[kThreads / 64];
    __shared__ unsigned long long base;
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
        base = all ? atomicAdd(&st->count, (unsigned long long)all) : 0ull;
    }
    __syncthreads();
    unsigned long long at = base + wave_sum[wave] + (incl - mine);
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
            // a wave's 64 pairs at distance j <= 64 are 128 neighbouring
            // values, its own: the workgroup meets only around wider steps
            // (2048 values: 20 us with a barrier after every step)
            if (max(j, j > 1 ? j / 2 : kk) > 64) {
                __syncthreads();
            } else {
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
            }
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

// Codes of both columns.  A dictionary of at most kLdsDict values is put into
// an LDS hash table by each workgroup when the columns are long enough to
// repay it (kLdsMinN): 2^24 records with 32 distinct values 38 us (5.3 TB/s)
// against 72 us through the table in memory.
constexpr int kLookThreads = 512;
constexpr int kLdsDict = 2048;
constexpr int kLdsBits = 12;
constexpr unsigned kLdsSlots = 1u << kLdsBits;  // 32 KB of values, 8 KB of codes
constexpr int64_t kLdsMinN = (int64_t)1 << 19;

template <int PER>
__global__ void __launch_bounds__(kLookThreads)
dict_lookup_kernel(const long long *__restrict__ a, int64_t n_a, const long long *__restrict__ b,
                   int64_t n, const long long *__restrict__ sorted, Table t, const DictState *st,
                   int *__restrict__ codes_a, int *__restrict__ codes_b) {
    __shared__ unsigned long long lv[kLdsSlots];
    __shared__ uint16_t lc[kLdsSlots];
    if (st->overflow || st->count > t.max_count) return;
    const int64_t k = (int64_t)st->count;
    const int shift = st->has_min ? 1 : 0;
    const bool lds = k <= kLdsDict && n >= kLdsMinN;
    if (lds) {
        for (unsigned i = threadIdx.x; i < kLdsSlots; i += kLookThreads) lv[i] = kEmpty;
        __syncthreads();
        for (int r = threadIdx.x; r < (int)k; r += kLookThreads) {
            const unsigned long long v = (unsigned long long)sorted[r];
            // at most half of the slots are taken, so a free one is met
            unsigned h = lds_hash(v, kLdsBits);
            while (atomicCAS(lv + h, kEmpty, v) != kEmpty) h = (h + 1) & (kLdsSlots - 1);
            lc[h] = (uint16_t)(r + shift);
        }
        __syncthreads();
    }
    const int64_t step = (int64_t)gridDim.x * kLookThreads * PER;
    for (int64_t i0 = (int64_t)blockIdx.x * kLookThreads * PER; i0 < n; i0 += step) {
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

// Workgroups of a kernel over the columns: `per` records each, at most four of
// 512 threads per CU (more records then take more rounds).
constexpr int64_t kStreamWgs = 1024;
inline unsigned stream_grid(int64_t n, int per) {
    return (unsigned)std::min<int64_t>(kStreamWgs, (n + per - 1) / per);
}
// columns that one value per thread covers in two rounds
inline bool short_columns(int64_t n) { return n <= 2 * kStreamWgs * kInsThreads; }

struct Columns {
    const long long *a, *b;
    int64_t n_a, n;
};

// Steps 1-2 on one table.
void enqueue_insert(const Columns &c, const Table &t, long long *distinct, DictState *st,
                    hipStream_t s) {
    const size_t slots = (size_t)t.mask + 1;
    const size_t clear_blocks = (slots + kThreads - 1) / kThreads;
    dict_clear_kernel<<<(unsigned)std::min<size_t>(clear_blocks, 65536), kThreads, 0, s>>>(t, st);
    if (c.n > 0 && short_columns(c.n))
        dict_insert_kernel<1><<<stream_grid(c.n, kInsThreads), kInsThreads, 0, s>>>(
            c.a, c.n_a, c.b, c.n, t, st);
    else if (c.n > 0)
        dict_insert_kernel<4><<<stream_grid(c.n, kInsThreads * 4), kInsThreads, 0, s>>>(
            c.a, c.n_a, c.b, c.n, t, st);
    // slots per thread: few enough workgroups that their atomics are not the
    // time, enough of them to fill the chip
    if (slots <= ((size_t)1 << 20))
        dict_compact_kernel<4><<<(unsigned)((slots + kThreads * 4 - 1) / (kThreads * 4)), kThreads,
                                 0, s>>>(t, distinct, st);
    else
        dict_compact_kernel<32><<<(unsigned)((slots + kThreads * 32 - 1) / (kThreads * 32)),
                                  kThreads, 0, s>>>(t, distinct, st);
}

// Steps 3-4 for at most `most` distinct values.
void enqueue_codes(const Columns &c, const Table &t, int64_t most, long long *sorted,
                   const DictState *st, long long *dict, int *codes_a, int *codes_b,
                   hipStream_t s) {
    long long *other = reinterpret_cast<long long *>(t.code);  // free until the ranks
    if (most > 0)
        dict_sort_runs_kernel<<<(unsigned)((most + kRunLen - 1) / kRunLen), kSortThreads, 0, s>>>(
            sorted, other, t, st);
    int64_t run = kRunLen;
    for (int p = 0; p < merge_passes(most); ++p, run *= kFan)
        dict_merge_kernel<<<grid_for(most), kThreads, 0, s>>>(sorted, other, run, p, t, st);
    dict_rank_kernel<<<grid_for(most > 0 ? most : 1), kThreads, 0, s>>>(sorted, t, st, dict);
    if (c.n > 0 && short_columns(c.n))
        dict_lookup_kernel<1><<<stream_grid(c.n, kLookThreads), kLookThreads, 0, s>>>(
            c.a, c.n_a, c.b, c.n, sorted, t, st, codes_a, codes_b);
    else if (c.n > 0)
        dict_lookup_kernel<4><<<stream_grid(c.n, kLookThreads * 4), kLookThreads, 0, s>>>(
            c.a, c.n_a, c.b, c.n, sorted, t, st, codes_a, codes_b);
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
        const int64_t most = std::min<int64_t>(c.n, (int64_t)(slots / 2));
        enqueue_insert(c, t, sorted, st, s);
        hipError_t e = hipSuccess;
        if (attempt < 2) {
            enqueue_codes(c, t, most, sorted, st, dict, codes_a, codes_b, s);
            e = read_state(st, &host, s);
        } else {
            // the sort's grids and passes from the count itself
            e = read_state(st, &host, s);
            if (e == hipSuccess && !host.overflow && host.count <= t.max_count)
                enqueue_codes(c, t, (int64_t)host.count, sorted, st, dict, codes_a, codes_b, s);
        }
        if (e != hipSuccess) return e;
        if (!host.overflow && host.count <= t.max_count) break;
        if (slots == full) return hipErrorUnknown;  // cannot happen by sizing
    }
    *k_out = (int64_t)host.count + (host.has_min ? 1 : 0);
    return hipGetLastError();
}

}  // namespace tcu
