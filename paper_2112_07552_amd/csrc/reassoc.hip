// reassoc.hip -- queries Q3 and Q4 of TCUDB Section 3.3 in re-associated
// form: the group-by SUM (or COUNT) over a join whose left side forms a
// single group.
//
// Lemma Q3 writes the answer as 1^T mat(A) mat(B)^T.  Multiplying the ones
// vector in first turns the left factor into a histogram over join keys,
//   hA[k] = sum of a.val over the A records with key k      (1^T X),
// and the product with B's encoding into one pass over B's records,
//   c[h]  = sum over B records b with group h of hA[b.key] * b.val,
// so neither X nor Y is ever formed: both steps stream over the records
// (HBM-bound), O(n_A + n_B) work instead of O(K N).  Q4 (the aggregate
// without GROUP BY) is the case N = 1 with every B record in group 0.
// COUNT runs alongside with integer histograms, exact.
//
// Both scatters privatise their target array in LDS when it fits (K or N up
// to 2048 entries): each workgroup sums into several copies of every bin, a
// lane's copy given by its number, so that few distinct keys or groups (the
// paper's microbenchmarks use 32) do not meet in one LDS address, and writes
// its bins' sums to its own row of a table that a small kernel adds up in
// order.  One copy per workgroup and global atomics at its end took 101 and 96
// us for 2^24 records with 32 keys and 32 groups, 48 and 40 now (4.2 and 3.4
// TB/s of the columns) and 9 for each table; 10^6 records in 500 groups, where
// the atomics were the time, 51 and now 15 + 5.  More keys
// than that are summed tile by tile (binned.hip) when the workspace has the
// scratch; else, and for more groups, FP64 atomics go to global memory
// directly.  Such sums, and those in LDS, are order-dependent at the last
// bits; counts are exact.
#include <algorithm>

#include "internal.h"

namespace tcu {
namespace {

constexpr int kThreads = 512;
constexpr int kLdsBins = 2048;
constexpr int kPer = 4;           // records per thread and round, loaded together
constexpr int kCopies = 32;       // of a bin, at most
constexpr int kLdsEntries = 2048; // bins times copies: 32 KB, four workgroups per CU
constexpr int kMaxWgs = 1024;

// Copies of each of `bins` bins (a power of two).
__host__ __device__ inline int bin_copies(int bins) {
    int r = kCopies;
    while (r > 1 && r * bins > kLdsEntries) r >>= 1;
    return r;
}

// Rows of the workgroups' table: enough workgroups to fill the chip, each with
// at least 8 records per bin it writes (and that later is read).
inline int table_rows(int64_t n, int bins) {
    const int64_t per = std::max<int64_t>(kThreads * kPer, (int64_t)8 * bins);
    return (int)std::max<int64_t>(1, std::min<int64_t>(kMaxWgs, (n + per - 1) / per));
}

// The workgroup's sums and counts of its bins into its row of the table.
__device__ inline void flush_bins(int bins, int copies, const double *sh,
                                  const unsigned long long *sc, double *tv,
                                  unsigned long long *tc) {
    __syncthreads();
    for (int i = threadIdx.x; i < bins; i += kThreads) {
        double v = 0.0;
        unsigned long long c = 0;
        // copies starting at another one per bin: no two lanes on one bank
        for (int r = 0; r < copies; ++r) {
            const int at = i * copies + ((r + i) & (copies - 1));
            v += sh[at];
            c += sc[at];
        }
        tv[(int64_t)blockIdx.x * bins + i] = v;
        tc[(int64_t)blockIdx.x * bins + i] = c;
    }
}

// out[i] = sum of the table's column i in row order over 32 interleaved shares
// of the rows, then over the shares: the same result on every run.
constexpr int kSumBins = 32, kSumShares = 32;
__global__ void __launch_bounds__(kSumBins * kSumShares)
sum_rows_kernel(int bins, int rows, const double *__restrict__ tv,
                const unsigned long long *__restrict__ tc, double *__restrict__ v,
                unsigned long long *__restrict__ c) {
    __shared__ double sv[kSumShares][kSumBins];
    __shared__ unsigned long long sc[kSumShares][kSumBins];
    const int b = threadIdx.x % kSumBins, share = threadIdx.x / kSumBins;
    const int i = (int)blockIdx.x * kSumBins + b;
    double x = 0.0;
    unsigned long long y = 0;
    if (i < bins)
#pragma unroll 8
        for (int r = share; r < rows; r += kSumShares) {
            x += tv[(int64_t)r * bins + i];
            y += tc[(int64_t)r * bins + i];
        }
    sv[share][b] = x;
    sc[share][b] = y;
    __syncthreads();
    if (share != 0 || i >= bins) return;
    for (int r = 1; r < kSumShares; ++r) {
        x += sv[r][b];
        y += sc[r][b];
    }
    v[i] = x;
    if (c != nullptr) c[i] = y;
}

__device__ inline void report(bool bad, StatusBlock *st, int which) {
    const unsigned long long mask = __ballot(bad);
    if (mask != 0ull && (threadIdx.x & 63) == 0) {
        atomicOr(&st->flags, kFlagKeyRange);
        atomicAdd(which == 0 ? &st->skipped_a : &st->skipped_b,
                  (unsigned long long)__popcll(mask));
    }
}

// hA[key] += val, hc[key] += 1 over A's records (key in [0, K)); PRIV: into
// the workgroup's row of the table (h, hc).
template <typename T, bool PRIV>
__global__ void __launch_bounds__(kThreads)
key_hist_kernel(int64_t n, const int32_t *__restrict__ key, const T *__restrict__ val, int K,
                double *__restrict__ h, unsigned long long *__restrict__ hc, StatusBlock *st) {
    __shared__ double sh[PRIV ? kLdsEntries : 1];
    __shared__ unsigned long long sc[PRIV ? kLdsEntries : 1];
    const int copies = bin_copies(K);
    if (PRIV) {
        for (int i = threadIdx.x; i < K * copies; i += kThreads) { sh[i] = 0.0; sc[i] = 0ull; }
        __syncthreads();
    }
    const int64_t step = (int64_t)gridDim.x * kThreads * kPer;
    const int mine = threadIdx.x & (copies - 1);
    bool bad = false;
    for (int64_t i0 = (int64_t)blockIdx.x * kThreads * kPer; i0 < n; i0 += step) {
        int k[kPer];
        double v[kPer];
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            const int64_t i = i0 + j * kThreads + threadIdx.x;
            const int64_t c = i < n ? i : i0;  // past the end: not used
            k[j] = key[c];
            v[j] = val ? (double)val[c] : 1.0;
        }
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            if (i0 + j * kThreads + threadIdx.x >= n) continue;
            if ((unsigned)k[j] >= (unsigned)K) { bad = true; continue; }
            if (PRIV) {
                atomicAdd(sh + k[j] * copies + mine, v[j]);
                atomicAdd(sc + k[j] * copies + mine, 1ull);
            } else {
                unsafeAtomicAdd(h + k[j], v[j]);
                atomicAdd(hc + k[j], 1ull);
            }
        }
    }
    report(bad, st, 0);
    if (PRIV) flush_bins(K, copies, sh, sc, h, hc);
}

// c[group] += h[key] * val, cnt[group] += hc[key] over B's records; PRIV: into
// the workgroup's row of the table (c, cnt).
template <typename T, bool PRIV>
__global__ void __launch_bounds__(kThreads)
group_sum_kernel(int64_t n, const int32_t *__restrict__ key, const int32_t *__restrict__ grp,
                 const T *__restrict__ val, int K, int N, const double *__restrict__ h,
                 const unsigned long long *__restrict__ hc, double *__restrict__ c,
                 unsigned long long *__restrict__ cnt, StatusBlock *st) {
    __shared__ double sh[PRIV ? kLdsEntries : 1];
    __shared__ unsigned long long sc[PRIV ? kLdsEntries : 1];
    const int copies = bin_copies(N);
    if (PRIV) {
        for (int i = threadIdx.x; i < N * copies; i += kThreads) { sh[i] = 0.0; sc[i] = 0ull; }
        __syncthreads();
    }
    const int64_t step = (int64_t)gridDim.x * kThreads * kPer;
    const int mine = threadIdx.x & (copies - 1);
    bool bad = false;
    for (int64_t i0 = (int64_t)blockIdx.x * kThreads * kPer; i0 < n; i0 += step) {
        int k[kPer], g[kPer];
        double w[kPer], v[kPer];
        unsigned long long m[kPer];
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            const int64_t i = i0 + j * kThreads + threadIdx.x;
            const int64_t at = i < n ? i : i0;  // past the end: not used
            k[j] = key[at];
            g[j] = grp[at];
            w[j] = val ? (double)val[at] : 1.0;
            if (i >= n) g[j] = -1;
            else if ((unsigned)k[j] >= (unsigned)K || (unsigned)g[j] >= (unsigned)N) {
                bad = true;
                g[j] = -1;
            }
        }
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            const int at = g[j] < 0 ? 0 : k[j];
            m[j] = hc[at];
            v[j] = h[at];
        }
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            if (g[j] < 0 || m[j] == 0ull) continue;  // no partner in A
            if (PRIV) {
                atomicAdd(sh + g[j] * copies + mine, v[j] * w[j]);
                atomicAdd(sc + g[j] * copies + mine, m[j]);
            } else {
                unsafeAtomicAdd(c + g[j], v[j] * w[j]);
                atomicAdd(cnt + g[j], m[j]);
            }
        }
    }
    report(bad, st, 1);
    if (PRIV) flush_bins(N, copies, sh, sc, c, cnt);
}

inline unsigned stream_grid(int64_t n) {
    const int64_t per = (int64_t)kThreads * kPer;
    return (unsigned)std::max<int64_t>(1, std::min<int64_t>(1024, (n + per - 1) / per));
}

// The workgroups' table: sums, then counts.
struct Table {
    double *v;
    unsigned long long *c;
};

size_t table_bytes(int bins) {
    return bins <= kLdsBins ? (size_t)kMaxWgs * (size_t)bins * 16 : 0;
}

Table table_at(void *p, int rows, int bins) {
    double *v = static_cast<double *>(p);
    return Table{v, reinterpret_cast<unsigned long long *>(v + (size_t)rows * bins)};
}

hipError_t sum_rows(const Table &t, int bins, int rows, double *v, unsigned long long *c,
                    hipStream_t s) {
    sum_rows_kernel<<<(unsigned)((bins + kSumBins - 1) / kSumBins), kSumBins * kSumShares, 0, s>>>(
        bins, rows, t.v, t.c, v, c);
    return hipGetLastError();
}

hipError_t zero_bins(int bins, double *v, unsigned long long *c, hipStream_t s) {
    hipError_t e = launch_zero_f64(v, (size_t)bins, s);
    if (e == hipSuccess) e = launch_zero_f64(reinterpret_cast<double *>(c), (size_t)bins, s);
    return e;
}

template <typename T>
hipError_t hist_t(const tcu_relation &R, int K, double *h, unsigned long long *hc, void *table,
                  StatusBlock *st, hipStream_t s) {
    const T *v = static_cast<const T *>(R.val);
    if (K <= kLdsBins) {
        const int rows = table_rows(R.n, K);
        const Table t = table_at(table, rows, K);
        key_hist_kernel<T, true><<<(unsigned)rows, kThreads, 0, s>>>(R.n, R.key, v, K, t.v, t.c,
                                                                     st);
        const hipError_t e = hipGetLastError();
        return e == hipSuccess ? sum_rows(t, K, rows, h, hc, s) : e;
    }
    const hipError_t e = zero_bins(K, h, hc, s);
    if (e != hipSuccess || R.n == 0) return e;
    key_hist_kernel<T, false><<<stream_grid(R.n), kThreads, 0, s>>>(R.n, R.key, v, K, h, hc, st);
    return hipGetLastError();
}

template <typename T>
hipError_t group_t(const tcu_relation &R, int K, int N, const double *h,
                   const unsigned long long *hc, double *c, unsigned long long *cnt, void *table,
                   StatusBlock *st, hipStream_t s) {
    const T *v = static_cast<const T *>(R.val);
    if (N <= kLdsBins) {
        const int rows = table_rows(R.n, N);
        const Table t = table_at(table, rows, N);
        group_sum_kernel<T, true><<<(unsigned)rows, kThreads, 0, s>>>(R.n, R.key, R.group, v, K, N,
                                                                      h, hc, t.v, t.c, st);
        const hipError_t e = hipGetLastError();
        return e == hipSuccess ? sum_rows(t, N, rows, c, cnt, s) : e;
    }
    const hipError_t e = zero_bins(N, c, cnt, s);
    if (e != hipSuccess || R.n == 0) return e;
    group_sum_kernel<T, false><<<stream_grid(R.n), kThreads, 0, s>>>(R.n, R.key, R.group, v, K, N,
                                                                     h, hc, c, cnt, st);
    return hipGetLastError();
}

}  // namespace

// status block, histogram (sums and counts), B's counts where the caller takes
// none, and the larger of the two tables
size_t row_workspace_bytes(int K, int N) {
    return sizeof(StatusBlock) + align_up((size_t)K * 8) + align_up((size_t)K * 8) +
           align_up((size_t)N * 8) + align_up(std::max(table_bytes(K), table_bytes(N)));
}

size_t row_scratch_bytes(const tcu_relation &A, int K) {
    return K > kLdsBins ? binned_hist_scratch_bytes(A, K) : 0;
}

hipError_t run_join_agg_row(const tcu_relation &A, const tcu_relation &B, int K, int N, double *c,
                            unsigned long long *count, void *ws, size_t ws_bytes, hipStream_t s) {
    char *p = static_cast<char *>(ws);
    StatusBlock *st = reinterpret_cast<StatusBlock *>(p);
    p += sizeof(StatusBlock);
    double *h = reinterpret_cast<double *>(p);
    p += align_up((size_t)K * 8);
    auto *hc = reinterpret_cast<unsigned long long *>(p);
    p += align_up((size_t)K * 8);
    auto *cnt = count ? count : reinterpret_cast<unsigned long long *>(p);
    p += align_up((size_t)N * 8);
    hipError_t e = launch_clear_status(st, s);
    if (e != hipSuccess) return e;
    const size_t base = row_workspace_bytes(K, N), bin = row_scratch_bytes(A, K);
    if (bin > 0 && ws_bytes >= base + bin)
        e = launch_binned_hist(A, K, h, hc, st, static_cast<char *>(ws) + base, s);
    else
        e = A.dtype == TCU_F32 ? hist_t<float>(A, K, h, hc, p, st, s)
                               : hist_t<double>(A, K, h, hc, p, st, s);
    if (e != hipSuccess) return e;
    return B.dtype == TCU_F32 ? group_t<float>(B, K, N, h, hc, c, cnt, p, st, s)
                              : group_t<double>(B, K, N, h, hc, c, cnt, p, st, s);
}

}  // namespace tcu
