// Per-filter optimal split: alpha, beta, K and the split descriptor (gfx950).
//
// Theorem 2 and Algorithm 1 of arXiv 1804.02941 (Sections 4.1, 4.3.1): sort the n weights
// of a filter, take prefix sums P_i, score every split with
//   D_i = P_i^2 / i + (T - P_i)^2 / (n - i),   i = 1 .. n-1,
// and keep the largest i of maximal D.  The two groups' means are alpha and beta.
// Section 4.3.1 handles all filters of a layer together; here a filter is a segment and
// one workgroup owns one segment, so the sorted row, P and D never leave the chip:
//
//   1. load the row, map fp32 -> order-preserving uint32 keys (-0.0 folded onto +0.0), pad
//      to THREADS * ITEMS keys with 0xFFFFFFFF (above every finite key);
//   2. least-significant-digit radix sort in LDS, 8 passes of 4 bits.  A thread owns ITEMS
//      consecutive keys and holds them in registers for the whole pass; its sixteen digit
//      counters (each at most ITEMS <= 15) live in one 64-bit register, 4 bits apiece, so
//      counting costs no memory traffic.  The counters go to LDS packed two to a word
//      (digit d and d + 8), one scan over the words in (digit, thread) order turns them
//      into stable offsets, and the keys are scattered back into the same buffer;
//   3. fp64 prefix sums (serial per thread, scanned across threads) and the arg-max of D_i,
//      compared as fractions (numerators cross-multiplied) so that no division is needed
//      per element; ties prefer the larger i;
//   4. the split descriptor: the value at the split and, among equal values, the original
//      index up to which they belong to the lower group (recovered from the unsorted row,
//      so the sort itself carries no indices).
//
// Rows (but for many of at most 192 weights) first go through a search that needs no full sort (bucket_row in
// estimate_rows.h, beside the sort: value buckets with exact sums, a bound on D inside every bucket,
// exact ranking of the few elements that can hold the arg-max), and only rows it cannot finish are
// sorted: by the same workgroup for rows below 4096 weights (one launch), and for longer rows by
// the sort kernel launched behind, which then only works on the rows handed over (and does every
// row when the caller gives no workspace for the hand-over flags).  This file holds the kernels
// around the two row procedures, the calls that take the filters of several layers at once (and pack
// each filter's mask, and in workgroups of their own the layers' activations, in the same launches) and the host side.
#include "dab_internal.h"

#include "estimate_rows.h"
#include "pack_act.h"
#include "pack_mask.h"

namespace dab {

// Long rows: a flag per row for the sort kernel launched behind.
template <int THREADS, int ITEMS, int NB, int CAP>
__global__ __launch_bounds__(THREADS) void estimate_bucket_kernel(const float* __restrict__ Wt, int n,
                                                                  float* __restrict__ alpha, float* __restrict__ beta,
                                                                  int32_t* Kout, float* __restrict__ thr_val,
                                                                  int32_t* __restrict__ thr_idx, uint8_t* alpha_is_upper,
                                                                  const int32_t* K_prev, const uint8_t* upper_prev,
                                                                  int max_change, uint8_t* __restrict__ fallback) {
    DAB_RESERVE_VGPRS();
    const int f = static_cast<int>(blockIdx.x);
    float x[ITEMS];
    load_row<THREADS, ITEMS>(Wt + static_cast<size_t>(f) * n, n, x);
    const bool done = bucket_row<THREADS, ITEMS, NB, CAP>(x, n, f, alpha, beta, Kout, thr_val, thr_idx, alpha_is_upper,
                                                          K_prev, upper_prev, max_change);
    if (threadIdx.x == 0) fallback[f] = done ? 0 : 1;
}

// Short rows: a row the buckets cannot finish is sorted by the same workgroup, so one launch does the
// layer.
template <int THREADS, int ITEMS, int NB, int CAP>
__global__ __launch_bounds__(THREADS) void estimate_short_kernel(const float* __restrict__ Wt, int n,
                                                                 float* __restrict__ alpha, float* __restrict__ beta,
                                                                 int32_t* Kout, float* __restrict__ thr_val,
                                                                 int32_t* __restrict__ thr_idx, uint8_t* alpha_is_upper,
                                                                 const int32_t* K_prev, const uint8_t* upper_prev,
                                                                 int max_change) {
    DAB_RESERVE_VGPRS();
    const int f = static_cast<int>(blockIdx.x);
    float x[ITEMS];
    load_row<THREADS, ITEMS>(Wt + static_cast<size_t>(f) * n, n, x);
    if (bucket_row<THREADS, ITEMS, NB, CAP, 1>(x, n, f, alpha, beta, Kout, thr_val, thr_idx, alpha_is_upper, K_prev, upper_prev,
                                            max_change))
        return;
    __syncthreads();
    sort_row<THREADS, ITEMS>(Wt, n, f, alpha, beta, Kout, thr_val, thr_idx, alpha_is_upper, K_prev, upper_prev, max_change);
}

// ---------------------------------------------------------------- estimation and packing of several layers
// Section 4.3.1 treats all filters of a layer at once; nothing ties a filter to its layer, so the
// filters of several layers can share a launch, and the mask of a filter (Corollary 1) can be packed
// by the workgroup that has just found its split, while the row is still in L2: the weights are
// read from memory once, and a network's weight side is two or three launches whatever its depth.
constexpr int kMaxEstJobs = 16;
constexpr int kSortRowsPerGroup = 8;               // rows a workgroup of the sort kernel looks after
struct EstJob {
    const float* W;
    float* alpha; float* beta; int32_t* K; float* thr_val; int32_t* thr_idx; uint8_t* aiu;
    const int32_t* K_prev; const uint8_t* upper_prev;
    MaskShape mask;                                // where the packed mask goes (E and ecnt nullptr: nowhere)
    uint8_t* flags;                                // long rows: one hand-over flag per filter
    int n, F, max_change;
    unsigned blk_end;                              // first workgroup past this job's range
};
struct EstJobs {
    int n;
    EstJob job[kMaxEstJobs];
};

__device__ __forceinline__ const EstJob& find_job(const EstJobs& jobs, unsigned block, unsigned* blk0) {
    int j = 0;
    *blk0 = 0;
    while (j + 1 < jobs.n && block >= jobs.job[j].blk_end) *blk0 = jobs.job[j++].blk_end;
    return jobs.job[j];
}

// Rows of up to THREADS * ITEMS weights, one per workgroup: buckets first; where they cannot finish
// the row, the sort by the same workgroup (SORT_HERE) or a flag for the sort kernel launched
// behind; then the packing.
// (The pool is declared in a function of its own, so that two classes of rows in one kernel share it.)
template <int THREADS, int ITEMS, int NB, int CAP>
constexpr size_t kRowPool = sizeof(BucketLds<THREADS, NB, CAP>) > THREADS * ITEMS ? sizeof(BucketLds<THREADS, NB, CAP>) : THREADS * ITEMS;
template <size_t BYTES>
__device__ __forceinline__ unsigned char* row_pool() {
    __shared__ __align__(16) unsigned char pool[BYTES];
    return pool;
}
template <int THREADS, int ITEMS, int NB, int CAP, bool SORT_HERE, size_t POOL = kRowPool<THREADS, ITEMS, NB, CAP>>
__device__ __forceinline__ void binarize_row_of_block(const EstJobs& jobs, unsigned block) {
    using Lds = BucketLds<THREADS, NB, CAP>;
    unsigned char* const pool = row_pool<POOL>();                  // the search's arrays, then the mask, a byte per weight
    __shared__ SplitInfo info;
    unsigned blk0;
    const EstJob& q = find_job(jobs, block, &blk0);
    const int f = column_of_block(block - blk0, q.mask.Fp);
    if (f >= q.mask.Fp) return;
    float x[ITEMS];
    bool done = true;
    if (f < q.F) {
        load_row<THREADS, ITEMS>(q.W + static_cast<size_t>(f) * q.n, q.n, x);
        done = bucket_row<THREADS, ITEMS, NB, CAP, SORT_HERE ? 1 : kMaxLists>(*reinterpret_cast<Lds*>(pool), x, q.n, f, q.alpha, q.beta, q.K, q.thr_val,
                                                   q.thr_idx, q.aiu, q.K_prev, q.upper_prev, q.max_change, &info);
        if constexpr (SORT_HERE) {
            if (!done) {
                __syncthreads();
                sort_row<THREADS, ITEMS>(q.W, q.n, f, q.alpha, q.beta, q.K, q.thr_val, q.thr_idx, q.aiu, q.K_prev, q.upper_prev,
                                         q.max_change, &info);
                done = true;
            }
        } else if (threadIdx.x == 0) {
            q.flags[f] = done ? 0 : 1;
        }
        lds_barrier();
    }
    if (q.mask.E && f >= q.F) {
        pack_padding<THREADS>(q.mask, f);
    } else if (q.mask.E && done) {
        pack_row<THREADS, ITEMS>(q.mask, f, info, x, pool);
    }
}

// The weight side of the layers in `jobs`, and beside it a share of the activation packing in
// `packs`.  The two do not depend on each other and load different parts of the chip: the estimation is
// bound by vector instructions and LDS, the packing by memory, so the launch's first n_pack workgroups
// pack and the others take a row each: every compute unit holds wavefronts of both kinds, and the memory
// stream of the ones runs under the arithmetic of the others.  (Config 3 at batch 256, inputs not in the
// caches: packing alone 43 us, weight sides alone 35.5, together 56.5; with a row and then a share of the
// packing in every workgroup, half of them the other way round, 64.3.)
// Across launches on different streams this overlap does not happen (measured: the times add up).
template <int THREADS, int ITEMS, int NB, int CAP, bool SORT_HERE, int MIN_WAVES>
__global__ __launch_bounds__(THREADS, MIN_WAVES) void binarize_rows_kernel(const EstJobs jobs) {
    DAB_RESERVE_VGPRS();
    binarize_row_of_block<THREADS, ITEMS, NB, CAP, SORT_HERE>(jobs, blockIdx.x);
}
template <int THREADS, int ITEMS, int NB, int CAP, bool SORT_HERE, int MIN_WAVES>
__global__ __launch_bounds__(THREADS, MIN_WAVES) void prepare_rows_kernel(const EstJobs jobs, const PackJobs packs, unsigned n_pack) {
    DAB_RESERVE_VGPRS();
    if (blockIdx.x < n_pack) pack_share<THREADS / 64>(packs, blockIdx.x);
    else binarize_row_of_block<THREADS, ITEMS, NB, CAP, SORT_HERE>(jobs, blockIdx.x - n_pack);
}

// Long rows, a row of up to 2304 weights each for the workgroups behind them, and in front of both the packing, in one launch:
// the short rows run where long ones leave compute units, instead of before them.  The long rows' registers leave
// room for four workgroups on a compute unit where the short ones alone would have seven, which pays while those are few.  (The trunk of the
// sketch network with its packing: batch 1 36.0 -> 30.5 us, 32 39.9 -> 33.5, 128 48.4 -> 41.5, 192 (180 MB) 51.7 -> 48.3; at 256, 240 MB, memory decides: 56.1 and 56.2, two launches.)
template <int ITEMS, int NB, int CAP>
__global__ __launch_bounds__(256, 4) void prepare_two_kernel(const EstJobs jobs, const PackJobs packs, unsigned n_pack, unsigned n_long) {
    DAB_RESERVE_VGPRS();
    constexpr size_t kLong = kRowPool<256, ITEMS, NB, CAP>, kShort = kRowPool<256, 9, 512, 256>, kPool = kLong > kShort ? kLong : kShort;
    if (blockIdx.x < n_pack) pack_share<4>(packs, blockIdx.x);
    else if (blockIdx.x < n_pack + n_long) binarize_row_of_block<256, ITEMS, NB, CAP, false, kPool>(jobs, blockIdx.x - n_pack);
    else binarize_row_of_block<256, 9, 512, 256, false, kPool>(jobs, blockIdx.x - n_pack);
}

// The rows the kernels above have flagged, kSortRowsPerGroup per workgroup.  Their flags are one aligned 8-byte
// read: the flags of all jobs are one array, each job's part padded to a multiple of 256 bytes.  That read comes
// first, since as a rule nothing is flagged and the launch is only what it takes to see that.
template <int THREADS, int ITEMS>
__global__ __launch_bounds__(THREADS) void binarize_sort_kernel(const uint8_t* flags, const EstJobs jobs) {
    static_assert(kSortRowsPerGroup == 8, "the flags of a workgroup's rows are read as one 64-bit word");
    unsigned long long fl = reinterpret_cast<const unsigned long long*>(flags)[blockIdx.x];
    if (fl == 0ull) return;                         // the bucket kernel has finished all of them
    __shared__ SplitInfo info;
    unsigned blk0;
    const EstJob& q = find_job(jobs, blockIdx.x, &blk0);
    const int f0 = static_cast<int>(blockIdx.x - blk0) * kSortRowsPerGroup;
    if (f0 >= q.F) return;                          // (padding: whatever the workspace held)
    if (f0 + kSortRowsPerGroup > q.F) fl &= (1ull << (8 * (q.F - f0))) - 1ull;     // rows past the last one are not ours
    if (fl == 0ull) return;
    for (int k = 0; k < kSortRowsPerGroup; ++k) {
        if (((fl >> (8 * k)) & 0xFFull) == 0ull) continue;
        const int f = f0 + k;
        sort_row<THREADS, ITEMS>(q.W, q.n, f, q.alpha, q.beta, q.K, q.thr_val, q.thr_idx, q.aiu, q.K_prev, q.upper_prev,
                                 q.max_change, &info);
        __syncthreads();
        if (q.mask.E) pack_row_from<THREADS, THREADS * ITEMS>(q.mask, f, info, q.W + static_cast<size_t>(f) * q.n);
        __syncthreads();
    }
}

// ---------------------------------------------------------------- sign split (XNOR-Net / BWN)
// The distribution-agnostic special case of Section 4.1: e = [w >= 0], alpha = mean |w|, beta = -alpha.
// One workgroup per filter, plain reductions; the outputs have the form of the estimator's, so the
// same weight packing and layer kernels consume them.
__global__ __launch_bounds__(256) void sign_split_kernel(const float* __restrict__ Wt, int n, float* __restrict__ alpha,
                                                         float* __restrict__ beta, int32_t* __restrict__ Kout,
                                                         float* __restrict__ thr_val, int32_t* __restrict__ thr_idx,
                                                         uint8_t* __restrict__ alpha_is_upper) {
    __shared__ double s_abs[4];
    __shared__ int s_cnt[4];
    __shared__ float s_max[4];
    __shared__ int s_idx[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const float* row = Wt + static_cast<size_t>(blockIdx.x) * n;
    double a = 0.0;
    int cnt = 0, idx = 0;
    float vmax = -INFINITY;                                   // largest negative value and its last index
    for (int i = tid; i < n; i += 256) {
        const float w = row[i];
        a += fabs(static_cast<double>(w));
        if (w >= 0.0f) {
            ++cnt;
        } else if (w > vmax || (w == vmax && i > idx)) {
            vmax = w;
            idx = i;
        }
    }
    for (int d = 32; d >= 1; d >>= 1) {
        a += __shfl_xor(a, d, 64);
        cnt += __shfl_xor(cnt, d, 64);
        const float ov = __shfl_xor(vmax, d, 64);
        const int oi = __shfl_xor(idx, d, 64);
        if (ov > vmax || (ov == vmax && oi > idx)) { vmax = ov; idx = oi; }
    }
    if (lane == 0) { s_abs[wave] = a; s_cnt[wave] = cnt; s_max[wave] = vmax; s_idx[wave] = idx; }
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < 4; ++w) {
            a += s_abs[w];
            cnt += s_cnt[w];
            if (s_max[w] > vmax || (s_max[w] == vmax && s_idx[w] > idx)) { vmax = s_max[w]; idx = s_idx[w]; }
        }
        const int f = blockIdx.x;
        const float al = static_cast<float>(a / static_cast<double>(n));
        alpha[f] = al;
        beta[f] = -al;
        Kout[f] = cnt;
        thr_val[f] = vmax;
        thr_idx[f] = vmax == -INFINITY ? 0 : idx;
        alpha_is_upper[f] = 1;
    }
}

constexpr int kEstimateMaxN = 1024 * 13;

constexpr int kBucketMinN = 4096;        // rows from here on: bucket kernel, then the sort kernel for the rows it flags
constexpr int kSortMaxN = 192;           // rows up to here, where there are many: the sort kernel

static size_t estimate_ws_bytes(int F, int n) {
    return n >= kBucketMinN ? (static_cast<size_t>(F) + 255) & ~static_cast<size_t>(255) : 0;
}

// Smallest padded size that holds the row; odd item counts keep the per-thread key runs off each
// other's LDS banks.
static int dispatch_estimate(const float* W, int F, int n, float* alpha, float* beta, int32_t* K, float* thr_val,
                             int32_t* thr_idx, uint8_t* aiu, const int32_t* K_prev, const uint8_t* upper_prev,
                             int max_change, void* ws, size_t ws_bytes, hipStream_t st) {
    // With a workspace for the per-row flags, the bucket kernel goes first and the sort kernel only
    // works on the rows it hands over; without one the sort kernel does every row.
    uint8_t* only = nullptr;
    if (n >= kBucketMinN && ws && ws_bytes >= estimate_ws_bytes(F, n)) {
        only = static_cast<uint8_t*>(ws);
        // (few long rows: eight wavefronts finish a row sooner, four finish more rows in the same time: 12544 weights, 512 rows
        // 16.3 us and 17.1, 1024 rows 27.4 and 26.3, 4096 rows 75.8 and 70.5)
        const int rc = n <= 256 * 18
            ? launch(estimate_bucket_kernel<256, 18, 1024, 256>, dim3(F), dim3(256), 0, st, W, n, alpha, beta, K, thr_val,
                     thr_idx, aiu, K_prev, upper_prev, max_change, only)
            : n <= 256 * 36
            ? launch(estimate_bucket_kernel<256, 36, 2048, 256>, dim3(F), dim3(256), 0, st, W, n, alpha, beta, K, thr_val,
                     thr_idx, aiu, K_prev, upper_prev, max_change, only)
            : F <= 2 * kNumCU
            ? launch(estimate_bucket_kernel<512, 26, 2048, 512>, dim3(F), dim3(512), 0, st, W, n, alpha, beta, K, thr_val,
                     thr_idx, aiu, K_prev, upper_prev, max_change, only)
            : launch(estimate_bucket_kernel<256, 52, 2048, 256>, dim3(F), dim3(256), 0, st, W, n, alpha, beta, K, thr_val,
                     thr_idx, aiu, K_prev, upper_prev, max_change, only);
        if (rc) return rc;
    }
    // shorter rows: one launch, buckets first and the sort inside the kernel where needed.  A wavefront per row sorts the
    // shortest rows; with a workgroup per row the search is faster until the rows fill the chip several times (64 weights:
    // 64 rows 5.9 us and 8.4 sorted, 512 rows 6.5 and 9.0, 4096 rows 20.2 and 14.0).
#define DAB_SHORT(T, I, NB) \
    return launch(estimate_short_kernel<T, I, NB, 256>, dim3(F), dim3(T), 0, st, W, n, alpha, beta, K, thr_val, thr_idx, \
                  aiu, K_prev, upper_prev, max_change)
    if (n < kBucketMinN && (n > kSortMaxN || F <= 6 * kNumCU)) {
        if (n <= 256 * 3) DAB_SHORT(256, 3, 512);
        if (n <= 256 * 5) DAB_SHORT(256, 5, 1024);
        if (n <= 256 * 7) DAB_SHORT(256, 7, 1024);
        if (n <= 256 * 9) DAB_SHORT(256, 9, 1024);
        if (n <= 256 * 11) DAB_SHORT(256, 11, 1024);
        if (n <= 512 * 7) DAB_SHORT(512, 7, 2048);
        DAB_SHORT(512, 9, 2048);
    }
#undef DAB_SHORT
#define DAB_EST(T, I) \
    return launch(estimate_kernel<T, I>, dim3(F), dim3(T), 0, st, W, n, alpha, beta, K, thr_val, thr_idx, aiu, K_prev, \
                  upper_prev, max_change, only)
    if (n <= kSortMaxN) DAB_EST(64, 3);
    if (n <= 512 * 9) DAB_EST(512, 9);
    if (n <= 512 * 11) DAB_EST(512, 11);
    if (n <= 1024 * 7) DAB_EST(1024, 7);
    if (n <= 1024 * 9) DAB_EST(1024, 9);
    if (n <= 1024 * 11) DAB_EST(1024, 11);
    DAB_EST(1024, 13);
#undef DAB_EST
}

// ---------------------------------------------------------------- host side of the multi-layer call
constexpr int kSmallMaxN = 256 * 9;                // rows up to here: 256 threads and 512 buckets per row
constexpr int kShortMaxN = 512 * 9;                // rows up to here: 512 threads x 9 and 2048 buckets, sorted in the same kernel if need be (or 256 x 18 and 1024 buckets, handed over)
constexpr int kMidMaxN = 512 * 18;                 // rows up to here: 18 weights per thread, longer ones 26; both hand rows over to the sort kernel

static int check_weight_job(const dab_weight_job& j) {
    if (!j.W || !j.alpha || !j.beta || !j.K || !j.thr_val || !j.thr_idx || !j.alpha_is_upper) return DAB_ERR_NULL;
    if ((j.E_packed == nullptr) != (j.ecnt == nullptr)) return DAB_ERR_NULL;
    if ((j.K_prev == nullptr) != (j.alpha_is_upper_prev == nullptr)) return DAB_ERR_NULL;
    if (j.F < 1 || j.C < 1 || j.kh < 1 || j.kw < 1 || 1ll * j.C * j.kh * j.kw < 2 || (j.K_prev && j.max_change < 0))
        return DAB_ERR_SHAPE;
    if (misaligned(j.W, 4) || misaligned(j.alpha, 4) || misaligned(j.beta, 4) || misaligned(j.K, 4) || misaligned(j.thr_val, 4) ||
        misaligned(j.thr_idx, 4) || (j.E_packed && (misaligned(j.E_packed, 64) || misaligned(j.ecnt, 4))) ||
        (j.K_prev && misaligned(j.K_prev, 4)))
        return DAB_ERR_ALIGN;
    if (1ll * j.C * j.kh * j.kw > kEstimateMaxN) return DAB_ERR_UNSUPPORTED;
    if (j.E_packed && j.kh * j.kw > kPackMaxTaps) return DAB_ERR_UNSUPPORTED;
    return DAB_OK;
}

// Rows up to 4608 weights can be finished in one launch: the workgroup that cannot finish a row with
// the buckets sorts it itself.  Flagging such rows for the sort kernel instead frees the LDS of the
// in-kernel sort, and more workgroups share a compute unit: seven instead of five of the 256-thread
// kernel; the rows of 2305 .. 4608 weights then take 256 threads with eighteen elements each and
// 1024 buckets, six workgroups per compute unit instead of the two of the 512-thread kernel that can
// sort (4096 rows of 4096 weights: 63 us instead of 85; these kernels are bound by the latency of a
// row's chain of phases, so rows in flight count).  That is done where it pays for the extra launch:
// for a class with many rows, and for the short rows whenever the sort kernel is launched anyway.
struct HandOver {
    bool small, medium;        // rows up to 2304 weights, rows of 2305 .. 4608
};
static HandOver hand_over_plan(const dab_weight_job* jobs, int n_jobs) {
    long long small = 0, medium = 0, longer = 0;
    for (int i = 0; i < n_jobs; ++i) {
        const long long n = 1ll * jobs[i].C * jobs[i].kh * jobs[i].kw;
        (n <= kSmallMaxN ? small : (n <= kShortMaxN ? medium : longer)) += jobs[i].F;
    }
    HandOver h;
    h.medium = medium >= 6 * kNumCU;
    h.small = small >= 6 * kNumCU || (small > 0 && (longer > 0 || h.medium));
    return h;
}

// Hand-over flags of a job with F filters.
static size_t flag_bytes(int F) { return (static_cast<size_t>(F) + 255) & ~static_cast<size_t>(255); }

static size_t weight_jobs_ws_bytes(const dab_weight_job* jobs, int n_jobs) {
    size_t total = 0;
    const HandOver h = hand_over_plan(jobs, n_jobs);
    for (int i = 0; i < n_jobs; ++i) {
        const long long n = 1ll * jobs[i].C * jobs[i].kh * jobs[i].kw;
        if (n > kShortMaxN || (n > kSmallMaxN ? h.medium : h.small))
            total += flag_bytes(jobs[i].F);
    }
    return total;
}

// Duration of a class's launch by its rows, in us (measured on MI355X over 256 to 4096 rows), for dealing
// the activation packing out over the launches.
static double rows_us(int c, long long rows) {
    constexpr double kLaunch[4] = {6.0, 6.0, 8.0, 8.0}, kRow[4] = {0.0045, 0.0062, 0.0100, 0.0135};
    return rows > 0 ? kLaunch[c] + kRow[c] * static_cast<double>(rows) : 0.0;
}

constexpr double kWidePackBytes = 8e7;
constexpr int kTogetherRows = 20 * kNumCU;         // short and long rows, up to these many, in one launch,
constexpr double kTogetherPackBytes = 2e8;         // beside up to this much packing

static int run_weight_jobs(const dab_weight_job* jobs, int n_jobs, void* ws, size_t ws_bytes, hipStream_t st,
                           const dab_pack_job* packs = nullptr, int n_packs = 0) {
    // four classes of rows, a launch each where present, and one behind them for the rows they flag
    constexpr int kClasses = 4;
    EstJobs cls[kClasses], sortj;
    unsigned end[kClasses] = {0, 0, 0, 0}, sort_end = 0;
    long long rows[kClasses] = {0, 0, 0, 0};
    for (int c = 0; c < kClasses; ++c) cls[c].n = 0;
    sortj.n = 0;
    uint8_t* flags = static_cast<uint8_t*>(ws);
    const HandOver hand = hand_over_plan(jobs, n_jobs);
    for (int i = 0; i < n_jobs; ++i) {
        const dab_weight_job& in = jobs[i];
        EstJob q{};
        q.W = in.W; q.alpha = in.alpha; q.beta = in.beta; q.K = in.K; q.thr_val = in.thr_val; q.thr_idx = in.thr_idx;
        q.aiu = in.alpha_is_upper; q.K_prev = in.K_prev; q.upper_prev = in.alpha_is_upper_prev; q.max_change = in.max_change;
        q.F = in.F;
        q.mask = make_mask_shape(in.E_packed, in.ecnt, in.F, in.C, in.kh * in.kw);
        q.n = q.mask.n;
        const unsigned columns = static_cast<unsigned>(kNumXCD * ceil_div(q.mask.Fp, kNumXCD));
        const int c = q.n <= kSmallMaxN ? 0 : (q.n <= kShortMaxN ? 1 : (q.n <= kMidMaxN ? 2 : 3));
        const bool flagged = c >= 2 || (c == 1 ? hand.medium : hand.small);
        if (flagged) {
            q.flags = flags;
            flags += flag_bytes(in.F);
        }
        end[c] += columns;
        rows[c] += in.F;
        q.blk_end = end[c];
        cls[c].job[cls[c].n++] = q;
        if (flagged) {
            sort_end += static_cast<unsigned>(flag_bytes(in.F) / kSortRowsPerGroup);
            q.blk_end = sort_end;
            sortj.job[sortj.n++] = q;
        }
    }
    (void)ws_bytes;
    // Short rows beside long ones: in the long ones' launch while they are few (both hand rows over to the sort kernel then).
    // (us, two launches | one: 512 rows of 1152 weights and 256 of 8192 22.6 | 14.9, 1536 of 2304 and 512 of 12544 37.0 | 32.2, 512 of
    // 1152 and 2048 of 9216 45.9 | 40.3, 4096 of 288 and 512 of 12544 44.7 | 44.2; 2048 of 1152 and 4096 of 5000 64.4 | 65.2,
    // 4096 of 2304 and 4096 of 5000 77.9 | 80.2.)
    const int longest = rows[3] ? 3 : 2;
    const unsigned n_long = end[longest];
    double pack_bytes = 0.0;
    for (int i = 0; i < n_packs; ++i) pack_bytes += 4.0 * packs[i].B * packs[i].H * packs[i].W * packs[i].C;
    const bool together = rows[0] > 0 && rows[longest] > 0 && rows[0] + rows[longest] <= kTogetherRows && pack_bytes < kTogetherPackBytes;
    if (together) {
        for (int i = 0; i < cls[0].n; ++i) {
            EstJob q = cls[0].job[i];
            q.blk_end += end[longest];
            cls[longest].job[cls[longest].n++] = q;
        }
        end[longest] += end[0];
        cls[0].n = 0;
    }
    // the activation packing, dealt out over the launches in proportion to their duration: every tensor's
    // pixels are cut at the same fractions
    PackJobs pk[kClasses];
    unsigned n_pack[kClasses] = {0, 0, 0, 0};
    double us[kClasses], total = 0.0;
    for (int c = 0; c < kClasses; ++c) {
        pk[c].n = 0;
        us[c] = together && c == 0 ? 0.0 : rows_us(c, rows[c]);
        total += us[c];
    }
    // Rows of 9217 .. 13312 weights: 512 threads finish a row sooner, 256 finish more rows in the same time and leave
    // room for packing workgroups: 512 rows 18.5 us and 19.3, 1024 rows 30.5 and 28.4, 4096 rows 83.8 and 75.3; the
    // rows of config 3 with its packing at batch 32 (30 MB) 40.1 and 41.9, at 96 45.6 and 46.0, at 128 (120 MB) 50.7 and
    // 48.2, at 256 62.7 and 55.8.
    const bool wide = rows[3] <= 2 * kNumCU && pack_bytes < kWidePackBytes && !together;
    const int class_waves[kClasses] = {4, hand.medium ? 4 : 8, 4, wide ? 8 : 4};   // (wavefronts of the class's workgroups)
    double done = 0.0;
    for (int c = 0; c < kClasses && n_packs > 0; ++c) {
        if (us[c] <= 0.0) continue;
        const double lo = done / total, hi = (done + us[c]) / total;
        done += us[c];
        for (int i = 0; i < n_packs; ++i) {
            const long long pixels = 1ll * packs[i].B * packs[i].H * packs[i].W;
            const long long p0 = static_cast<long long>(lo * static_cast<double>(pixels));
            const long long p1 = done >= total ? pixels : static_cast<long long>(hi * static_cast<double>(pixels));
            if (p1 > p0) pk[c].job[pk[c].n++] = make_pack_job(packs[i], p0, p1);
        }
        // eight wavefronts of packing per compute unit beside the rows' (four: 59.8 us for config 3 at batch 256, eight 56.5,
        // twelve 56.4)
        if (pk[c].n) n_pack[c] = share_pack_blocks(&pk[c], 8 * kNumCU / class_waves[c], class_waves[c]);
    }
#define DAB_ROWS(C, T, I, NB, CAP, SORT, MINW) \
    (pk[C].n ? launch(prepare_rows_kernel<T, I, NB, CAP, SORT, MINW>, dim3(end[C] + n_pack[C]), dim3(T), 0, st, cls[C], pk[C], n_pack[C]) \
             : launch(binarize_rows_kernel<T, I, NB, CAP, SORT, MINW>, dim3(end[C]), dim3(T), 0, st, cls[C]))
    if (cls[0].n)
        if (int rc = hand.small ? DAB_ROWS(0, 256, 9, 512, 256, false, 7) : DAB_ROWS(0, 256, 9, 512, 256, true, 4)) return rc;
    if (cls[1].n)
        if (int rc = hand.medium ? DAB_ROWS(1, 256, 18, 1024, 256, false, 6) : DAB_ROWS(1, 512, 9, 2048, 256, true, 4)) return rc;
    if (together) {
        const int c = longest;
        const dim3 grid(end[c] + n_pack[c]);
        if (int rc = c == 3 ? launch(prepare_two_kernel<52, 2048, 256>, grid, dim3(256), 0, st, cls[c], pk[c], n_pack[c], n_long)
                            : launch(prepare_two_kernel<36, 2048, 256>, grid, dim3(256), 0, st, cls[c], pk[c], n_pack[c], n_long))
            return rc;
        cls[c].n = 0;
    }
    if (cls[2].n)
        if (int rc = DAB_ROWS(2, 256, 36, 2048, 256, false, 4)) return rc;
    if (cls[3].n)
        if (int rc = wide ? DAB_ROWS(3, 512, 26, 2048, 512, false, 4) : DAB_ROWS(3, 256, 52, 2048, 256, false, 3)) return rc;
    if (sortj.n) {
        if (int rc = launch(binarize_sort_kernel<1024, 13>, dim3(sort_end), dim3(1024), 0, st, static_cast<const uint8_t*>(ws), sortj)) return rc;
    }
#undef DAB_ROWS
    return DAB_OK;
}

// ---------------------------------------------------------------- hand-over flags owned by the library
// dab_estimate_alpha_beta_noalloc keeps the per-row flags of the bucket kernel in this array instead
// of a caller's workspace.  The name is a host-side stand-in for the symbol: the device address is
// looked up once per device (every GPU holds its own copy) and only that address is passed on.
constexpr int kNoAllocMaxFilters = 65536;
static __device__ __align__(256) unsigned char scratch[kNoAllocMaxFilters];
static unsigned char* g_scratch_ptr[kMaxDevices];              // written under the set-up lock of api.hip

int init_estimate(int dev) {
    unsigned char* ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(reinterpret_cast<void**>(&ptr), HIP_SYMBOL(scratch));
    if (e != hipSuccess) return hip_failed(e);
    if (!ptr) return hip_failed(hipErrorInvalidSymbol);
    g_scratch_ptr[dev] = ptr;
    return DAB_OK;
}

}  // namespace dab

extern "C" {

size_t dab_estimate_workspace_bytes(int32_t F, int32_t n) { return F < 1 || n < 2 ? 0 : dab::estimate_ws_bytes(F, n); }
int32_t dab_estimate_max_n(void) { return dab::kEstimateMaxN; }

int dab_estimate_alpha_beta(const float* W, int32_t F, int32_t n, float* alpha, float* beta, int32_t* K,
                            float* thr_val, int32_t* thr_idx, uint8_t* alpha_is_upper, void* ws, size_t ws_bytes,
                            void* stream) {
    using namespace dab;
    if (!W || !alpha || !beta || !K || !thr_val || !thr_idx || !alpha_is_upper) return DAB_ERR_NULL;
    if (F < 1 || n < 2) return DAB_ERR_SHAPE;
    if (misaligned(W, 4) || misaligned(alpha, 4) || misaligned(beta, 4) || misaligned(K, 4) ||
        misaligned(thr_val, 4) || misaligned(thr_idx, 4))
        return DAB_ERR_ALIGN;
    if (n > kEstimateMaxN) return DAB_ERR_UNSUPPORTED;
    return dispatch_estimate(W, F, n, alpha, beta, K, thr_val, thr_idx, alpha_is_upper, nullptr, nullptr, 0, ws, ws_bytes,
                             static_cast<hipStream_t>(stream));
}

size_t dab_binarize_weights_multi_workspace_bytes(const dab_weight_job* jobs, int32_t n_jobs) {
    if (!jobs || n_jobs < 1 || n_jobs > dab::kMaxEstJobs) return 0;
    return dab::weight_jobs_ws_bytes(jobs, n_jobs);
}

int dab_binarize_weights_multi(const dab_weight_job* jobs, int32_t n_jobs, void* ws, size_t ws_bytes, void* stream) {
    using namespace dab;
    if (!jobs) return DAB_ERR_NULL;
    if (n_jobs < 1) return DAB_ERR_SHAPE;
    if (n_jobs > kMaxEstJobs) return DAB_ERR_UNSUPPORTED;
    for (int i = 0; i < n_jobs; ++i)
        if (int rc = check_weight_job(jobs[i])) return rc;
    const size_t need = weight_jobs_ws_bytes(jobs, n_jobs);
    if (need && (!ws || ws_bytes < need)) return DAB_ERR_WORKSPACE;
    if (need && misaligned(ws, 8)) return DAB_ERR_ALIGN;
    return run_weight_jobs(jobs, n_jobs, ws, ws_bytes, static_cast<hipStream_t>(stream));
}

int dab_prepare_layers(const dab_weight_job* wjobs, int32_t n_wjobs, const dab_pack_job* pjobs, int32_t n_pjobs, void* ws,
                       size_t ws_bytes, void* stream) {
    using namespace dab;
    if (!wjobs || !pjobs) return DAB_ERR_NULL;
    if (n_wjobs < 1 || n_pjobs < 1) return DAB_ERR_SHAPE;
    if (n_wjobs > kMaxEstJobs || n_pjobs > kMaxPackJobs) return DAB_ERR_UNSUPPORTED;
    for (int i = 0; i < n_wjobs; ++i)
        if (int rc = check_weight_job(wjobs[i])) return rc;
    for (int i = 0; i < n_pjobs; ++i)
        if (int rc = check_pack_job(pjobs[i])) return rc;
    const size_t need = weight_jobs_ws_bytes(wjobs, n_wjobs);
    if (need && (!ws || ws_bytes < need)) return DAB_ERR_WORKSPACE;
    if (need && misaligned(ws, 8)) return DAB_ERR_ALIGN;
    long long filters = 0;
    for (int i = 0; i < n_wjobs; ++i) filters += wjobs[i].F;
    if (filters < n_pjobs) return DAB_ERR_UNSUPPORTED;            // fewer weight workgroups than tensors to pack
    return run_weight_jobs(wjobs, n_wjobs, ws, ws_bytes, static_cast<hipStream_t>(stream), pjobs, n_pjobs);
}

int32_t dab_estimate_noalloc_max_filters(void) { return dab::kNoAllocMaxFilters; }

int dab_estimate_alpha_beta_noalloc(const float* W, int32_t F, int32_t n, float* alpha, float* beta, int32_t* K,
                                    float* thr_val, int32_t* thr_idx, uint8_t* alpha_is_upper, void* stream) {
    using namespace dab;
    if (!W || !alpha || !beta || !K || !thr_val || !thr_idx || !alpha_is_upper) return DAB_ERR_NULL;
    if (F < 1 || n < 2) return DAB_ERR_SHAPE;
    if (misaligned(W, 4) || misaligned(alpha, 4) || misaligned(beta, 4) || misaligned(K, 4) ||
        misaligned(thr_val, 4) || misaligned(thr_idx, 4))
        return DAB_ERR_ALIGN;
    if (n > kEstimateMaxN || F > kNoAllocMaxFilters) return DAB_ERR_UNSUPPORTED;
    int dev = 0;
    if (int rc = ensure_device_ready(&dev)) return rc;
    // every flag the sort kernel reads (rows 0 .. F-1) is written by the bucket kernel of this call,
    // so the array needs no clearing between calls
    return dispatch_estimate(W, F, n, alpha, beta, K, thr_val, thr_idx, alpha_is_upper, nullptr, nullptr, 0,
                             g_scratch_ptr[dev], kNoAllocMaxFilters, static_cast<hipStream_t>(stream));
}

int dab_estimate_alpha_beta_bounded(const float* W, int32_t F, int32_t n, const int32_t* K_prev,
                                    const uint8_t* alpha_is_upper_prev, int32_t max_change, float* alpha, float* beta,
                                    int32_t* K, float* thr_val, int32_t* thr_idx, uint8_t* alpha_is_upper, void* ws,
                                    size_t ws_bytes, void* stream) {
    using namespace dab;
    if (!W || !K_prev || !alpha_is_upper_prev || !alpha || !beta || !K || !thr_val || !thr_idx || !alpha_is_upper)
        return DAB_ERR_NULL;
    if (F < 1 || n < 2 || max_change < 0) return DAB_ERR_SHAPE;
    if (misaligned(W, 4) || misaligned(K_prev, 4) || misaligned(alpha, 4) || misaligned(beta, 4) || misaligned(K, 4) ||
        misaligned(thr_val, 4) || misaligned(thr_idx, 4))
        return DAB_ERR_ALIGN;
    if (n > kEstimateMaxN) return DAB_ERR_UNSUPPORTED;
    return dispatch_estimate(W, F, n, alpha, beta, K, thr_val, thr_idx, alpha_is_upper, K_prev, alpha_is_upper_prev,
                             max_change, ws, ws_bytes, static_cast<hipStream_t>(stream));
}

int dab_estimate_sign_split(const float* W, int32_t F, int32_t n, float* alpha, float* beta, int32_t* K,
                            float* thr_val, int32_t* thr_idx, uint8_t* alpha_is_upper, void* stream) {
    using namespace dab;
    if (!W || !alpha || !beta || !K || !thr_val || !thr_idx || !alpha_is_upper) return DAB_ERR_NULL;
    if (F < 1 || n < 1) return DAB_ERR_SHAPE;
    if (misaligned(W, 4) || misaligned(alpha, 4) || misaligned(beta, 4) || misaligned(K, 4) ||
        misaligned(thr_val, 4) || misaligned(thr_idx, 4))
        return DAB_ERR_ALIGN;
    return launch(sign_split_kernel, dim3(F), dim3(256), 0, static_cast<hipStream_t>(stream), W, n, alpha, beta, K,
                  thr_val, thr_idx, alpha_is_upper);
}

}  // extern "C"
