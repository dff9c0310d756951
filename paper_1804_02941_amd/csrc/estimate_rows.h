// The two per-row procedures of the estimator as device functions (gfx950): sort_row, the full
// sort of Algorithm 1 (Section 4.3.1 of arXiv 1804.02941), and bucket_row, the search that needs
// no full sort.  Kept apart from the kernels so that a host build can run them thread by thread
// (every wavefront operation below goes through a handful of builtins that such a build supplies).
#pragma once

#ifndef DAB_HOST_EMULATION
#include "dab_internal.h"
#define DAB_RCP_F32(x) __builtin_amdgcn_rcpf(x)
#define DAB_OPAQUE_F32(x) asm volatile("" : "+v"(x))   // the value as the compiler knows nothing about
#define DAB_OPAQUE_I32(x) asm volatile("" : "+v"(x))
#else
#define DAB_OPAQUE_I32(x) asm volatile("" : "+m"(x))
#define DAB_OPAQUE_F32(x) asm volatile("" : "+m"(x))
#define DAB_RCP_F32(x) (1.0f / (x))
#endif

#include <type_traits>

namespace dab {

__device__ __forceinline__ uint32_t float_to_key(float x) {
    const uint32_t u = __float_as_uint(x + 0.0f);                  // -0.0 + 0.0 = +0.0
    return u ^ ((u >> 31) ? 0xFFFFFFFFu : 0x80000000u);
}
__device__ __forceinline__ float key_to_float(uint32_t k) {
    return __uint_as_float(k ^ ((k >> 31) ? 0x80000000u : 0xFFFFFFFFu));
}

// The scans over a wavefront sit on the critical path between two barriers (the 32-bit one once
// per sort pass), so they use data-parallel-primitive moves (register to register, no LDS crossbar round trips): shifts
// by 1, 2, 4, 8 inside each row of 16 lanes (lanes without a source add 0), then lane 15 of row 0
// and 2 into rows 1 and 3, then lane 31 into rows 2 and 3.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ uint32_t dpp_add(uint32_t v) {
    return v + static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), CTRL, ROW_MASK, 0xf, false));
}
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_add(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROW_MASK, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROW_MASK, 0xf, false);
    return v + __hiloint2double(hi, lo);                   // lanes without a source add +0.0
}
__device__ __forceinline__ double wave_inclusive_scan_f64(double v) {
    v = dpp_add<0x111, 0xf>(v);
    v = dpp_add<0x112, 0xf>(v);
    v = dpp_add<0x114, 0xf>(v);
    v = dpp_add<0x118, 0xf>(v);
    v = dpp_add<0x142, 0xa>(v);
    v = dpp_add<0x143, 0xc>(v);
    return v;
}
__device__ __forceinline__ uint32_t wave_inclusive_scan_u32(uint32_t v) {
    v = dpp_add<0x111, 0xf>(v);   // row_shr:1
    v = dpp_add<0x112, 0xf>(v);   // row_shr:2
    v = dpp_add<0x114, 0xf>(v);   // row_shr:4
    v = dpp_add<0x118, 0xf>(v);   // row_shr:8
    v = dpp_add<0x142, 0xa>(v);   // row_bcast:15 into rows 1 and 3
    v = dpp_add<0x143, 0xc>(v);   // row_bcast:31 into rows 2 and 3
    return v;
}

template <int CTRL, int ROW_MASK>
__device__ __forceinline__ long long dpp_add(long long v) {
    const uint32_t lo = static_cast<uint32_t>(
        __builtin_amdgcn_update_dpp(0, static_cast<int>(static_cast<uint32_t>(v)), CTRL, ROW_MASK, 0xf, false));
    const uint32_t hi = static_cast<uint32_t>(
        __builtin_amdgcn_update_dpp(0, static_cast<int>(static_cast<unsigned long long>(v) >> 32), CTRL, ROW_MASK, 0xf, false));
    return v + static_cast<long long>((static_cast<unsigned long long>(hi) << 32) | lo);
}
__device__ __forceinline__ long long wave_inclusive_scan_i64(long long v) {
    v = dpp_add<0x111, 0xf>(v);
    v = dpp_add<0x112, 0xf>(v);
    v = dpp_add<0x114, 0xf>(v);
    v = dpp_add<0x118, 0xf>(v);
    v = dpp_add<0x142, 0xa>(v);
    v = dpp_add<0x143, 0xc>(v);
    return v;
}
// The same moves for reductions: a lane without a source gets its own value back, and after the six
// steps lane 63 holds the result over the wavefront (the other lanes hold partial ones).
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ int dpp_from(int v) {
    return __builtin_amdgcn_update_dpp(v, v, CTRL, ROW_MASK, 0xf, false);
}
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp_from(float v) {
    return __int_as_float(dpp_from<CTRL, ROW_MASK>(__float_as_int(v)));
}
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_from(double v) {
    return __hiloint2double(dpp_from<CTRL, ROW_MASK>(__double2hiint(v)), dpp_from<CTRL, ROW_MASK>(__double2loint(v)));
}
#define DAB_DPP_STEPS(STEP) \
    STEP(0x111, 0xf) STEP(0x112, 0xf) STEP(0x114, 0xf) STEP(0x118, 0xf) STEP(0x142, 0xa) STEP(0x143, 0xc)
__device__ __forceinline__ void wave_min_max_f32(float& mn, float& mx) {      // results in lane 63
#define DAB_STEP(C, M) { const float a = dpp_from<C, M>(mn), b = dpp_from<C, M>(mx); mn = fminf(mn, a); mx = fmaxf(mx, b); }
    DAB_DPP_STEPS(DAB_STEP)
#undef DAB_STEP
}
__device__ __forceinline__ double wave_max_f64(double v) {                    // result in lane 63
#define DAB_STEP(C, M) v = fmax(v, dpp_from<C, M>(v));
    DAB_DPP_STEPS(DAB_STEP)
#undef DAB_STEP
    return v;
}
__device__ __forceinline__ float wave_max_f32(float v) {                      // result in lane 63
#define DAB_STEP(C, M) v = fmaxf(v, dpp_from<C, M>(v));
    DAB_DPP_STEPS(DAB_STEP)
#undef DAB_STEP
    return v;
}

// Set bits of a wavefront mask (the same in every lane) below this lane.
__device__ __forceinline__ uint32_t lanes_below(unsigned long long mask) {
#ifndef DAB_HOST_EMULATION
    return __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(mask >> 32), __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(mask), 0u));
#else
    return static_cast<uint32_t>(__builtin_popcountll(mask & ((1ull << (threadIdx.x & 63u)) - 1ull)));
#endif
}
// A value of lane l (the same l in every lane), as a scalar.
__device__ __forceinline__ uint32_t lane_of(uint32_t v, int l) {
    return static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(v), l));
}
__device__ __forceinline__ int lane_of(int v, int l) { return __builtin_amdgcn_readlane(v, l); }
__device__ __forceinline__ long long lane_of(long long v, int l) {
    const unsigned long long u = static_cast<unsigned long long>(v);
    return static_cast<long long>((static_cast<unsigned long long>(lane_of(static_cast<uint32_t>(u >> 32), l)) << 32) |
                                  lane_of(static_cast<uint32_t>(u), l));
}
__device__ __forceinline__ double lane_of(double v, int l) {
    return __hiloint2double(lane_of(__double2hiint(v), l), lane_of(__double2loint(v), l));
}

// Candidate split: D = num / den with den > 0; P is the prefix sum at the split.
struct Best {
    double num, den, P;
    int i;
};
__device__ __forceinline__ bool better(const Best& a, const Best& b) {   // a beats b
    const double l = a.num * b.den, r = b.num * a.den;
    return l > r || (l == r && a.i > b.i);
}
__device__ __forceinline__ Best wave_best_of(Best v) {                        // result in lane 63
#define DAB_STEP(C, M) \
    { \
        const Best o{dpp_from<C, M>(v.num), dpp_from<C, M>(v.den), dpp_from<C, M>(v.P), dpp_from<C, M>(v.i)}; \
        if (better(o, v)) v = o; \
    }
    DAB_DPP_STEPS(DAB_STEP)
#undef DAB_STEP
    return v;
}

// The split descriptor of the row a workgroup has just estimated, left in LDS for the packing that
// follows in the same kernel (nullptr where nothing follows).
struct SplitInfo {
    float thr_val;
    int thr_idx;
    int upper;
};

// Row f of the layer, by the workgroup's THREADS threads (all of them call this together).
template <int THREADS, int ITEMS>
__device__ __forceinline__ void sort_row(const float* __restrict__ Wt, int n, int f, float* __restrict__ alpha,
                                         float* __restrict__ beta, int32_t* Kout, float* __restrict__ thr_val,
                                         int32_t* __restrict__ thr_idx, uint8_t* alpha_is_upper, const int32_t* K_prev,
                                         const uint8_t* upper_prev, int max_change, SplitInfo* info = nullptr) {
    static_assert(ITEMS >= 1 && ITEMS <= 15, "a digit counter has 4 bits");
    constexpr int NW = THREADS / 64;
    constexpr int N = THREADS * ITEMS;
    __shared__ uint32_t keys[N];
    __shared__ __align__(16) uint32_t counters[8 * THREADS];   // word w*THREADS + t: digits w (low half), w + 8 (high half)
    __shared__ uint32_t wave_tot[NW];
    __shared__ double wave_sum[NW];
    __shared__ Best wave_best[NW];
    __shared__ double total_s;
    __shared__ int r_s;
    __shared__ float thr_s;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const float* row = Wt + static_cast<size_t>(f) * n;

    for (int i = tid; i < N; i += THREADS) keys[i] = i < n ? float_to_key(row[i]) : 0xFFFFFFFFu;
    __syncthreads();

    // ---- radix sort
    for (int shift = 0; shift < 32; shift += 4) {
        uint32_t k[ITEMS];
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) k[j] = keys[tid * ITEMS + j];
        // digit counters of this thread and, per key, how many earlier keys of the thread share its digit
        unsigned long long cnt = 0, pfx = 0;
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) {
            const int sh = ((k[j] >> shift) & 15u) * 4;
            pfx |= ((cnt >> sh) & 15ull) << (4 * j);
            cnt += 1ull << sh;
        }
#pragma unroll
        for (int w = 0; w < 8; ++w)
            counters[w * THREADS + tid] = static_cast<uint32_t>((cnt >> (4 * w)) & 15ull) |
                                          (static_cast<uint32_t>((cnt >> (4 * w + 32)) & 15ull) << 16);
        __syncthreads();
        // exclusive scan over the words in linear order (both halves at once: totals stay below 2^16)
        uint32_t c[8];
        {
            const uint4 lo = *reinterpret_cast<const uint4*>(&counters[tid * 8]);
            const uint4 hi = *reinterpret_cast<const uint4*>(&counters[tid * 8 + 4]);
            c[0] = lo.x; c[1] = lo.y; c[2] = lo.z; c[3] = lo.w; c[4] = hi.x; c[5] = hi.y; c[6] = hi.z; c[7] = hi.w;
        }
        uint32_t run = 0;
#pragma unroll
        for (int w = 0; w < 8; ++w) { const uint32_t t = c[w]; c[w] = run; run += t; }
        const uint32_t inc = wave_inclusive_scan_u32(run);
        if (lane == 63) wave_tot[wave] = inc;
        __syncthreads();
        uint32_t base = inc - run, all = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const uint32_t t = wave_tot[w];
            if (w < wave) base += t;
            all += t;
        }
        // keys with digits 0..7 precede digits 8..15: their total goes into the high halves here,
        // so the scatter only picks a half
        base += (all & 0xFFFFu) << 16;
        *reinterpret_cast<uint4*>(&counters[tid * 8]) = make_uint4(c[0] + base, c[1] + base, c[2] + base, c[3] + base);
        *reinterpret_cast<uint4*>(&counters[tid * 8 + 4]) = make_uint4(c[4] + base, c[5] + base, c[6] + base, c[7] + base);
        __syncthreads();
        // every thread holds its keys in registers, so the buffer can be overwritten in place
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) {
            const uint32_t d = (k[j] >> shift) & 15u;
            const uint32_t word = counters[(d & 7u) * THREADS + tid];
            const uint32_t off = (word >> ((d & 8u) * 2u)) & 0xFFFFu;
            keys[off + static_cast<uint32_t>((pfx >> (4 * j)) & 15ull)] = k[j];
        }
        __syncthreads();
    }

    // ---- prefix sums in fp64: thread t owns sorted positions [t*ITEMS, t*ITEMS + ITEMS), clipped to n
    const int lo = min(n, tid * ITEMS), hi = min(n, lo + ITEMS);
    double x[ITEMS];
    double local = 0.0;
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        x[j] = lo + j < hi ? static_cast<double>(key_to_float(keys[lo + j])) : 0.0;
        local += x[j];
    }
    const double inc = wave_inclusive_scan_f64(local);
    if (lane == 63) wave_sum[wave] = inc;
    __syncthreads();
    double base = inc - local;
    for (int w = 0; w < wave; ++w) base += wave_sum[w];
    if (tid == THREADS - 1) total_s = base + local;
    __syncthreads();
    const double T = total_s;

    // ---- D_i over this thread's positions; split i = position + 1, i in 1 .. n-1, or in the
    // window around the previous split when one is given (read before any output is written, so
    // the previous outputs may be the buffers this call overwrites)
    int wlo = 1, whi = n - 1;
    if (K_prev) {
        int ip = upper_prev[f] ? n - K_prev[f] : K_prev[f];
        ip = min(max(ip, 1), n - 1);
        const int d = min(max(max_change, 0), n);
        wlo = max(1, ip - d);
        whi = min(n - 1, ip + d);
    }
    Best best{-1.0, 1.0, 0.0, 0};
    double P = base;
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        P += x[j];
        const int i = lo + j + 1;
        if (lo + j < hi && i >= wlo && i <= whi) {
            const double rest = T - P;
            const double fi = static_cast<double>(i), fr = static_cast<double>(n - i);
            const Best cand{P * P * fr + rest * rest * fi, fi * fr, P, i};
            if (better(cand, best)) best = cand;
        }
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        const Best o{__shfl_xor(best.num, d, 64), __shfl_xor(best.den, d, 64), __shfl_xor(best.P, d, 64),
                     __shfl_xor(best.i, d, 64)};
        if (better(o, best)) best = o;
    }
    if (lane == 0) wave_best[wave] = best;
    __syncthreads();

    if (tid == 0) {
        Best b = wave_best[0];
        for (int w = 1; w < NW; ++w)
            if (better(wave_best[w], b)) b = wave_best[w];
        const int is = b.i;
        const double mu_lower = b.P / static_cast<double>(is);
        const double mu_upper = (T - b.P) / static_cast<double>(n - is);
        const bool upper = fabs(mu_upper) >= fabs(mu_lower);
        alpha[f] = static_cast<float>(upper ? mu_upper : mu_lower);
        beta[f] = static_cast<float>(upper ? mu_lower : mu_upper);
        Kout[f] = upper ? n - is : is;
        alpha_is_upper[f] = upper ? 1 : 0;
        // value at the split and how many of its duplicates fall in the lower group
        const uint32_t tk = keys[is - 1];
        int a = 0, c = is - 1;                      // first position holding tk (lower bound)
        while (a < c) {
            const int mid = (a + c) >> 1;
            if (keys[mid] < tk) a = mid + 1; else c = mid;
        }
        thr_s = key_to_float(tk);
        thr_val[f] = thr_s;
        r_s = is - a;                               // >= 1 copies of the value are "lower"
        if (info) { info->thr_val = thr_s; info->upper = upper ? 1 : 0; }
    }
    __syncthreads();

    // ---- original index of the r-th copy (in index order) of the split value
    const float tv = thr_s;
    const uint32_t r = static_cast<uint32_t>(r_s);
    uint32_t cnt = 0;
    for (int i = lo; i < hi; ++i) cnt += (row[i] == tv) ? 1u : 0u;
    const uint32_t cinc = wave_inclusive_scan_u32(cnt);
    if (lane == 63) wave_tot[wave] = cinc;
    __syncthreads();
    uint32_t cbase = cinc - cnt;
    for (int w = 0; w < wave; ++w) cbase += wave_tot[w];
    if (cnt > 0 && r > cbase && r <= cbase + cnt) {
        uint32_t seen = cbase;
        for (int i = lo; i < hi; ++i) {
            if (row[i] == tv && ++seen == r) {
                thr_idx[f] = i;
                if (info) info->thr_idx = i;
                break;
            }
        }
    }
}

template <int THREADS, int ITEMS>
__global__ __launch_bounds__(THREADS) void estimate_kernel(const float* __restrict__ Wt, int n,
                                                           float* __restrict__ alpha, float* __restrict__ beta,
                                                           int32_t* Kout, float* __restrict__ thr_val,
                                                           int32_t* __restrict__ thr_idx, uint8_t* alpha_is_upper,
                                                           const int32_t* K_prev, const uint8_t* upper_prev,
                                                           int max_change, const uint8_t* __restrict__ only) {
    if (only && !only[blockIdx.x]) return;      // the bucket kernel below has finished this row
    DAB_RESERVE_VGPRS();   // the 7-items-per-thread instantiations would land on exactly 64 VGPRs
    sort_row<THREADS, ITEMS>(Wt, n, static_cast<int>(blockIdx.x), alpha, beta, Kout, thr_val, thr_idx, alpha_is_upper, K_prev,
                             upper_prev, max_change);
}

// ---------------------------------------------------------------- estimation without the full sort
// The arg-max of D needs the sorted order only near the optimum.  One pass of LDS atomics puts the
// row into NB value buckets (count and exact fixed-point sum each), a scan gives, for every
// bucket, the number and sum of all smaller elements, and with them D at the last element of every
// bucket and an upper bound of D at the positions inside it.  Only buckets whose bound reaches the
// best bucket-end value can hold the arg-max; their elements (a few dozen for the weight
// distributions of a network) are ranked exactly, with exact prefix sums, and the split is chosen
// among them by the same comparison as in the sort.  All copies of a value share a bucket, and the
// ranking goes by value and then by index, so the winner's index is the split descriptor's.  A row
// whose candidates exceed the list (many equal values, a constant row) is left to the sort.
//
// Sums are integers: with 2^e > max |w| the values are scaled by 2^(48 - e) and rounded to int64,
// which is exact for every element within 2^-24 of the row's largest magnitude (smaller ones are
// rounded at 2^-49 of it), and integer atomics make the result independent of their order.
//
// What bounds this is vector instructions, then LDS atomics, then the latency of the chain of
// phases.  So an element costs one 64-bit atomic (15 clocks of a compute unit's LDS for a wavefront, whatever the
// distribution) and five vector instructions in the histogram: the fused multiply-add that rounds it to an integer
// q >= 0 (counted from the row's minimum) leaves q in the low bits of a double, whose upper word holds the bucket
// (q >> sh) and gets the count of one put above the 52 bits that are left to the sum of the offsets inside the bucket.
// A bucket costs about 45 instructions, all but a thread's first in fp32.  No LDS atomic has the address in common
// among lanes (the compiler turns those into a loop over the lanes).  Search alone, one launch: 4096 rows of 9216
// weights 47 us (83 with a count and a sum atomic per element, fp64 bounds and a branch per listed element), of 4096
// 31.6 (46.5), 512 rows of 12544 14.5 (20.3), 1408 of 1800 10.8 (14.0), 256 of 2304 6.7 (9.5).
constexpr int kBucketChunk = 4;         // elements of a thread handled without a branch between them
constexpr int kExactN = 256;            // rows up to here: sums without any rounding
constexpr int kNarrow = 128;            // candidates, and what lies between them, up to here are compared each with each
constexpr uint32_t kParts = 64;         // buckets with a part of a list
constexpr int kMaxLists = 4;            // of candidates; a row with more is left to the sort
constexpr int kPartedRow = 2304;        // rows of the classes up to here: a part of the list for every bucket where there are many
constexpr int kBucketTurns = 12;        // scattered candidate buckets taken one at a time before the row is left to the sort

// f(first element of the chunk, one past its last) over the chunks of ITEMS elements, both as compile-time constants (the
// elements are registers), until it returns false.
template <int ITEMS, int C = 0, typename F>
__device__ __forceinline__ void for_chunks(F&& f) {
    if constexpr (C < ITEMS) {
        constexpr int E = C + kBucketChunk < ITEMS ? C + kBucketChunk : ITEMS;
        if (f(std::integral_constant<int, C>{}, std::integral_constant<int, E>{})) for_chunks<ITEMS, E>(f);
    }
}

// A bit per element of a thread.
template <int ITEMS>
using mask_t = std::conditional_t<(ITEMS > 32), unsigned long long, uint32_t>;
// Element j of a thread's registers, j different in every lane.
template <int LO, int HI, int ITEMS>
__device__ __forceinline__ float pick(const float (&x)[ITEMS], int j) {
    if constexpr (HI - LO == 1) {
        return x[LO];
    } else {
        constexpr int P = HI - LO > 32 ? 32 : (HI - LO > 16 ? 16 : (HI - LO > 8 ? 8 : (HI - LO > 4 ? 4 : (HI - LO > 2 ? 2 : 1))));
        const float a = pick<LO, LO + P>(x, j), b = pick<LO + P, HI>(x, j);
        return (j & P) ? b : a;
    }
}

// A barrier for what the workgroup's threads hand each other in LDS.  (__syncthreads() also waits until every global
// store so far is acknowledged, which at the end of a row is most of a microsecond of nothing.)
__device__ __forceinline__ void lds_barrier() {
#ifndef DAB_HOST_EMULATION
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
#else
    __syncthreads();
#endif
}

// The row as a buffer: a load is one instruction with the thread's offset and the element's (a constant), and past the
// end it gives zero and reads nothing.  (With plain loads every element costs three vector instructions for its address.)
#ifndef DAB_HOST_EMULATION
using RowWindow = __amdgpu_buffer_rsrc_t;
__device__ __forceinline__ RowWindow row_window(const float* row, int n) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(row), 0, 4 * n, 0x00020000);
}
__device__ __forceinline__ float load_from(RowWindow w, int lane_bytes, int step_bytes) {
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(w, lane_bytes, step_bytes, 0));
}
#else
struct RowWindow { const float* row; int n; };
inline RowWindow row_window(const float* row, int n) { return RowWindow{row, n}; }
inline float load_from(RowWindow w, int lane_bytes, int step_bytes) {
    const int i = (lane_bytes + step_bytes) / 4;
    return i < w.n ? w.row[i] : 0.0f;
}
#endif

// The row is read once, every load in flight at once, and stays in registers: element j of thread t
// is row[t + j * THREADS]; positions past the end hold NaN, which no comparison below selects.
template <int THREADS, int ITEMS>
__device__ __forceinline__ void load_row(const float* __restrict__ row, int n, float (&x)[ITEMS]) {
    const int tid = threadIdx.x;
    const RowWindow win = row_window(row, n);
    for_chunks<ITEMS>([&](auto c, auto e) {
        if (e * THREADS <= n) {
#pragma unroll
            for (int j = c; j < e; ++j) x[j] = load_from(win, tid * 4, j * THREADS * 4);
        } else {
#pragma unroll
            for (int j = c; j < e; ++j) {                          // (the scalar offset is no part of what is checked against the end)
                const float v = c * THREADS < n ? load_from(win, (tid + j * THREADS) * 4, 0) : 0.0f;
                x[j] = tid + j * THREADS < n ? v : __uint_as_float(0x7FC00000u);
            }
        }
        return true;
    });
}

// THREADS threads with up to ITEMS elements each (as load_row leaves them), NB value buckets, at most
// CAP candidate elements at a time.  Little LDS is needed and several workgroups share a compute unit:
// every phase is a short latency chain between barriers.  The result says whether the row is done
// (the same for every thread of the workgroup); nothing has been written when it is not.
struct alignas(16) Listed {
    uint32_t idx, key, q_lo, q_hi;                                 // index in the row, above it where its part of the list starts; value as a key; q
};
template <int THREADS, int NB, int CAP>
struct BucketLds {
    static constexpr int NW = THREADS / 64;
    alignas(16) unsigned long long hist[NB];                       // a bucket's count (top 12 bits) and the sum of its offsets
    alignas(16) uint16_t first[NB];                                // elements in lower buckets
    unsigned long long below[THREADS];                             // sum of q in the buckets below those of a thread
    Listed list[CAP + 4];                                          // candidates
    unsigned long long acc_s[CAP];                                 // rank of a candidate and sum up to it
    uint32_t acc_n[CAP];
    uint32_t cmask[THREADS];                                       // candidates among a thread's buckets, a bit each: still to be listed, listed now; their first entry
    uint32_t seg[kParts];                                           // of a listed bucket: start of its part of the list, elements there
    float w_min[NW], w_max[NW], w_g[NW];
    uint32_t w_cnt[NW];
    long long w_sum[NW];
    int w_lo[NW], w_hi[NW];                                        // first and last candidate bucket
    Best wave_best[NW];
    uint32_t nlist;                                                // places asked for, entries asked for
    uint32_t ncand, listed;                                        // elements in candidate buckets, in the list
};
template <int THREADS, int ITEMS, int NB, int CAP, int LISTS = kMaxLists>
__device__ __forceinline__ bool bucket_row(BucketLds<THREADS, NB, CAP>& lds, const float (&x)[ITEMS], int n, int f,
                                           float* __restrict__ alpha, float* __restrict__ beta, int32_t* Kout,
                                           float* __restrict__ thr_val, int32_t* __restrict__ thr_idx, uint8_t* alpha_is_upper,
                                           const int32_t* K_prev, const uint8_t* upper_prev, int max_change,
                                           SplitInfo* info = nullptr) {
    constexpr int NW = THREADS / 64;
    constexpr int BPT = NB / THREADS;                              // buckets per thread
    constexpr int LOG_NB = NB == 512 ? 9 : (NB == 1024 ? 10 : 11);
    static_assert(NB == 1 << LOG_NB && BPT >= 1 && NB % THREADS == 0 && BPT <= 8, "whole buckets per thread, a bit each");
    static_assert(THREADS * ITEMS <= 65535 && LOG_NB >= 9, "16-bit counts; the offsets of up to 4095 elements sum to less than 2^52");
    static_assert(CAP <= THREADS, "a candidate per thread");
    auto& hist = lds.hist;
    auto& first = lds.first;
    auto& below = lds.below;
    auto& list = lds.list;
    auto& acc_n = lds.acc_n;
    auto& acc_s = lds.acc_s;
    auto& cmask = lds.cmask;
    auto& seg = lds.seg;
    auto& w_min = lds.w_min;
    auto& w_max = lds.w_max;
    auto& w_g = lds.w_g;
    auto& w_cnt = lds.w_cnt;
    auto& w_sum = lds.w_sum;
    auto& w_lo = lds.w_lo;
    auto& w_hi = lds.w_hi;
    auto& wave_best = lds.wave_best;
    auto& nlist_s = lds.nlist;
    auto& ncand_s = lds.ncand;
    auto& listed_s = lds.listed;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    // ---- range of the row
#pragma unroll
    for (int k = 0; k < BPT; ++k) hist[tid + k * THREADS] = 0ull;
    if (tid < CAP) { acc_n[tid] = 0u; acc_s[tid] = 0ull; }
    if (tid == 0) { nlist_s = 0u; ncand_s = 0u; listed_s = 0u; seg[0] = 0u; }
    float mn = x[0], mx = x[0];
    for_chunks<ITEMS>([&](auto c, auto e) {
        if (c * THREADS >= n) return false;                        // (the whole workgroup, here and below)
#pragma unroll
        for (int j = c; j < e; ++j) {
            mn = fminf(mn, x[j]);
            mx = fmaxf(mx, x[j]);
        }
        return true;
    });
    wave_min_max_f32(mn, mx);
    if (lane == 63) { w_min[wave] = mn; w_max[wave] = mx; }
    lds_barrier();
    mn = w_min[0];
    mx = w_max[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) { mn = fminf(mn, w_min[w]); mx = fmaxf(mx, w_max[w]); }
    mn = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(mn)));
    mx = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(mx)));
    if (!(mx > mn) || !(fabsf(mn) < INFINITY) || !(fabsf(mx) < INFINITY)) return false;   // constant row (or not finite)
    const float M = fmaxf(fabsf(mn), fabsf(mx));
    const int ex = static_cast<int>((__float_as_uint(M) >> 23) & 0xFFu) - 126;     // M < 2^ex
    const double scale = ldexp(1.0, 48 - ex), unscale = ldexp(1.0, ex - 48);
    // x 2^(48 - ex) rounded to an integer (|.| < 2^48): added to 1.5 * 2^52, the integer sits in the low bits of the double;
    // q = that integer + off, in the low bits of the double near 2^52: off is even, so that ties round the same way, and leaves q
    // at 2 or more before the rounding (below 2^52 doubles are half as far apart: a smallest weight of which the scaling leaves a
    // fraction, one below 2^-24 of the largest, would round to 2^52 - 1/2 there if it could reach it, into the last bucket)
    const long long fmin_i = __double_as_longlong(fma(static_cast<double>(mn), scale, 6755399441055744.0)) - 0x4338000000000000ll;
    const long long off = 2 - fmin_i + (fmin_i & 1);
    const double magic = 4503599627370496.0 + static_cast<double>(off);
    auto q_of = [&](float v) -> double { return fma(static_cast<double>(v), scale, magic); };
    // bucket = q >> sh, at least half of the buckets in use (a row whose range is below an eighth of its largest magnitude
    // uses fewer); 35 <= sh <= 49 - LOG_NB, so buckets are decided in the upper word alone
    const uint32_t qmax_hi = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(__double2hiint(q_of(mx)))) & 0xFFFFFu;
    const int sh = max(35, 64 - __builtin_clz(qmax_hi | 1u) - LOG_NB);
    const uint32_t in_bucket = (1u << (sh - 32)) - 1u;             // upper word: offset inside the bucket
    const int to_addr = sh - 35;
    auto bucket_of = [&](uint32_t hi) -> int { return static_cast<int>((hi & 0xFFFFFu) >> (sh - 32)); };   // from a q's upper word

    // ---- histogram: count and exact sum of offsets per bucket
    // Rows of up to kExactN weights keep all their digits, as the sort does: a group of such a row may be a weight or two,
    // its mean as small as the weight.  One that is rounded is not counted, and the row is left to the sort.
    constexpr bool kExact = THREADS * ITEMS <= 3 * kExactN;
    const float rounded = kExact && n <= kExactN ? ldexpf(1.0f, ex - 25) : 0.0f;
    {
        auto add = [&](float v) {
            if (kExact && (v != 0.0f) & (fabsf(v) < rounded)) return;
            const double q = q_of(v);
            const uint32_t hi = static_cast<uint32_t>(__double2hiint(q)), lo = static_cast<uint32_t>(__double2loint(q));
            unsigned long long* cell = reinterpret_cast<unsigned long long*>(reinterpret_cast<char*>(hist) +
                                                                            ((hi >> to_addr) & ((NB - 1u) << 3)));
            atomicAdd(cell, (static_cast<unsigned long long>((hi & in_bucket) | 0x100000u) << 32) | lo);
        };
        for_chunks<ITEMS>([&](auto c, auto e) {
            if (c * THREADS >= n) return false;
            if (e * THREADS <= n) {
#pragma unroll
                for (int j = c; j < e; ++j) add(x[j]);
            } else {
#pragma unroll
                for (int j = c; j < e; ++j)
                    if (tid + j * THREADS < n) add(x[j]);
            }
            return true;
        });
    }
    lds_barrier();

    // ---- prefixes over the buckets (thread t has buckets t*BPT ..).  A bucket with 4096 elements or more spoils
    // the counts: their sum is then not n, and the row is left to the sort.
    uint32_t bc[BPT];                                              // counts
    float bf[BPT];                                                 // the offsets' sum in buckets' widths
    uint32_t crun = 0, cb = 0;
    unsigned long long srun = 0;
    {
        const float per_width = __uint_as_float(static_cast<uint32_t>(127 + 24 - sh) << 23);   // 2^(24 - sh)
        unsigned long long cell[BPT];
#pragma unroll
        for (int k = 0; k < BPT; ++k) cell[k] = hist[tid * BPT + k];
#pragma unroll
        for (int k = 0; k < BPT; ++k) {
            const uint32_t hi = static_cast<uint32_t>(cell[k] >> 32), lo = static_cast<uint32_t>(cell[k]);
            bc[k] = hi >> 20;
            bf[k] = static_cast<float>(((hi & 0xFFFFFu) << 8) | (lo >> 24)) * per_width;
            crun += bc[k];
            cb += bc[k] * static_cast<uint32_t>(tid * BPT + k);
            srun += cell[k] & 0xFFFFFFFFFFFFFull;
        }
        srun += static_cast<unsigned long long>(cb) << sh;
    }
    const uint32_t cinc = wave_inclusive_scan_u32(crun);
    const unsigned long long sinc = static_cast<unsigned long long>(wave_inclusive_scan_i64(static_cast<long long>(srun)));
    if (lane == 63) { w_cnt[wave] = cinc; w_sum[wave] = static_cast<long long>(sinc); }
    lds_barrier();
    // (the wavefronts' totals: a lane each, scanned like the rest)
    uint32_t wc = w_cnt[NW == 1 ? 0 : lane & (NW - 1)];
    long long wsum = w_sum[NW == 1 ? 0 : lane & (NW - 1)];
    if (NW > 1) { wc = dpp_add<0x111, 0xf>(wc); wsum = dpp_add<0x111, 0xf>(wsum); }
    if (NW > 2) { wc = dpp_add<0x112, 0xf>(wc); wsum = dpp_add<0x112, 0xf>(wsum); }
    if (NW > 4) { wc = dpp_add<0x114, 0xf>(wc); wsum = dpp_add<0x114, 0xf>(wsum); }
    if (NW > 8) { wc = dpp_add<0x118, 0xf>(wc); wsum = dpp_add<0x118, 0xf>(wsum); }
    if (lane_of(wc, NW - 1) != static_cast<uint32_t>(n)) return false;
    const unsigned long long s_all = static_cast<unsigned long long>(lane_of(wsum, NW - 1));
    uint32_t i_run = cinc - crun + (wave ? lane_of(wc, wave - 1) : 0u);
    const unsigned long long s_base = sinc - srun + (wave ? static_cast<unsigned long long>(lane_of(wsum, wave - 1)) : 0ull);
    const long long T_fix = static_cast<long long>(s_all) - static_cast<long long>(n) * off;    // the row's sum

    below[tid] = s_base;

    // ---- allowed splits: 1 .. n-1, or the window around the previous split
    int wlo = 1, whi = n - 1;
    if (K_prev) {
        int ip = upper_prev[f] ? n - K_prev[f] : K_prev[f];
        ip = min(max(ip, 1), n - 1);
        const int d = min(max(max_change, 0), n);
        wlo = max(1, ip - d);
        whi = min(n - 1, ip + d);
    }

    // ---- D at the end of every bucket and a bound inside it.  D = T^2/n + n (P - i T/n)^2 / (i (n - i)), and the
    // second term does not change when every value is shifted, so it is taken of the q; P - i T/n is at most 0 for
    // ascending values, so D is the larger the smaller P is.  With j of the bucket's c elements below the split,
    // P is at least L(j) = max(S_b + j lo, S_e - (c - j) hi), lo and hi the bucket's limits, and D is convex along
    // both lines: it is at most the largest of its values at the bucket's start, at its end and where the two
    // lines cross, at c - (sum of the offsets / width).  In units of a bucket's width and in fp32, from differences
    // formed in fp64 at a thread's first bucket.
    const double mean = static_cast<double>(s_all) / static_cast<double>(n);
    const float nf = static_cast<float>(n);
    float ub[BPT];                                                 // bound over the bucket
    float gbest = -1.0f;                                           // largest value at an allowed end
    {
        auto spread = [&](float Q, float i) -> float { return Q * Q * DAB_RCP_F32(fmaxf(i * (nf - i), 0.5f)); };
        float Q0 = static_cast<float>(ldexp(static_cast<double>(s_base) - static_cast<double>(i_run) * mean, -sh));
        float i0 = static_cast<float>(i_run), g0 = spread(Q0, i0);
        float dist = static_cast<float>(static_cast<double>(tid * BPT) - ldexp(mean, -sh));     // bucket's lower limit - mean
        uint32_t i = i_run, pair = 0;
#pragma unroll
        for (int k = 0; k < BPT; ++k) {
            if (BPT == 1) first[tid] = static_cast<uint16_t>(i);
            else if (k % 2 == 0) pair = i;
            else reinterpret_cast<uint32_t*>(first)[tid * (BPT / 2) + k / 2] = pair | (i << 16);
            const int start = static_cast<int>(i);
            i += bc[k];
            const int end = static_cast<int>(i);
            const float c = static_cast<float>(bc[k]), js = c - bf[k], i1 = static_cast<float>(i);
            const float Q1 = Q0 + fmaf(c, dist, bf[k]);
            const float g1 = spread(Q1, i1), gs = spread(fmaf(js, dist, Q0), i0 + js);
            float bound = fmaxf(fmaxf(g0, g1), gs), at_end = g1;
            DAB_OPAQUE_F32(bound);                                 // (evaluated here, not in branches on the conditions below)
            DAB_OPAQUE_F32(at_end);
            ub[k] = ((bc[k] != 0u) & (end >= wlo) & (start < whi)) ? bound : -INFINITY;
            gbest = ((bc[k] != 0u) & (end >= wlo) & (end <= whi)) ? fmaxf(gbest, at_end) : gbest;
            Q0 = Q1;
            i0 = i1;
            g0 = g1;
            dist += 1.0f;
        }
    }
    gbest = wave_max_f32(gbest);
    if (lane == 63) w_g[wave] = gbest;
    lds_barrier();
    gbest = w_g[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) gbest = fmaxf(gbest, w_g[w]);
    // a margin of 4e-6 of D (the fp32 evaluation is good to 1e-6); no allowed end: every bucket of the window
    const float mean_f = static_cast<float>(ldexp(mean - static_cast<double>(off), -sh));
    const float need = gbest < 0.0f ? -3.0e38f : gbest - 4e-6f * (gbest + mean_f * mean_f);

    // ---- candidates: buckets that can hold a split reaching `need`
    constexpr bool kParted = THREADS * ITEMS <= kPartedRow;
    // (an atomic whose address is known to be the same in all lanes becomes a scan over them)
    auto no_offset = []() -> int {
        int zero = 0;
        DAB_OPAQUE_I32(zero);
        return zero;
    };
    {
        uint32_t mask = 0;
#pragma unroll
        for (int k = 0; k < BPT; ++k) mask |= ub[k] >= need ? 1u << k : 0u;
        cmask[tid] = mask;
        if (mask && kParted) {
            uint32_t c = 0;
#pragma unroll
            for (int k = 0; k < BPT; ++k) c += (mask >> k) & 1u ? bc[k] : 0u;
            atomicAdd(&ncand_s + no_offset(), c);
        }
        const unsigned long long any = __ballot(mask != 0u);
        int lo = NB, hi = -1;
        if (any != 0ull) {
            const int l0 = __builtin_ctzll(any), l1 = 63 - __builtin_clzll(any);
            lo = (wave * 64 + l0) * BPT + __builtin_ctz(lane_of(mask, l0));
            hi = (wave * 64 + l1) * BPT + 31 - __builtin_clz(lane_of(mask, l1));
        }
        if (lane == 0) { w_lo[wave] = lo; w_hi[wave] = hi; }
    }
    lds_barrier();
    int lo = w_lo[0], hi = w_hi[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) { lo = min(lo, w_lo[w]); hi = max(hi, w_hi[w]); }
    lo = __builtin_amdgcn_readfirstlane(lo);
    const int last = __builtin_amdgcn_readfirstlane(hi);
    if (last < 0) return false;                                    // no bucket in the window: not expected

    Best best{-1.0, 1.0, 0.0, 0};                                  // of this thread's candidates
    uint32_t my_key = 0, my_idx = 0;
    int nblk = 0;                                                  // wavefronts that had candidates
    auto elements_below = [&](int b) -> int { return b < NB ? static_cast<int>(first[b]) : n; };
    auto uniform = [](int v) -> int { return __builtin_amdgcn_readfirstlane(v); };
    if constexpr (kParted) {
        // Most rows have few candidates, neighbours: one list, every element compared with every other.  Heavy tails put
        // hundreds of elements into a few buckets, or buckets that are no candidates between them: then every bucket gets a
        // part of the list to itself and its elements are compared with each other only, in as many lists as it takes (one
        // where the workgroup itself sorts what is left, which takes less than a second list).  us, weight sides, all between
        // the first and the last candidate in one list | now: the 128 x 1600 Laplacian weights of configuration 2 17.7 | 11.5,
        // other Laplacian ones 128 x 1600 12.9 | 10.5, 256 x 2304 23.1 | 19.0, 1024 x 1152 19.5 | 13.9; Gaussian ones
        // 256 x 2304 9.05 | 9.3, the others within 1 %.  In the classes of longer rows the registers for it cost a wavefront
        // per SIMD (4096 Gaussian rows of 9216 57.0 | 61.5): they keep the other form below.
        const int total = __builtin_amdgcn_readfirstlane(static_cast<int>(ncand_s));
        const int span = __builtin_amdgcn_readfirstlane(elements_below(last + 1) - elements_below(lo));
        const bool narrow = span <= kNarrow;
        if (!narrow && total > LISTS * CAP) return false;
        // the parts of as many of this thread's candidate buckets as the list still holds
        auto take_places = [&]() {
            const uint32_t mask = cmask[tid] & 0xFFu;
            uint32_t m = 0, entry = 0;
            if (mask) {
                auto count = [&](int k) -> uint32_t {
                    return static_cast<uint32_t>(elements_below(tid * BPT + k + 1) - static_cast<int>(first[tid * BPT + k]));
                };
                uint32_t whole = 0;
#pragma unroll
                for (int k = 0; k < BPT; ++k) whole += (mask >> k) & 1u ? count(k) : 0u;
                m = whole <= CAP ? mask : mask & (~mask + 1u);         // (too many for one list: the lowest bucket's)
                const uint32_t c = whole <= CAP ? whole : count(__builtin_ctz(mask));
                const uint32_t taken = atomicAdd(&nlist_s + no_offset(), (static_cast<uint32_t>(__builtin_popcount(m)) << 16) | c);
                uint32_t at = taken & 0xFFFFu, e = taken >> 16;
                entry = e;
                if (at + c <= CAP && e + static_cast<uint32_t>(__builtin_popcount(m)) <= kParts) atomicAdd(&listed_s + no_offset(), c);
                else m = 0;
#pragma unroll
                for (int k = 0; k < BPT; ++k)
                    if ((m >> k) & 1u) {
                        seg[e++] = at;
                        at += count(k);
                    }
            }
            cmask[tid] = (mask & ~m) | (m << 8) | (entry << 16);
        };
        // q >= A (even) says x 2^(48 - ex) + off >= A - 1/2, so the elements of buckets lo .. last are those from the smallest
        // float at or above one value to below another
        auto at_least = [&](int b) -> float {
            const double t = (ldexp(static_cast<double>(b), sh) - 0.5 - static_cast<double>(off)) * unscale;   // (exact)
            const float v = static_cast<float>(t);
            return __int_as_float(__builtin_amdgcn_readfirstlane(
                __float_as_int(key_to_float(float_to_key(v) + (static_cast<double>(v) < t ? 1u : 0u)))));
        };
        const float xlo = at_least(lo), xhi = at_least(last + 1);
        int left = narrow ? span : total;
        for (;;) {
            int nc = left;
            if (!narrow) {
                take_places();
                lds_barrier();
                nc = __builtin_amdgcn_readfirstlane(static_cast<int>(listed_s));
                if (nc == 0) return false;                             // (a bucket alone is too much for the list)
            }
            {
                // A thread notes its elements in a mask, then files its few, each selected from the registers by a tree of
                // selects: a branch per element costs more than that, and ten times the code.
                uint32_t part[(ITEMS + 31) / 32] = {};
                for_chunks<ITEMS>([&](auto c, auto e) {
                    if (c * THREADS >= n) return false;
                    uint32_t four = 0;
#pragma unroll
                    for (int j = c; j < e; ++j) four |= ((x[j] >= xlo) & (x[j] < xhi)) ? 1u << (j - c) : 0u;
                    part[c / 32] |= four << (c % 32);
                    return true;
                });
                mask_t<ITEMS> mine = part[0];
                if constexpr (ITEMS > 32) mine |= static_cast<mask_t<ITEMS>>(part[1]) << 32;
                while (mine) {
                    const int j = __builtin_ctzll(mine);
                    mine &= mine - 1;
                    const float v = pick<0, ITEMS>(x, j);
                    const double q = q_of(v);
                    const uint32_t q_hi = static_cast<uint32_t>(__double2hiint(q)) & 0xFFFFFu;
                    uint32_t entry = 0;
                    if (!narrow) {
                        const int b = bucket_of(q_hi);
                        const uint32_t m = cmask[b / BPT];
                        if (!((m >> (8 + b % BPT)) & 1u)) continue;    // (not a candidate, or not in this list)
                        entry = (m >> 16) + static_cast<uint32_t>(__builtin_popcount((m >> 8) & ((1u << (b % BPT)) - 1u)));
                    }
                    const uint32_t old = atomicAdd(&seg[entry] + no_offset(), 1u << 16), start = old & 0xFFFFu;
                    list[start + (old >> 16)] = Listed{(start << 16) | static_cast<uint32_t>(tid + j * THREADS), float_to_key(v),
                                                       static_cast<uint32_t>(__double2loint(q)), q_hi};
                }
            }
            lds_barrier();
            if (tid == 0) { nlist_s = 0u; listed_s = 0u; }             // (for the next list)
            left -= nc;

            // exact rank and prefix sum of every candidate in its part of the list: the elements up to it in the order of
            // value, then index.  The wavefronts share every part out.
            constexpr int kTrip = 2;                               // entries read together, as many as the classes have registers for
            const int nb = (nc + 63) >> 6;
            {
                for (int v = 0; v < nb; ++v) {
                    const int e = v * 64 + lane;
                    const Listed& me = list[min(e, nc - 1)];
                    const unsigned long long key = (static_cast<unsigned long long>(me.key) << 32) | me.idx;
                    uint32_t cnt = 0;
                    unsigned long long sum = 0;
                    auto compare_with = [&](int q0, int q1) {
                        for (int q = q0; q < q1; q += kTrip) {
                            Listed o[kTrip];
#pragma unroll
                            for (int u = 0; u < kTrip; ++u) o[u] = list[q + u];
#pragma unroll
                            for (int u = 0; u < kTrip; ++u) DAB_OPAQUE_I32(o[u].q_lo);   // (read with the rest, not behind the comparison)
#pragma unroll
                            for (int u = 0; u < kTrip; ++u) {
                                const bool le = (q + u < q1) & (((static_cast<unsigned long long>(o[u].key) << 32) | o[u].idx) <= key);
                                cnt += le ? 1u : 0u;
                                sum += le ? (static_cast<unsigned long long>(o[u].q_hi) << 32) | o[u].q_lo : 0ull;
                            }
                        }
                    };
                    if (narrow) {                                      // (the same entries in every lane)
                        const int per = (nc + NW - 1) / NW, q0 = wave * per;
                        compare_with(q0, min(q0 + per, nc));
                    } else {
                        const int b = bucket_of(me.q_hi), start = static_cast<int>(me.idx >> 16);
                        const int size = elements_below(b + 1) - elements_below(b), per = (size + NW - 1) / NW, q0 = start + wave * per;
                        compare_with(q0, min(q0 + per, start + size));
                    }
                    if (e < nc) {
                        atomicAdd(&acc_n[e], cnt);
                        atomicAdd(&acc_s[e], sum);
                    }
                }
            }
            lds_barrier();
            // the split behind it
            if (tid < nc) {
                const int b = narrow ? lo : bucket_of(list[tid].q_hi), b0 = b / BPT * BPT;   // the lowest bucket of the part
                unsigned long long sum = below[b / BPT] + acc_s[tid];
#pragma unroll
                for (int k = 0; k < BPT - 1; ++k) {
                    const unsigned long long cell = hist[b0 + k];
                    const unsigned long long in = (cell & 0xFFFFFFFFFFFFFull) +
                                                  (static_cast<unsigned long long>(static_cast<uint32_t>(cell >> 52) * static_cast<uint32_t>(b0 + k)) << sh);
                    sum += b0 + k < b ? in : 0ull;
                }
                const int i = static_cast<int>(first[b]) + static_cast<int>(acc_n[tid]);
                acc_s[tid] = 0ull;
                acc_n[tid] = 0u;
                if (i >= wlo && i <= whi) {
                    const double T = static_cast<double>(T_fix);
                    const double Pi = static_cast<double>(static_cast<long long>(sum) - static_cast<long long>(i) * off);
                    const double rest = T - Pi;
                    const double fi = static_cast<double>(i), fr = static_cast<double>(n - i);
                    const Best c{Pi * Pi * fr + rest * rest * fi, fi * fr, Pi, i};
                    if (better(c, best)) { best = c; my_key = list[tid].key; my_idx = list[tid].idx & 0xFFFFu; }
                }
            }
            nblk = max(nblk, nb);
            if (left == 0) break;
        }
    } else {
        // ---- the candidates are neighbours as a rule: everything between the first and the last of them is taken
        // at once.  Where that is too much (D has two maxima of nearly the same height) one bucket is taken at a time.
        hi = last;
        for (int turns = 1;; ++turns) {
            const int n_lo = uniform(elements_below(lo));
            if (uniform(elements_below(hi + 1)) - n_lo > CAP) hi = lo;
            const int in_reach = uniform(elements_below(hi + 1)) - n_lo;
            if (in_reach > CAP || turns > kBucketTurns) return false;

            // the candidates' elements.  q >= A (even) says x 2^(48 - ex) + off >= A - 1/2, so the elements of
            // buckets lo .. hi are those from the smallest float at or above one value to below another.
            {
                auto at_least = [&](int b) -> float {
                    const double t = (ldexp(static_cast<double>(b), sh) - 0.5 - static_cast<double>(off)) * unscale;   // (exact)
                    const float v = static_cast<float>(t);
                    return key_to_float(float_to_key(v) + (static_cast<double>(v) < t ? 1u : 0u));
                };
                const float xlo = at_least(lo), xhi = at_least(hi + 1);
                // A thread notes its elements in a mask, then the wavefront takes places in the list together and every thread
                // files its few, each selected from the registers by a tree of selects: a branch per element costs more than
                // that, and ten times the code.
                uint32_t part[(ITEMS + 31) / 32] = {};
                for_chunks<ITEMS>([&](auto c, auto e) {
                    if (c * THREADS >= n) return false;
                    uint32_t four = 0;
#pragma unroll
                    for (int j = c; j < e; ++j) four |= ((x[j] >= xlo) & (x[j] < xhi)) ? 1u << (j - c) : 0u;
                    part[c / 32] |= four << (c % 32);
                    return true;
                });
                mask_t<ITEMS> mine = part[0];
                if constexpr (ITEMS > 32) mine |= static_cast<mask_t<ITEMS>>(part[1]) << 32;
                const uint32_t have = static_cast<uint32_t>(__builtin_popcountll(mine));
                const uint32_t upto = wave_inclusive_scan_u32(have), count = lane_of(upto, 63);
                if (count != 0u) {
                    uint32_t base = 0;
                    if (lane == 0) base = atomicAdd(&nlist_s, count);
                    uint32_t slot = lane_of(base, 0) + upto - have;
                    while (mine) {
                        const int j = __builtin_ctzll(mine);
                        mine &= mine - 1;
                        const float v = pick<0, ITEMS>(x, j);
                        const double q = q_of(v);
                        if (slot < static_cast<uint32_t>(CAP))
                            list[slot] = Listed{static_cast<uint32_t>(tid + j * THREADS), float_to_key(v),
                                                static_cast<uint32_t>(__double2loint(q)),
                                                static_cast<uint32_t>(__double2hiint(q)) & 0xFFFFFu};
                        ++slot;
                    }
                }
            }
            lds_barrier();
            const int nc = __builtin_amdgcn_readfirstlane(static_cast<int>(nlist_s));
            if (nc != in_reach) return false;                          // (not expected: the counts said otherwise)

            // exact rank and prefix sum of every candidate: the listed elements up to it in the order of value, then
            // index.  The wavefronts share the list out.
            const int nb = (nc + 63) >> 6;
            {
                const int per = (nc + NW - 1) / NW;
                const int q0 = wave * per, q1 = min(q0 + per, nc);
                for (int v = 0; v < nb; ++v) {
                    const int e = v * 64 + lane;
                    const Listed& me = list[min(e, nc - 1)];
                    const unsigned long long key = (static_cast<unsigned long long>(me.key) << 32) | me.idx;
                    uint32_t cnt = 0;
                    unsigned long long sum = 0;
                    for (int q = q0; q < q1; q += 4) {
                        Listed o[4];
#pragma unroll
                        for (int u = 0; u < 4; ++u) o[u] = list[q + u];
#pragma unroll
                        for (int u = 0; u < 4; ++u) DAB_OPAQUE_I32(o[u].q_lo);   // (read with the rest, not behind the comparison)
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            const bool le = (q + u < q1) & (((static_cast<unsigned long long>(o[u].key) << 32) | o[u].idx) <= key);
                            cnt += le ? 1u : 0u;
                            sum += le ? (static_cast<unsigned long long>(o[u].q_hi) << 32) | o[u].q_lo : 0ull;
                        }
                    }
                    if (e < nc) {
                        atomicAdd(&acc_n[e], cnt);
                        atomicAdd(&acc_s[e], sum);
                    }
                }
            }
            lds_barrier();
            // the split behind it
            if (tid < nc) {
                unsigned long long sum = below[lo / BPT] + acc_s[tid];
#pragma unroll
                for (int k = 0; k < BPT - 1; ++k) {
                    const int b = lo / BPT * BPT + k;
                    const unsigned long long cell = hist[b];
                    const unsigned long long in = (cell & 0xFFFFFFFFFFFFFull) +
                                                  (static_cast<unsigned long long>(static_cast<uint32_t>(cell >> 52) * static_cast<uint32_t>(b)) << sh);
                    sum += b < lo ? in : 0ull;
                }
                const int i = n_lo + static_cast<int>(acc_n[tid]);
                if (i >= wlo && i <= whi) {
                    const double T = static_cast<double>(T_fix);
                    const double Pi = static_cast<double>(static_cast<long long>(sum) - static_cast<long long>(i) * off);
                    const double rest = T - Pi;
                    const double fi = static_cast<double>(i), fr = static_cast<double>(n - i);
                    const Best c{Pi * Pi * fr + rest * rest * fi, fi * fr, Pi, i};
                    if (better(c, best)) { best = c; my_key = list[tid].key; my_idx = list[tid].idx; }
                }
            }
            nblk = max(nblk, nb);
            if (hi >= last) break;
            // the next candidate bucket; the list and its sums start again
            int next = NB;
            for (int w = hi / BPT / 64; w < NW && next == NB; ++w) {
                uint32_t mask = cmask[w * 64 + lane];
                const int b0 = (w * 64 + lane) * BPT;                  // (a thread's bucket k counts if b0 + k > hi)
                if (hi >= b0) mask = hi - b0 >= 31 ? 0u : mask & ~((2u << (hi - b0)) - 1u);
                const unsigned long long any = __ballot(mask != 0u);
                if (any != 0ull) {
                    const int l0 = __builtin_ctzll(any);
                    next = (w * 64 + l0) * BPT + __builtin_ctz(lane_of(mask, l0));
                }
            }
            lo = next;
            hi = last;
            lds_barrier();
            if (tid < CAP) { acc_n[tid] = 0u; acc_s[tid] = 0ull; }
            if (tid == 0) nlist_s = 0u;
            lds_barrier();
        }
    }

    int won;                                                       // the winning position
    if (nblk == 1) {
        // one wavefront holds them all: those within rounding of the largest quotient, one as a rule
        if (wave != 0) return true;
        const double d = best.num / best.den;
        const double dmax = lane_of(wave_max_f64(d), 63);
        unsigned long long top = __ballot(d >= dmax * (1.0 - 1e-13));
        Best bb{-1.0, 1.0, 0.0, 0};
        for (; top != 0ull; top &= top - 1ull) {
            const int l = __builtin_ctzll(top);
            const Best o{lane_of(best.num, l), lane_of(best.den, l), 0.0, lane_of(best.i, l)};
            if (better(o, bb)) bb = o;
        }
        won = bb.i;
    } else {
        if (wave < nblk) {
            const Best wb = wave_best_of(best);
            if (lane == 63) wave_best[wave] = wb;
        }
        lds_barrier();
        Best bb = wave_best[0];
        for (int w = 1; w < nblk; ++w)
            if (better(wave_best[w], bb)) bb = wave_best[w];
        won = bb.i;
    }
    if (best.i == won) {                                           // exactly one thread holds the winning position
        const double T = static_cast<double>(T_fix);
        const double mu_lower = best.P / static_cast<double>(won) * unscale;
        const double mu_upper = (T - best.P) / static_cast<double>(n - won) * unscale;
        const bool upper = fabs(mu_upper) >= fabs(mu_lower);
        if (info) { info->thr_val = key_to_float(my_key); info->thr_idx = static_cast<int>(my_idx); info->upper = upper ? 1 : 0; }
        alpha[f] = static_cast<float>(upper ? mu_upper : mu_lower);
        beta[f] = static_cast<float>(upper ? mu_lower : mu_upper);
        Kout[f] = upper ? n - won : won;
        alpha_is_upper[f] = upper ? 1 : 0;
        thr_val[f] = key_to_float(my_key);
        thr_idx[f] = static_cast<int32_t>(my_idx);
    }
    return true;
}
template <int THREADS, int ITEMS, int NB, int CAP, int LISTS = kMaxLists>
__device__ __forceinline__ bool bucket_row(const float (&x)[ITEMS], int n, int f, float* __restrict__ alpha,
                                           float* __restrict__ beta, int32_t* Kout, float* __restrict__ thr_val,
                                           int32_t* __restrict__ thr_idx, uint8_t* alpha_is_upper, const int32_t* K_prev,
                                           const uint8_t* upper_prev, int max_change) {
    __shared__ BucketLds<THREADS, NB, CAP> lds;
    return bucket_row<THREADS, ITEMS, NB, CAP, LISTS>(lds, x, n, f, alpha, beta, Kout, thr_val, thr_idx, alpha_is_upper, K_prev,
                                               upper_prev, max_change);
}

}  // namespace dab
