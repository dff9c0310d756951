// The mask of a filter (Corollary 1 of arXiv 1804.02941: bit = [the weight belongs to the alpha group], by stable
// rank, from the split descriptor) packed into its column of E by one workgroup, as device functions (gfx950): shared by
// the packing kernel and by the estimators that pack a row while they hold it.
#pragma once

#include "dab_internal.h"

#include "estimate_rows.h"

namespace dab {

constexpr int kPackMaxTaps = 128;                  // of a window whose counts these functions keep in LDS
struct MaskShape {
    uint32_t* E;                                   // packed mask [T*Cw][Fp]
    uint32_t* ecnt;                                // per-tap counts [F][T]
    int n, C, T, Cw, Fp;                           // n = C*T weights, T taps, Cw words per tap, Fp filter columns
};
inline MaskShape make_mask_shape(uint32_t* E, uint32_t* ecnt, int F, int C, int T) {
    return MaskShape{E, ecnt, C * T, C, T, ceil_div(C, 32), 64 * ceil_div(F, 64)};
}

// Workgroup r of a layer takes filter column f: consecutive workgroups go to consecutive XCDs, and a
// column of E is one 4-byte word per row, so an XCD gets a contiguous range of columns and the
// partial lines of neighbouring filters merge in one L2.
__device__ __forceinline__ int column_of_block(unsigned r, int Fp) {
    const int per_xcd = (Fp + kNumXCD - 1) / kNumXCD;
    const int f = static_cast<int>(r % kNumXCD) * per_xcd + static_cast<int>(r / kNumXCD);
    return static_cast<int>(r / kNumXCD) < per_xcd ? f : Fp;
}

// Column f past the last filter: zeros.
template <int THREADS>
__device__ __forceinline__ void pack_padding(const MaskShape& job, int f) {
    uint32_t* const E = job.E;
    const int R = job.T * job.Cw, Fp = job.Fp;
    for (int r = threadIdx.x; r < R; r += THREADS) E[static_cast<size_t>(r) * Fp + f] = 0u;
}

// v with lane l (the same in every lane) replaced by the scalar s.
__device__ int amdgcn_writelane(int s, int l, int v) __asm("llvm.amdgcn.writelane.i32");
__device__ __forceinline__ uint32_t write_lane(uint32_t v, uint32_t s, int l) {
    return static_cast<uint32_t>(amdgcn_writelane(static_cast<int>(s), l, static_cast<int>(v)));
}

// Column f of E and the filter's per-tap counts from the mask, a byte per weight in LDS: one thread per
// packed word gathers its 32 channels (stride T), writes the word and adds its ones to the tap's count.  (A
// wavefront per word pair with a ballot is slower: its address arithmetic is per word instead of per lane.)
template <int THREADS>
__device__ __forceinline__ void pack_bytes(const MaskShape& job, int f, const uint8_t* maskb, uint32_t* tapcnt) {
    const int tid = threadIdx.x;
    // the job's fields by value: behind a reference into the kernel's arguments every store below
    // would make the compiler read them again
    uint32_t* const E = job.E;
    uint32_t* const ecnt = job.ecnt;
    const int C = job.C, T = job.T, Cw = job.Cw, Fp = job.Fp;
    const int R = T * Cw;
    for (int t = tid; t < T; t += THREADS) tapcnt[t] = 0u;
    lds_barrier();
    // (all reads of a word in flight together)
    for (int r = tid; r < R; r += THREADS) {
        const int tap = r / Cw, w = r - tap * Cw;
        const int c0 = 32 * w, nc = min(32, C - c0);
        const uint8_t* src = maskb + c0 * T + tap;
        uint32_t word = 0;
        if (nc == 32) {
#pragma unroll
            for (int k = 0; k < 32; ++k) word |= static_cast<uint32_t>(src[k * T]) << k;
        } else {
            for (int k = 0; k < nc; ++k) word |= static_cast<uint32_t>(src[k * T]) << k;
        }
        E[static_cast<size_t>(r) * Fp + f] = word;
        atomicAdd(&tapcnt[tap], static_cast<uint32_t>(__builtin_popcount(word)));
    }
    lds_barrier();
    for (int t = tid; t < T; t += THREADS) ecnt[static_cast<size_t>(f) * T + t] = tapcnt[t];
}

// The mask of filter column f as bits (Corollary 1, by stable rank: the split descriptor), by the
// whole workgroup, from the row as load_row left it in registers.
// A window of one tap (fully-connected layers, 1 x 1 convolutions) has its channels in the order of the
// row, so the 64 elements a wavefront holds under one j already are two words: a ballot each, kept by
// lane j, no LDS.  (Through LDS the 32-byte stride of the gather put 64 lanes on eight banks: 4096 rows of
// 9216 weights and 4096 of 4096, weight side of both in one call: 175.6 us, 157.6 with the ballots.)  Only
// as many ballots as the row has steps of the workgroup's threads: with all of its class's, short rows were
// slower than through LDS (16384 rows of 256 weights: LDS 91.0 us, nine ballots 97.5, one 87.8; 4096 of 64:
// 28.6, 29.4, 27.3; 8192 of 512: 51.5, 53.9, 50.0).
template <int THREADS, int ITEMS>
__device__ __forceinline__ void pack_row(const MaskShape& job, int f, const SplitInfo& info, const float (&x)[ITEMS], uint8_t* maskb) {
    __shared__ uint32_t tapcnt[kPackMaxTaps];
    const int tid = threadIdx.x;
    const int n = job.n;
    const float tv = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(info.thr_val)));
    const int ti = __builtin_amdgcn_readfirstlane(info.thr_idx);
    const bool upper = __builtin_amdgcn_readfirstlane(info.upper) != 0;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // The lower group: w < tv, or w = tv up to index ti, that is w <= tv in a thread's elements up to j_tie and w <= the
    // float below tv in those behind it.  (Not below -inf or NaN: nothing is lower then, as nothing is where tv or w is NaN.)
    const uint32_t tkey = float_to_key(tv);
    const float below = tv != tv ? tv : key_to_float(tkey == 0x80000000u ? tkey - 2u : tkey - 1u);   // (below zero: not -0)
    const int j_tie = ti < tid ? -1 : (ti - tid) / THREADS;
    if (job.T == 1) {
        static_assert(ITEMS <= 64 && THREADS / 64 <= kPackMaxTaps, "a lane per j, a count per wavefront");
        uint32_t w0 = 0, w1 = 0;
        uint32_t ones = 0;
        auto words = [&](auto in_alpha) {
            for_chunks<ITEMS>([&](auto c, auto e) {
                if (c * THREADS >= n) return false;                // (the whole workgroup)
                auto keep = [&](int j, unsigned long long m) {
                    ones += static_cast<uint32_t>(__builtin_popcountll(m));
                    w0 = write_lane(w0, static_cast<uint32_t>(m), j);
                    w1 = write_lane(w1, static_cast<uint32_t>(m >> 32), j);
                };
                if (e * THREADS <= n) {
#pragma unroll
                    for (int j = c; j < e; ++j) keep(j, __ballot(in_alpha(x[j], j <= j_tie ? tv : below)));
                } else {
#pragma unroll
                    for (int j = c; j < e; ++j)
                        keep(j, __ballot(in_alpha(x[j], j <= j_tie ? tv : below)) & __ballot(tid + j * THREADS < n));
                }
                return true;
            });
        };
        if (upper) words([](float v, float t) { return !(v <= t); });
        else words([](float v, float t) { return v <= t; });
        uint32_t* const E = job.E;
        const int R = job.Cw, Fp = job.Fp;
        const int r = lane * (THREADS / 32) + wave * 2;
        if (lane < ITEMS && r < R) E[static_cast<size_t>(r) * Fp + f] = w0;
        if (lane < ITEMS && r + 1 < R) E[static_cast<size_t>(r + 1) * Fp + f] = w1;
        if (lane == 0) tapcnt[wave] = ones;
        lds_barrier();
        if (tid == 0) {
            uint32_t total = 0;
            for (int w = 0; w < THREADS / 64; ++w) total += tapcnt[w];
            job.ecnt[f] = total;
        }
        return;
    }
    const uint8_t in_lower = upper ? 0 : 1, in_upper = upper ? 1 : 0;
    for_chunks<ITEMS>([&](auto c, auto e) {
        if (c * THREADS >= n) return false;
#pragma unroll
        for (int j = c; j < e; ++j)                                // (past n: nobody reads it)
            maskb[tid + j * THREADS] = x[j] <= (j <= j_tie ? tv : below) ? in_lower : in_upper;
        return true;
    });
    pack_bytes<THREADS>(job, f, maskb, tapcnt);
}
// The same from the row in memory (rows that were sorted).
template <int THREADS, int MAX_N>
__device__ __forceinline__ void pack_row_from(const MaskShape& job, int f, const SplitInfo& info, const float* __restrict__ row) {
    __shared__ uint8_t maskb[MAX_N];
    __shared__ uint32_t tapcnt[kPackMaxTaps];
    const float tv = info.thr_val;
    const int ti = info.thr_idx;
    const bool upper = info.upper != 0;
    for (int i = threadIdx.x; i < job.n; i += THREADS) {
        const float w = row[i];
        maskb[i] = (w < tv || (w == tv && i <= ti)) != upper ? 1 : 0;
    }
    pack_bytes<THREADS>(job, f, maskb, tapcnt);
}

}  // namespace dab
