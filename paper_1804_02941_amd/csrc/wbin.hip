// The weights-only layer (Section 5.1 of arXiv 1804.02941, WBin: real inputs, binarized weights) on the
// matrix cores, in one launch and without a copy of the operands in memory:
//   y = (alpha - beta) * sum x e + beta * sum x   (taps inside the image).
// Every fp32 input is split exactly into three bf16 pieces of eight significant bits, the mask bits become
// bf16 0 / 1, and v_mfma_f32_32x32x16_bf16 multiplies them: products exact, fp32 sums.  sum x is accumulated
// in double.  The instruction loses low bits of products much smaller than the accumulator, so the pieces are
// summed in one of two ways: rounded pieces (signs of their own, the losses cancel) in one accumulator, or cut
// pieces with a second accumulator for the last two.  Error against 64 bits, of the norm, over 1600 terms 5.5e-7
// and 8.6e-8 (cut pieces in one accumulator: 1.0e-6); over 4096 terms in eight shares 2.9e-7 and 1.0e-7.
//
// Both kernels read the fp32 input and the packed masks as they lie.
//   patch   layers of several taps: a workgroup owns 32 * NB consecutive output pixels x 128 filters.  The
//           padded pixels under its windows (one contiguous range of the flattened padded images) are split
//           once per 16 channels into LDS, and all taps read them there.
//   direct  one tap, few pixels, or windows whose pixels do not fit: fragments come straight from global
//           memory into registers and are split there; a workgroup's wavefronts share the reduction.
#include "mfma_tools.h"
#include "wbin.h"

namespace dab {

typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

constexpr uint32_t kOutside = 0x80000000u;             // a buffer offset past every tensor: the load returns zeros

// Orders LDS accesses of the workgroup without waiting for loads and stores of global memory.
__device__ __forceinline__ void wbin_lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// The upper halves of a and b (their leading eight bits as bf16) side by side, a in the low half; what is left of each
// stays in it, exactly.
__device__ __forceinline__ uint32_t take_piece(float& a, float& b) {
    const uint32_t p = __builtin_amdgcn_perm(__float_as_uint(b), __float_as_uint(a), 0x07060302u);
    a -= __uint_as_float(__float_as_uint(a) & 0xFFFF0000u);
    b -= __uint_as_float(__float_as_uint(b) & 0xFFFF0000u);
    return p;
}

// The same with a and b rounded to bf16 (to nearest even).
__device__ __forceinline__ uint32_t take_rounded_piece(float& a, float& b) {
    typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
    typedef float v2f __attribute__((ext_vector_type(2)));
    const uint32_t p = __builtin_bit_cast(uint32_t, __builtin_convertvector(v2f{a, b}, v2bf));
    a -= __uint_as_float(p << 16);
    b -= __uint_as_float(p & 0xFFFF0000u);
    return p;
}

// Eight mask bits (the rest zero) as eight bf16 values 0 / 1: bit pairs two bits apart in both halves of a
// word, then one multiplication per pair moves and widens them (0x3F80 = 1.0).
__device__ __forceinline__ v8bf expand_mask(uint32_t bits) {
    const uint32_t t = bits | (bits << 15);
    v4i w;
    w.x = __umul24(t & 0x00010001u, 0x3F80u);
    w.y = __umul24(t & 0x00040004u, 0x3F80u >> 2);
    w.z = __umul24(t & 0x00100010u, 0x3F80u >> 4);
    w.w = __umul24(t & 0x00400040u, 0x3F80u >> 6);
    return __builtin_bit_cast(v8bf, w);
}

// Four consecutive channels of one pixel (off: their byte offset, or kOutside or a little more).  Offsets are multiples
// of four, and a buffer load is checked per dword, so any channel count will do: the last pixel's channels past C lie past
// the end and read as zeros.  The whole offset is the vector one: the scalar offset is no part of what is checked.
__device__ __forceinline__ float4 load_channels(__amdgpu_buffer_rsrc_t x, uint32_t off) {
    const auto v = __builtin_amdgcn_raw_buffer_load_b128(x, off, 0, 0);
    return make_float4(__uint_as_float(v[0]), __uint_as_float(v[1]), __uint_as_float(v[2]), __uint_as_float(v[3]));
}
// Zeros in place of the n channels of v from c that lie past C (they are the next pixel's).
template <int N>
__device__ __forceinline__ void cut_channels(float (&v)[N], int c, int C) {
#pragma unroll
    for (int k = 0; k < N; ++k) v[k] = c + k < C ? v[k] : 0.0f;
}

__device__ __forceinline__ void store_y(float* y, float v, bool stream_out) {
    if (stream_out) __builtin_nontemporal_store(v, y);
    else *y = v;
}

// ---------------------------------------------------------------- patch
template <int NB, int WM>
__global__ __launch_bounds__(256, 2) void wbin_patch_kernel(const WbinGeom g, const float* __restrict__ X,
                                                            const uint32_t* __restrict__ E,
                                                            const float* __restrict__ alpha,
                                                            const float* __restrict__ beta, float* __restrict__ Y) {
    DAB_RESERVE_VGPRS();
    constexpr int WN = 4 / WM;                           // wavefronts along the filters; WM along the pixels
    constexpr int kFilters = 32 * NB * WN, kTile = 32 * WM;
    constexpr int SLOTS = kPatchSlots, kPix = SLOTS * 64; // pixels of the patch
    constexpr int kMaskTaps = 256 / kFilters;            // taps whose mask words one instruction brings
    extern __shared__ __align__(16) char lds[];          // [3 pieces][2 halves][kPix][16 bytes], then the mask words
    uint32_t* const mask = reinterpret_cast<uint32_t*>(lds + 6 * kPix * 16);     // [2][taps, rounded up to kMaskTaps][kFilters]
    const int unit = static_cast<int>(blockIdx.x & (kNumXCD - 1)) * g.per_xcd + static_cast<int>(blockIdx.x / kNumXCD);
    if (unit >= g.units) return;
    const int mt = fdiv(unit, g.d_ntiles);               // neighbouring workgroups of an XCD share pixels
    const int f0 = (unit - mt * g.n_ntiles) * kFilters;
    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;
    auto padded_pixel = [&](int m) {
        const int b = fdiv(m, g.d_HoWo);
        const int r = m - b * g.HoWo;
        const int oy = fdiv(r, g.d_Wo);
        return (b * g.Hp + oy * g.sh) * g.Wp + (r - oy * g.Wo) * g.sw;
    };
    const int m0 = mt * kTile;
    const int pp0 = padded_pixel(m0);
    const int np = padded_pixel(min(m0 + kTile, g.M) - 1) + (g.kh - 1) * g.Wp + g.kw - pp0;

    // A thread's slots: four channels of a pixel each, the same pixel for every group of 16 channels.
    const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(X), 0, g.x_bytes, 0x00020000);
    const int q = tid & 3;
    uint32_t off[SLOTS];
#pragma unroll
    for (int s = 0; s < SLOTS; ++s) {
        const int px = s * 64 + (tid >> 2);
        const int pp = pp0 + px;
        const int b = fdiv(pp, g.d_HpWp);
        const int r = pp - b * g.Hp * g.Wp;
        const int yp = fdiv(r, g.d_Wp);
        const int y = yp - g.ph, x = r - yp * g.Wp - g.pw;
        const bool in = px < np && y >= 0 && y < g.H && x >= 0 && x < g.W;
        off[s] = in ? static_cast<uint32_t>((b * g.H + y) * g.W + x) * static_cast<uint32_t>(g.C * 4) + 16 * q : kOutside;
    }
    float4 stage[SLOTS];
    auto load_group = [&](int grp) {
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) stage[s] = load_channels(xr, off[s] + 64 * grp);
    };
    // The mask words of 32 channels go straight into LDS, 1 KB (kMaskTaps taps) per wavefront instruction; filters past
    // the padded count and taps past the last repeat a valid word (nothing of them is used).
    const int tpad = (g.T + kMaskTaps - 1) / kMaskTaps * kMaskTaps;
    const int fq = min(f0 + 4 * (lane % (kFilters / 4)), g.Fp - 4), tq = lane / (kFilters / 4);
    auto load_mask = [&](int w) {
        uint32_t* const dst = mask + (w & 1) * tpad * kFilters;
        for (int t = kMaskTaps * wave; t < tpad; t += 4 * kMaskTaps) {
            const int tap = min(t + tq, g.T - 1);
            __builtin_amdgcn_global_load_lds(E + static_cast<size_t>(tap * g.Cw + w) * g.Fp + fq, dst + t * kFilters, 16, 0, 0);
        }
    };
    load_mask(0);
    load_group(0);

    const int m = min(m0 + wm * 32 + (lane & 31), g.M - 1);
    const char* const abase = lds + (half * kPix + padded_pixel(m) - pp0) * 16;
    const uint8_t* const bbase = reinterpret_cast<const uint8_t*>(mask + wn * NB * 32 + (lane & 31)) + half;
    double sum[SLOTS];
#pragma unroll
    for (int s = 0; s < SLOTS; ++s) sum[s] = 0.0;
    v16f acc[NB];                                        // (one set: rounded pieces)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[j][v] = 0.0f;

    for (int grp = 0; grp < g.C16; ++grp) {
        if (grp) wbin_lds_barrier();                     // the previous group's readers are done
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
            if (s * 64 >= np) break;
            float v[4] = {stage[s].x, stage[s].y, stage[s].z, stage[s].w};
            if (16 * grp + 16 > g.C) cut_channels(v, 16 * grp + 4 * q, g.C);
            sum[s] += (static_cast<double>(v[0]) + static_cast<double>(v[1])) + (static_cast<double>(v[2]) + static_cast<double>(v[3]));
            char* const dst = lds + ((q >> 1) * kPix + s * 64 + (tid >> 2)) * 16 + (q & 1) * 8;
#pragma unroll
            for (int p = 0; p < 3; ++p) {
                const uint32_t lo = take_rounded_piece(v[0], v[1]);
                *reinterpret_cast<uint2*>(dst + p * 2 * kPix * 16) = make_uint2(lo, take_rounded_piece(v[2], v[3]));
            }
        }
        __builtin_amdgcn_s_waitcnt(0);                   // the mask words have landed too (issued before these pixels)
        wbin_lds_barrier();
        if (grp + 1 < g.C16) {
            if (grp & 1) load_mask((grp + 1) >> 1);
            load_group(grp + 1);
        }
        // taps, the fragments of the next one read while this one multiplies
        const uint8_t* const bgrp = bbase + ((grp >> 1) & 1) * tpad * (4 * kFilters) + 2 * (grp & 1);
        v4i a[2][3];
        uint32_t bits[2][NB];
        int tap = 0, kx = 0, aoff = 0;
        const int row_step = (g.Wp - g.kw + 1) * 16;
        auto fetch = [&](int set) {
            const char* const ap = abase + aoff;
#pragma unroll
            for (int p = 0; p < 3; ++p) a[set][p] = *reinterpret_cast<const v4i*>(ap + p * 2 * kPix * 16);
#pragma unroll
            for (int j = 0; j < NB; ++j) bits[set][j] = bgrp[tap * (4 * kFilters) + j * 128];
            // past the end the last tap is read again (no branch: the waits would be merged at its end)
            const int more = tap + 1 < g.T, wrap = kx + 1 == g.kw;
            tap += more;
            kx = wrap ? 0 : kx + 1;
            aoff += more ? (wrap ? row_step : 16) : 0;
        };
        // One tap: the next tap's reads first, then the multiplies; the next tap's masks are widened between the
        // multiplies of the second and third piece (left to itself the compiler sinks the reads to their uses).
        v8bf b[2][NB];
        auto step = [&](int set) {
            fetch(set ^ 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int p = 0; p < 3; ++p) {
#pragma unroll
                for (int j = 0; j < NB; ++j)
                    acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, a[set][p]), b[set][j], acc[j], 0, 0, 0);
            }
#pragma unroll
            for (int j = 0; j < NB; ++j) b[set ^ 1][j] = expand_mask(bits[set ^ 1][j]);
            __builtin_amdgcn_sched_group_barrier(0x008, NB, 0);
#pragma unroll
            for (int i = 0; i < 2 * NB; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x002, 5, 0);
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        fetch(0);
#pragma unroll
        for (int j = 0; j < NB; ++j) b[0][j] = expand_mask(bits[0][j]);
        for (int t = 0;; t += 2) {
            step(0);
            if (t + 1 >= g.T) break;
            step(1);
            if (t + 2 >= g.T) break;
        }
    }

    // window sums: per-pixel sums over the patch, then each row's box sum
    double* const psum = reinterpret_cast<double*>(lds);
    float* const rows = reinterpret_cast<float*>(lds + kPix * 8);
    wbin_lds_barrier();
#pragma unroll
    for (int s = 0; s < SLOTS; ++s) {
        double v = sum[s];
        v += __shfl_xor(v, 1, 64);
        v += __shfl_xor(v, 2, 64);
        if (q == 0) psum[s * 64 + (tid >> 2)] = v;
    }
    wbin_lds_barrier();
    if (tid < kTile) {
        const double* p = psum + padded_pixel(min(m0 + tid, g.M - 1)) - pp0;
        double v = 0.0;
        for (int ky = 0; ky < g.kh; ++ky, p += g.Wp)
            for (int x = 0; x < g.kw; ++x) v += p[x];
        rows[tid] = static_cast<float>(v);
    }
    wbin_lds_barrier();
    float dcol[NB], bcol[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        const int f = min(f0 + (wn * NB + j) * 32 + (lane & 31), g.F - 1);
        bcol[j] = beta[f];
        dcol[j] = alpha[f] - bcol[j];
    }
    const int fl = f0 + wn * NB * 32 + (lane & 31);
    const bool whole = m0 + kTile <= g.M && f0 + kFilters <= g.F;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int r = wm * 32 + (v / 4) * 8 + half * 4 + v % 4;
        const float sx = rows[r];
        float* const y = Y + static_cast<size_t>(m0 + r) * g.F + fl;
#pragma unroll
        for (int j = 0; j < NB; ++j)
            if (whole || (m0 + r < g.M && fl + j * 32 < g.F))
                store_y(y + j * 32, fmaf(dcol[j], acc[j][v], bcol[j] * sx), g.stream_out);
    }
}

// ---------------------------------------------------------------- direct
constexpr int kDepth = 4;                                // steps in flight per wavefront

// ROWS pixels x 32 (ROWS = 32) or 16 filters a multiply, of 16 or 32 channels: lane l holds row (column) l % ROWS and
// the eight k of group l / ROWS; register v of the result is row (v / 4) * 8 + (l / ROWS) * 4 + v % 4, column l % ROWS.
template <int ROWS>
struct Tile;
template <>
struct Tile<32> {
    typedef v16f Acc;
    static __device__ __forceinline__ Acc multiply(v4i a, v8bf b, Acc c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, a), b, c, 0, 0, 0);
    }
};
template <>
struct Tile<16> {
    typedef float Acc __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ Acc multiply(v4i a, v8bf b, Acc c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, a), b, c, 0, 0, 0);
    }
};

template <int ROWS, int NB, int KS>
__global__ __launch_bounds__(512, ROWS * NB < 64 ? 4 : 2) void wbin_direct_kernel(const WbinGeom g, const float* __restrict__ X,
                                                                           const uint32_t* __restrict__ E,
                                                                           const float* __restrict__ alpha,
                                                                           const float* __restrict__ beta,
                                                                           float* __restrict__ Y) {
    DAB_RESERVE_VGPRS();
    constexpr int kBlocks = 8 / KS;                      // pixel blocks of a workgroup
    constexpr int kAcc = ROWS * ROWS / 64;               // accumulator registers of a multiply
    constexpr int kRegs = (kAcc * NB + KS - 1) / KS;     // of all, those that a wavefront finishes
    constexpr int kChan = 512 / ROWS;                    // channels of a step
    extern __shared__ __align__(16) char lds[];          // [8 wavefronts][ROWS] sums, then [8][kAcc NB][64] partial products
    const int unit = static_cast<int>(blockIdx.x & (kNumXCD - 1)) * g.per_xcd + static_cast<int>(blockIdx.x / kNumXCD);
    if (unit >= g.units) return;
    const int mt = fdiv(unit, g.d_ntiles);
    const int f0 = (unit - mt * g.n_ntiles) * ROWS * NB;
    const int lane = threadIdx.x & 63, col = lane & (ROWS - 1), kgrp = lane / ROWS;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int share = wave % KS;
    const int mb = (mt * kBlocks + wave / KS) * ROWS;
    const int m = min(mb + col, g.M - 1);
    const int b = fdiv(m, g.d_HoWo);
    const int r = m - b * g.HoWo;
    const int oy = fdiv(r, g.d_Wo);
    const int y0 = oy * g.sh - g.ph, x0 = (r - oy * g.Wo) * g.sw - g.pw;
    const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(X), 0, g.x_bytes, 0x00020000);

    const __amdgpu_buffer_rsrc_t er = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(E), 0, g.e_bytes, 0x00020000);

    // cursor over the steps [k0, k1): (tap, kChan channels), the channels fastest
    const int groups = kChan == 32 ? g.Cw : g.C16;
    const int steps = g.T * groups;
    const int per = (steps + KS - 1) / KS;
    const int k0 = min(share * per, steps), k1 = min(k0 + per, steps);
    int next = k0;
    int tap = fdiv(k0, kChan == 32 ? g.d_Cw : g.d_C16);
    int cg = k0 - tap * groups;
    int ky = fdiv(tap, g.d_kw), kx = tap - ky * g.kw;
    uint32_t off = 0;
    auto pixel_offset = [&]() {
        const int y = y0 + ky, x = x0 + kx;
        const bool in = y >= 0 && y < g.H && x >= 0 && x < g.W;
        return in ? static_cast<uint32_t>((b * g.H + y) * g.W + x) * static_cast<uint32_t>(g.C * 4) + 32 * kgrp : kOutside;
    };
    off = pixel_offset();
    float4 xq[kDepth][2];
    uint32_t bq[kDepth][NB];
    int cq[kDepth];                                      // the group of channels in a slot
    uint32_t fcol[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j) fcol[j] = 4 * min(f0 + j * ROWS + col, g.Fp - 1);
    auto fetch = [&](int slot) {
        // steps past the share read zeros (and some valid mask word)
        const uint32_t o = (next < k1 ? off : kOutside) + 4 * kChan * cg;
        xq[slot][0] = load_channels(xr, o);
        xq[slot][1] = load_channels(xr, o + 16);
        const int row = (tap * g.Cw + cg * kChan / 32) * g.Fp * 4;
#pragma unroll
        for (int j = 0; j < NB; ++j) bq[slot][j] = __builtin_amdgcn_raw_buffer_load_b32(er, fcol[j], row, 0);
        cq[slot] = cg;
        if (++next < k1 && ++cg == groups) {
            cg = 0;
            ++tap;
            if (++kx == g.kw) {
                kx = 0;
                ++ky;
            }
            off = pixel_offset();
        }
    };
    typename Tile<ROWS>::Acc acc[2][NB];                 // the first pieces' sums, the other two's
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int v = 0; v < kAcc; ++v) acc[p][j][v] = 0.0f;
    double sum = 0.0;
    if (k0 < k1) {
#pragma unroll
        for (int d = 0; d < kDepth; ++d) fetch(d);
        for (int s = k0; s < k1; s += kDepth) {
#pragma unroll
            for (int d = 0; d < kDepth; ++d) {
                float v[8] = {xq[d][0].x, xq[d][0].y, xq[d][0].z, xq[d][0].w, xq[d][1].x, xq[d][1].y, xq[d][1].z, xq[d][1].w};
                if (kChan * (cq[d] + 1) > g.C) cut_channels(v, kChan * cq[d] + 8 * kgrp, g.C);
                v8bf bv[NB];
#pragma unroll
                for (int j = 0; j < NB; ++j) bv[j] = expand_mask((bq[d][j] >> (kChan * cq[d] % 32 + 8 * kgrp)) & 0xFFu);
                fetch(d);
                sum += ((static_cast<double>(v[0]) + static_cast<double>(v[1])) + (static_cast<double>(v[2]) + static_cast<double>(v[3]))) +
                       ((static_cast<double>(v[4]) + static_cast<double>(v[5])) + (static_cast<double>(v[6]) + static_cast<double>(v[7])));
#pragma unroll
                for (int p = 0; p < 3; ++p) {
                    v4i a;
                    a.x = take_piece(v[0], v[1]);
                    a.y = take_piece(v[2], v[3]);
                    a.z = take_piece(v[4], v[5]);
                    a.w = take_piece(v[6], v[7]);
#pragma unroll
                    for (int j = 0; j < NB; ++j)
                        acc[p > 0][j] = Tile<ROWS>::multiply(a, bv[j], acc[p > 0][j]);
                }
            }
        }
    }

    // add the shares: every wavefront writes what it has and finishes its part of the registers
    double* const sums = reinterpret_cast<double*>(lds);
    float* const red = reinterpret_cast<float*>(lds + 8 * 32 * 8);
#pragma unroll
    for (int k = ROWS; k < 64; k *= 2) sum += __shfl_xor(sum, k, 64);
    if (kgrp == 0) sums[wave * 32 + col] = sum;
    if (KS > 1) {
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int v = 0; v < kAcc; ++v) red[((wave * NB + j) * kAcc + v) * 64 + lane] = acc[0][j][v] + acc[1][j][v];
    }
    wbin_lds_barrier();
    const int first = wave - share;                      // first wavefront of this pixel block
    if (kAcc * NB < KS && share >= kAcc * NB) return;
    constexpr int kCols = kRegs > kAcc ? kRegs / kAcc : 1, kRows = kRegs / kCols;
    const int j0 = share * kRegs / kAcc, v0 = share * kRegs % kAcc;
    float dcol[kCols], bcol[kCols];
#pragma unroll
    for (int j = 0; j < kCols; ++j) {
        const int f = min(f0 + (j0 + j) * ROWS + col, g.F - 1);
        bcol[j] = beta[f];
        dcol[j] = alpha[f] - bcol[j];
    }
#pragma unroll
    for (int i = 0; i < kRows; ++i) {
        const int v = v0 + i, rl = (v / 4) * 8 + kgrp * 4 + v % 4;
        double sx = sums[first * 32 + rl];
#pragma unroll
        for (int k = 1; k < KS; ++k) sx += sums[(first + k) * 32 + rl];
        const float sxf = static_cast<float>(sx);
        float* const y = Y + static_cast<size_t>(mb + rl) * g.F + f0 + j0 * ROWS + col;
#pragma unroll
        for (int j = 0; j < kCols; ++j) {
            float s1;
            if (KS > 1) {
                const float* const part = red + ((first * NB + j0 + j) * kAcc + v) * 64 + lane;
                s1 = part[0];
#pragma unroll
                for (int k = 1; k < KS; ++k) s1 += part[k * NB * kAcc * 64];
            } else {
                s1 = acc[0][j][i] + acc[1][j][i];
            }
            if (mb + rl < g.M && f0 + (j0 + j) * ROWS + col < g.F)
                store_y(y + j * ROWS, fmaf(dcol[j], s1, bcol[j] * sxf), g.stream_out);
        }
    }
}

// ---------------------------------------------------------------- host
static size_t patch_lds(int filters, int T) {
    const int taps = 256 / filters;
    return static_cast<size_t>(kPatchSlots) * 64 * 96 + 2 * static_cast<size_t>(ceil_div(T, taps) * taps) * filters * 4;
}
static size_t direct_lds(int rows, int nb, int ks) {
    return 8 * 32 * 8 + (ks > 1 ? static_cast<size_t>(8) * nb * rows * rows * 4 : 0);
}

// Pixels of the largest patch of n consecutive output pixels: whole rows and images in between, whatever their start.
static long long patch_pixels(const WbinGeom& g, int n) {
    n = n < g.M ? n : g.M;
    const long long rows = (n - 2 + g.Wo) / g.Wo, images = (n - 2 + g.HoWo) / g.HoWo;       // row and image changes at most
    const long long step = g.sw;
    const long long row = 1ll * g.sh * g.Wp - 1ll * (g.Wo - 1) * g.sw;
    const long long image = 1ll * g.Hp * g.Wp - (1ll * (g.Ho - 1) * g.sh * g.Wp + 1ll * (g.Wo - 1) * g.sw);
    const long long row_step = row > step ? row : step, image_step = image > row_step ? image : row_step;
    return (n - 1 - rows) * step + (rows - images) * row_step + images * image_step + 1ll * (g.kh - 1) * g.Wp + g.kw;
}

// The forms, with what their launches cost (us): a launch, then for every round of workgroups over the compute units a
// step of the reduction (of a wavefront's share), the round itself, and (direct) a tap of the share; (patch) per 16
// channels a tap, the group and 64 pixels of the patch, with one workgroup on a compute unit and with two.  Fitted to
// 304 random layers of 1e6 to 1.5e10 multiply-accumulates, every form timed on each (rms error 4-5 % patch, 6-11 %
// direct); on 152 others the form taken is 0.8 % slower than the fastest one in the geometric mean, at most 14 %, and
// 2.2 times faster than the kernels on expanded operands that these replaced (at least 1.08 times).  Times (us) at 61504 pixels x 128 filters x 25 taps x 64 channels:
// patch 4,4 68.7, 2,4 77.3, 2,2 74.2, direct 32,4,1 81.1, the others 96 and more (expanded: 81.8); 128 x 4096 x 1000, one
// tap: 155.5 (32,4,1), 44.6 (32,4,4), 21.2 (32,2,8), 13.7 (16,4,8), 12.4 (16,2,8), 19.7 (16,1,8), expanded 25.4;
// 51 x 152 x 8 x 23 -> 130, 3 x 3, stride 2: 10.4 (32,2,8), 13.0 (32,1,8), 29.5 (patch 2,2), expanded 33.6.
struct FormCost {
    WbinForm form;
    double launch, step, round, tap;                     // direct
    double tap1, group1, pix1, tap2, group2, pix2;       // patch
};
static const FormCost kForms[] = {
    {{0, 4, 4}, 6.96, 0, 0, 0, 0.259, 0.354, 0.0855, 0.576, 0.000, 0.1028},
    {{0, 2, 4}, 5.92, 0, 0, 0, 0.152, 0.421, 0.0759, 0.323, 0.579, 0.0000},
    {{0, 2, 2}, 6.36, 0, 0, 0, 0.151, 0.360, 0.0957, 0.270, 0.504, 0.0890},
    {{32, 4, 1}, 0.00, 0.582, 7.30, 0.133, 0, 0, 0, 0, 0, 0},
    {{32, 2, 1}, 0.00, 0.410, 5.96, 0.153, 0, 0, 0, 0, 0, 0},
    {{32, 4, 4}, 0.17, 0.593, 6.51, 0.334, 0, 0, 0, 0, 0, 0},
    {{32, 2, 4}, 1.10, 0.432, 4.18, 0.251, 0, 0, 0, 0, 0, 0},
    {{32, 2, 8}, 1.74, 0.445, 3.29, 0.253, 0, 0, 0, 0, 0, 0},
    {{32, 1, 8}, 3.49, 0.374, 1.07, 0.012, 0, 0, 0, 0, 0, 0},
    {{16, 4, 8}, 2.16, 0.552, 2.71, 0.000, 0, 0, 0, 0, 0, 0},
    {{16, 2, 8}, 3.65, 0.393, 0.84, 0.000, 0, 0, 0, 0, 0, 0},
    {{16, 1, 8}, 3.59, 0.343, 0.70, 0.000, 0, 0, 0, 0, 0, 0},
};

// The same for layers of more than 1e10 multiply-accumulates, where the many rounds of workgroups run into each other and the
// numbers above come out up to 19 % too high for the patch kernel: fitted to 98 layers of 6e9 to 6e10 (rms error 14-17 % patch,
// 8-14 % direct).  On the 81 of them above 1e10 the form taken is 0.6 % slower than the fastest one in the geometric mean, at most
// 13 %; by the numbers above 2.1 %, at most 19 %.  (us, form by those | by these: 57600 pixels x 9 taps x 256 channels -> 256
// 192 | 165, 50176 pixels 190 | 160, 28800 99.6 | 88.9.)
static const FormCost kLargeForms[] = {
    {{0, 4, 4}, 14.10, 0, 0, 0, 0.280, 0.190, 0.0000, 0.384, 0.728, 0.2271},
    {{0, 2, 4}, 9.52, 0, 0, 0, 0.172, 0.000, 0.0392, 0.228, 0.110, 0.2808},
    {{0, 2, 2}, 10.37, 0, 0, 0, 0.193, 0.000, 0.0000, 0.242, 0.479, 0.1556},
    {{32, 4, 1}, 3.76, 0.609, 7.03, 0.000, 0, 0, 0, 0, 0, 0},
    {{32, 2, 1}, 4.37, 0.457, 4.64, 0.000, 0, 0, 0, 0, 0, 0},
    {{32, 4, 4}, 5.51, 0.606, 5.25, 0.115, 0, 0, 0, 0, 0, 0},
    {{32, 2, 4}, 7.22, 0.440, 3.62, 0.045, 0, 0, 0, 0, 0, 0},
    {{32, 2, 8}, 9.26, 0.456, 2.84, 0.071, 0, 0, 0, 0, 0, 0},
    {{32, 1, 8}, 6.81, 0.375, 0.93, 0.000, 0, 0, 0, 0, 0, 0},
    {{16, 4, 8}, 4.96, 0.563, 2.60, 0.000, 0, 0, 0, 0, 0, 0},
    {{16, 2, 8}, 25.09, 0.348, 1.02, 0.000, 0, 0, 0, 0, 0, 0},
    {{16, 1, 8}, 24.02, 0.358, 0.80, 0.000, 0, 0, 0, 0, 0, 0},
};
constexpr double kLargeMacs = 1e10;

// What the layer may be, and the workspace that its callers bring: the room that the expanded operands once took.  The
// kernels use none of it, but a call with less is refused as it always was.
int wbin_workspace(const dab_conv_desc& d, size_t* bytes) {
    auto round256 = [](size_t n) { return (n + 255) & ~static_cast<size_t>(255); };
    const long long Ho = (1ll * d.H + 2ll * d.pad_h - d.kh) / d.stride_h + 1, Wo = (1ll * d.W + 2ll * d.pad_w - d.kw) / d.stride_w + 1;
    const long long M = 1ll * d.B * Ho * Wo, npix = 1ll * d.B * (d.H + 2ll * d.pad_h) * (d.W + 2ll * d.pad_w);
    const long long T = 1ll * d.kh * d.kw, c16 = ceil_div(d.C, 16), nk = 3 * T * c16, n_ntiles = ceil_div(d.F, 128);
    if (M >= (1ll << 30) || npix * c16 * 96 >= (1ll << 31) || nk >= (1 << 20) || M * d.F >= (1ll << 40) || n_ntiles * nk >= (1ll << 22))
        return DAB_ERR_UNSUPPORTED;
    *bytes = round256(static_cast<size_t>(npix * c16 * 96)) + static_cast<size_t>(n_ntiles * T * c16) * 4096 +
             round256(static_cast<size_t>(M) * 4) + round256(static_cast<size_t>(npix) * 4) + round256(static_cast<size_t>(nk + 16 + T) * 4);
    return DAB_OK;
}

void plan_wbin(const dab_conv_desc& d, WbinPlan* pl) {
    WbinGeom& g = pl->g;
    g = WbinGeom{};
    g.H = d.H; g.W = d.W; g.C = d.C; g.F = d.F; g.kh = d.kh; g.kw = d.kw;
    g.ph = d.pad_h; g.pw = d.pad_w; g.sh = d.stride_h; g.sw = d.stride_w;
    g.Cw = ceil_div(d.C, 32); g.C16 = ceil_div(d.C, 16); g.Fp = 64 * ceil_div(d.F, 64);
    g.Ho = (d.H + 2 * d.pad_h - d.kh) / d.stride_h + 1;
    g.Wo = (d.W + 2 * d.pad_w - d.kw) / d.stride_w + 1;
    g.HoWo = g.Ho * g.Wo; g.M = d.B * g.HoWo; g.T = d.kh * d.kw;
    g.Hp = d.H + 2 * d.pad_h; g.Wp = d.W + 2 * d.pad_w;
    g.x_bytes = static_cast<uint32_t>(4ll * d.B * d.H * d.W * d.C);
    g.e_bytes = static_cast<uint32_t>(4ll * g.T * g.Cw * g.Fp);
    g.d_HoWo = make_fastdiv(g.HoWo); g.d_Wo = make_fastdiv(g.Wo); g.d_Wp = make_fastdiv(g.Wp);
    g.d_HpWp = make_fastdiv(g.Hp * g.Wp); g.d_kw = make_fastdiv(g.kw); g.d_C16 = make_fastdiv(g.C16);
    g.d_Cw = make_fastdiv(g.Cw);
    g.stream_out = 4ll * g.M * g.F > (64ll << 20);

    pl->us = 1e30;
    static_assert(sizeof kForms == sizeof kLargeForms, "the same forms");
    const bool large = 1.0 * g.M * d.F * d.C * g.T > kLargeMacs;
    for (const FormCost& k : large ? kLargeForms : kForms) {
        const WbinForm& f = k.form;
        int pixels, filters;
        size_t lds;
        double us;
        if (f.rows == 0) {
            pixels = 32 * f.v;
            filters = 32 * f.nb * (4 / f.v);
            lds = patch_lds(filters, g.T);
            const long long slots = (patch_pixels(g, pixels) + 63) / 64;
            if (g.T < 2 || lds > kWbinMaxLds || slots > kPatchSlots) continue;
            const int resident = lds <= kWbinMaxLds / 2 ? 2 : 1;
            const long long units = 1ll * ceil_div(g.M, pixels) * ceil_div(g.F, filters);
            const long long full = units / (kNumCU * resident), rest = units % (kNumCU * resident);
            const long long n2 = (resident == 2 ? full : 0) + (rest > kNumCU), n1 = (resident == 1 ? full : 0) + (rest > 0 && rest <= kNumCU);
            us = k.launch + g.C16 * (static_cast<double>(n1) * (g.T * k.tap1 + k.group1 + static_cast<double>(slots) * k.pix1) +
                                     static_cast<double>(n2) * (g.T * k.tap2 + k.group2 + static_cast<double>(slots) * k.pix2));
        } else {
            pixels = f.rows * 8 / f.v;
            filters = f.rows * f.nb;
            lds = direct_lds(f.rows, f.nb, f.v);
            const int steps = ceil_div(g.T * (f.rows == 16 ? g.Cw : g.C16), f.v);
            const long long units = 1ll * ceil_div(g.M, pixels) * ceil_div(g.F, filters), rounds = (units + kNumCU - 1) / kNumCU;
            us = k.launch + static_cast<double>(rounds) * (steps * k.step + k.round + (g.T > 1 ? k.tap * g.T / f.v : 0.0));
        }
        if (us >= pl->us) continue;
        pl->us = us;
        pl->form = f;
        pl->lds_bytes = lds;
        g.n_ntiles = ceil_div(g.F, filters);
        g.units = ceil_div(g.M, pixels) * g.n_ntiles;
    }
    g.per_xcd = ceil_div(g.units, kNumXCD);
    g.d_ntiles = make_fastdiv(g.n_ntiles);
    pl->grid = static_cast<unsigned>(g.per_xcd) * kNumXCD;
}

// Calls f with the kernel of a form and its threads.
template <typename Fn>
static int with_kernel(const WbinForm& w, Fn f) {
    if (w.rows == 0) {
        if (w.nb == 4) return f(wbin_patch_kernel<4, 4>, 256);
        return w.v == 4 ? f(wbin_patch_kernel<2, 4>, 256) : f(wbin_patch_kernel<2, 2>, 256);
    }
    if (w.rows == 32) {
        if (w.nb == 4) return w.v == 1 ? f(wbin_direct_kernel<32, 4, 1>, 512) : f(wbin_direct_kernel<32, 4, 4>, 512);
        if (w.nb == 1) return f(wbin_direct_kernel<32, 1, 8>, 512);
        return w.v == 1 ? f(wbin_direct_kernel<32, 2, 1>, 512) : w.v == 4 ? f(wbin_direct_kernel<32, 2, 4>, 512)
                                                                          : f(wbin_direct_kernel<32, 2, 8>, 512);
    }
    if (w.nb == 4) return f(wbin_direct_kernel<16, 4, 8>, 512);
    return w.nb == 2 ? f(wbin_direct_kernel<16, 2, 8>, 512) : f(wbin_direct_kernel<16, 1, 8>, 512);
}

int launch_wbin(const WbinPlan& pl, hipStream_t st, const float* X, const uint32_t* E, const float* alpha, const float* beta,
                float* Y) {
    return with_kernel(pl.form, [&](auto kernel, int threads) {
        return launch(kernel, dim3(pl.grid), dim3(threads), pl.lds_bytes, st, pl.g, X, E, alpha, beta, Y);
    });
}

// The patches and partial products take more dynamic LDS than a launch is granted by default.
int init_wbin() {
    for (const FormCost& k : kForms) {
        const int rc = with_kernel(k.form, [](auto kernel, int) {
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, kWbinMaxLds);
            return e == hipSuccess ? static_cast<int>(DAB_OK) : hip_failed(e);
        });
        if (rc) return rc;
    }
    return DAB_OK;
}

}  // namespace dab
