// Binarized convolution / fully-connected product on the matrix cores (gfx950).
//
// Section 4.3.2 of arXiv 1804.02941: the layer output is the ordinary convolution of the
// +1/-1 input with the two-valued filter W~ = alpha*e + beta*(1-e) (Section 4.1), i.e.
//   y = alpha*s1 + beta*s2,  s1 = sum_i a_i e_i,  s1 + s2 = sA = sum_i a_i   (taps inside the image).
// s1 is a dense contraction, so it runs on the MFMA units: both operands are expanded from
// their packed bits to 4-bit floats (E2M1: +1 = 0x2, -1 = 0xA, 0 = 0x0 for padding), which
// every product and, in the fp32 accumulator, every sum below 2^24 represents exactly, and
// multiplied with v_mfma_f32_32x32x64_f8f6f4.  Measured on MI355X this
// instruction sustains 4.2e15 multiply-accumulates/s at 4 bits per operand element, 6.7 times
// the AND + BCNT ceiling of the vector ALU on the same bits, which is why the popcount form
// of the product is not the one that ships.
//
// A launch is two or three kernels:
//   prepare   one streaming kernel whose blocks (a) expand the activation bits to fp4, with a
//             zero halo of the padding width so the main loop needs no bounds checks, laid out
//             as planes [32-channel word][padded pixel][16 bytes] (a half-wavefront then reads
//             512 contiguous bytes for 32 neighbouring pixels), (b) expand the weight bits to
//             fp4 in the order B fragments are consumed, (c) sum the +1/-1 inputs of every
//             padded pixel, (d) write the table of A4 byte offsets of the k-steps (k-steps run
//             over the taps of one 64-channel block, then the next block, so consecutive steps
//             touch neighbouring pixels of the same planes), and, for split launches, (e) sA;
//   main      one workgroup owns 128 filters and keeps their B fragments in LDS (the whole
//             reduction if it fits in 144 KB, else chunk by chunk).  Each wavefront computes
//             64 pixels x 128 filters: A fragments (32 pixels x 64 channels, 16 bytes per lane)
//             come from global memory by buffer loads (pixel offset per lane, k-step offset in
//             a scalar register read from the table) through a queue of register slots, B
//             fragments from LDS one step ahead, accumulators stay in registers.  The eight
//             MFMAs of a k-step are issued with one LDS read or buffer load in the shadow of
//             each (measured: issued back to back in front of them, the memory instructions
//             cost their full issue time).  Big layers run persistent workgroups (one per
//             compute unit) that walk over pixel tiles and write y directly; sA of a row is the
//             box sum of the per-pixel sums over the window, read before the reduction loop.
//             Layers too small to fill the chip are also split along the reduction and write
//             their exact partial sums to the workspace;
//   finish    (split launches only) adds the partials, y = (alpha-beta)*s1 + beta*sA.
// Layers with at most 512 output blocks of 32 x 32 skip main and finish for the small-product
// kernel further down (one workgroup per block, no partial sums in memory).
#include "dab_internal.h"
#include "mfma_tools.h"
#include "wbin.h"

namespace dab {

constexpr int kNTile = 128;          // filters per workgroup
constexpr int kMaxChunk = 36;        // k-steps of B fragments held in LDS at a time (36 x 4 KB)
constexpr int kPrefetch = 4;         // A fragments in flight per 32-pixel row block
constexpr int kTabPad = 16;          // entries of the k-step offset table past the last step

struct MfmaGeom {
    int B, H, W, F, kh, kw, ph, pw, sh, sw;
    int C, Cw, KB;                 // channels, 32-bit words per pixel, 64-channel blocks per tap
    int Ho, Wo, HoWo, M, Hp, Wp, Fp;
    int nk;                        // k-steps of the whole reduction: taps x KB
    int ksplit, split_steps;       // reduction splits and k-steps per split
    int kchunk;                    // k-steps staged in LDS at a time
    int n_ntiles, n_mtiles;        // 128-filter tiles, pixel tiles of 64 * WAVES
    int wg_per_ntile;              // persistent workgroups per filter tile (direct mode)
    int T, npix, plane;            // taps, padded pixels, bytes of one 32-channel plane of A4
    int act_p, act_w, act_wt;      // prepare: pixels x words of a transpose tile (product 256), word tiles
    int sum_shift;                 // prepare: log2 of the lanes that share one pixel's row sum
    int n_fblocks;                 // 32-filter column blocks (small products)
    FastDiv d_HoWo, d_Wo, d_Wp, d_HpWp, d_nk, d_mtiles, d_ksplit, d_T, d_kw, d_act_wt, d_Cw, d_fblocks;
    // block ranges of the prepare kernel
    unsigned blk_act, blk_wgt, blk_sum, blk_tab, blk_sa;
};

// 8 bits -> 8 nibbles, bit i in bit 0 of nibble i.
__device__ __forceinline__ uint32_t spread8(uint32_t x) {
    x = (x | (x << 12)) & 0x000F000Fu;
    x = (x | (x << 6)) & 0x03030303u;
    x = (x | (x << 3)) & 0x11111111u;
    return x;
}

// 8 bits -> 8 fp4 codes (4 bytes): every byte holds two codes, so it takes one of four values, picked
// by a byte permute from `lut` (byte v = the codes of the bit pair v) with the bit pairs as selectors.
__device__ __forceinline__ uint32_t expand8(uint32_t x, uint32_t lut) {
    x = (x | (x << 12)) & 0x000F000Fu;
    x = (x | (x << 6)) & 0x03030303u;                       // byte j = bits 2j, 2j+1
    return __builtin_amdgcn_perm(0u, lut, x);
}
constexpr uint32_t kLutPlusMinus = 0x222AA2AAu;            // bit 1 -> +1.0 (0x2), bit 0 -> -1.0 (0xA)
constexpr uint32_t kLutOneZero = 0x22200200u;              // bit 1 -> 1.0 (0x2), bit 0 -> 0

// ---------------------------------------------------------------- prepare
__global__ __launch_bounds__(256) void binconv_prepare_kernel(const MfmaGeom g, const uint32_t* __restrict__ A,
                                                              const uint32_t* __restrict__ E,
                                                              uint4* __restrict__ A4, uint4* __restrict__ E4,
                                                              int32_t* __restrict__ pixsum, int32_t* __restrict__ ktab,
                                                              float* __restrict__ sA) {
    __shared__ uint4 tile[256];
    unsigned blk = blockIdx.x;
    if (blk < g.blk_act) {
        // activations: 32 channels (one bit word) of a padded pixel become 16 bytes of fp4, written as
        // planes [word][padded pixel] so that a half-wavefront of the main kernel reads 512 contiguous
        // bytes for 32 neighbouring pixels.  A block transposes a tile of act_p pixels x act_w words
        // through LDS: bit words are read along the channels, fp4 is written along the pixels.
        const int tp = fdiv(static_cast<int>(blk), g.d_act_wt);            // pixel tile
        const int tw = static_cast<int>(blk) - tp * g.act_wt;              // word tile
        {
            const int pl = threadIdx.x / g.act_w, wl = threadIdx.x - pl * g.act_w;
            const int pp = tp * g.act_p + pl, w = tw * g.act_w + wl;
            uint4 out = make_uint4(0, 0, 0, 0);
            if (pp < g.npix && w < g.Cw) {
                const int b = fdiv(pp, g.d_HpWp);
                const int r = pp - b * g.Hp * g.Wp;
                const int yp = fdiv(r, g.d_Wp);
                const int y = yp - g.ph, x = r - yp * g.Wp - g.pw;
                if (y >= 0 && y < g.H && x >= 0 && x < g.W) {
                    const uint32_t bits = A[((static_cast<size_t>(b) * g.H + y) * g.W + x) * g.Cw + w];
                    const int nv = min(32, g.C - 32 * w);
                    uint32_t o[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) o[q] = expand8((bits >> (8 * q)) & 0xFFu, kLutPlusMinus);
                    if (nv < 32) {                                      // channels past C -> 0
                        const uint32_t valid = (1u << nv) - 1u;
#pragma unroll
                        for (int q = 0; q < 4; ++q) o[q] &= spread8((valid >> (8 * q)) & 0xFFu) * 0xFu;
                    }
                    out = make_uint4(o[0], o[1], o[2], o[3]);
                }
            }
            tile[threadIdx.x] = out;
        }
        __syncthreads();
        {
            const int wl = threadIdx.x / g.act_p, pl = threadIdx.x - wl * g.act_p;
            const int pp = tp * g.act_p + pl, w = tw * g.act_w + wl;
            if (pp < g.npix && w < 2 * g.KB) A4[static_cast<size_t>(w) * g.npix + pp] = tile[pl * g.act_w + wl];
        }
        return;
    }
    blk -= g.blk_act;
    if (blk < g.blk_wgt) {
        // weights: bits [R][Fp] -> fragments [ntile][kstep][4 column blocks][k half][32 filters][16 bytes];
        // k-steps run over the taps of one 64-channel block, then the next block
        const long long i = 1ll * blk * 256 + threadIdx.x;
        if (i >= 1ll * g.n_ntiles * g.nk * 256) return;
        const int fl = static_cast<int>(i & 31);
        const int half = static_cast<int>((i >> 5) & 1);
        const int nf = static_cast<int>((i >> 6) & 3);
        const int tk = static_cast<int>(i >> 8);
        const int nt = fdiv(tk, g.d_nk);
        const int ks = tk - nt * g.nk;
        const int kb = fdiv(ks, g.d_T);
        const int tap = ks - kb * g.T;
        const int w = 2 * kb + half;
        const int f = nt * kNTile + nf * 32 + fl;
        uint4 out = make_uint4(0, 0, 0, 0);
        if (w < g.Cw && f < g.Fp) {
            const uint32_t bits = E[static_cast<size_t>(tap * g.Cw + w) * g.Fp + f];
            out = make_uint4(expand8(bits & 0xFFu, kLutOneZero), expand8((bits >> 8) & 0xFFu, kLutOneZero),
                             expand8((bits >> 16) & 0xFFu, kLutOneZero), expand8(bits >> 24, kLutOneZero));
        }
        E4[i] = out;
        return;
    }
    blk -= g.blk_wgt;
    if (blk < g.blk_sum) {
        // per padded pixel: sum of its +1/-1 inputs (0 in the halo); sA of an output is the box sum of
        // these.  sum_tpp lanes (a power of two) share one pixel's words.
        const int gi = static_cast<int>(blk * 256 + threadIdx.x);
        const int pp = gi >> g.sum_shift, sub = gi & ((1 << g.sum_shift) - 1);
        int ones = 0;
        bool inside = false;
        if (pp < g.npix) {
            const int b = fdiv(pp, g.d_HpWp);
            const int r = pp - b * g.Hp * g.Wp;
            const int yp = fdiv(r, g.d_Wp);
            const int y = yp - g.ph, x = r - yp * g.Wp - g.pw;
            inside = y >= 0 && y < g.H && x >= 0 && x < g.W;
            if (inside) {
                const uint32_t* px = A + ((static_cast<size_t>(b) * g.H + y) * g.W + x) * g.Cw;
                for (int w = sub; w < g.Cw; w += 1 << g.sum_shift) ones += __builtin_popcount(px[w]);
            }
        }
        for (int d = 1; d < (1 << g.sum_shift); d <<= 1) ones += __shfl_xor(ones, d, 64);
        if (pp >= g.npix || sub != 0) return;
        const int v = inside ? 2 * ones - g.C : 0;
        pixsum[pp] = v;
        return;
    }
    blk -= g.blk_sum;
    if (blk < g.blk_tab) {
        // byte offset into A4 of every k-step (taps of one 64-channel block, then the next block);
        // entries past the end repeat the last step
        const int i = static_cast<int>(blk * 256 + threadIdx.x);
        if (i >= g.nk + kTabPad) return;
        const int ks = min(i, g.nk - 1);
        const int kb = fdiv(ks, g.d_T);
        const int tap = ks - kb * g.T;
        const int ky = fdiv(tap, g.d_kw);
        const int kx = tap - ky * g.kw;
        ktab[i] = kb * 2 * g.plane + (ky * g.Wp + kx) * 16;
        return;
    }
    blk -= g.blk_tab;
    {
        // split launches only: sA of every output pixel, one wavefront per pixel, lanes over the
        // (tap, word) pairs of its window
        const int m = static_cast<int>(blk * 4 + (threadIdx.x >> 6));
        if (m >= g.M) return;
        const int lane = threadIdx.x & 63;
        const int b = fdiv(m, g.d_HoWo);
        const int r = m - b * g.HoWo;
        const int oy = fdiv(r, g.d_Wo);
        const int ox = r - oy * g.Wo;
        int acc = 0;
        for (int it = lane; it < g.T * g.Cw; it += 64) {
            const int tap = fdiv(it, g.d_Cw);
            const int w = it - tap * g.Cw;
            const int ky = fdiv(tap, g.d_kw);
            const int kx = tap - ky * g.kw;
            const int y = oy * g.sh - g.ph + ky, x = ox * g.sw - g.pw + kx;
            if (y >= 0 && y < g.H && x >= 0 && x < g.W) {
                const int nv = min(32, g.C - 32 * w);
                acc += 2 * __builtin_popcount(A[((static_cast<size_t>(b) * g.H + y) * g.W + x) * g.Cw + w]) - nv;
            }
        }
        for (int d = 1; d < 64; d <<= 1) acc += __shfl_xor(acc, d, 64);
        if (lane == 0) sA[m] = static_cast<float>(acc);
    }
}

// ---------------------------------------------------------------- main
// One group of the k-step schedule: an MFMA, then at most one LDS read or one buffer load in its shadow.
#define DAB_SLOT_DS()   do { __builtin_amdgcn_sched_group_barrier(0x008, 1, 0); __builtin_amdgcn_sched_group_barrier(0x100, 1, 0); } while (0)
#define DAB_SLOT_VMEM() do { __builtin_amdgcn_sched_group_barrier(0x008, 1, 0); __builtin_amdgcn_sched_group_barrier(0x020, 1, 0); } while (0)
#define DAB_SLOT_NONE() do { __builtin_amdgcn_sched_group_barrier(0x008, 1, 0); } while (0)

template <int WAVES, int MODE>
__global__ __launch_bounds__(64 * WAVES) void binconv_mfma_kernel(const MfmaGeom g, const char* __restrict__ A4,
                                                                  const uint4* __restrict__ E4,
                                                                  const float* __restrict__ alpha,
                                                                  const float* __restrict__ beta,
                                                                  float* __restrict__ Y, int32_t* __restrict__ dbg_s1,
                                                                  float* __restrict__ ws_s1, float* __restrict__ ws_sA,
                                                                  const int32_t* __restrict__ pixsum,
                                                                  const int32_t* __restrict__ ktab,
                                                                  const float* __restrict__ tau_out,
                                                                  uint32_t* __restrict__ out_bits) {
    constexpr int THREADS = 64 * WAVES;
    constexpr int MTILE = 64 * WAVES;
    extern __shared__ __align__(16) uint4 panel[];                 // [kchunk][4][64 lanes] 16-byte groups
    __shared__ __align__(16) float sA_lds[WAVES][64];              // row sums of each wavefront's 64 pixels

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int ntile, mt_first, mt_step, kbeg, kend, ksplit_id = 0;
    if (MODE == kOutSplit) {
        // one unit per workgroup: (filter tile, pixel tile, reduction split)
        const int u = fdiv(blockIdx.x, g.d_ksplit);
        const int ks = blockIdx.x - u * g.ksplit;
        ksplit_id = ks;
        ntile = fdiv(u, g.d_mtiles);
        mt_first = u - ntile * g.n_mtiles;
        mt_step = g.n_mtiles;                                      // a single tile
        kbeg = ks * g.split_steps;
        kend = min(g.nk, kbeg + g.split_steps);
    } else {
        ntile = blockIdx.x / g.wg_per_ntile;
        mt_first = blockIdx.x - ntile * g.wg_per_ntile;
        mt_step = g.wg_per_ntile;
        kbeg = 0;
        kend = g.nk;
    }
    const int f0 = ntile * kNTile;
    const uint4* Epanel = E4 + static_cast<size_t>(ntile) * g.nk * 256;
    const int nchunks = (kend - kbeg + g.kchunk - 1) / g.kchunk;
    // A4 as a buffer resource: the per-lane pixel offset rides in a VGPR, the k-step offset in an SGPR
    const __amdgpu_buffer_rsrc_t a4rsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(A4), 0, 2 * g.KB * g.plane, 0x00020000);

    // per-lane scalars of the four 32-filter column blocks
    float dcol[4], bcol[4], tcol[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int f = min(f0 + j * 32 + (lane & 31), g.F - 1);
        const float al = alpha[f], be = beta[f];
        dcol[j] = al - be;
        bcol[j] = be;
        tcol[j] = (MODE == kOutBits && tau_out) ? tau_out[f] : 0.0f;
    }

    // The B fragments go straight from global memory into LDS (16 bytes per lane, 1 KB per wavefront
    // instruction, no registers in between), all of a chunk in flight at once.  Workgroups of one
    // filter tile read the same panel; each starts at another KB.  Steps past the end of the chunk
    // (it is rounded up to the prefetch depth) hold zeros.
    auto stage_panel = [&](int ks0, int ks1, int steps) {
        const int nkb = (ks1 - ks0) * 4;                           // 1 KB pieces: 64 groups of 16 bytes
        const int rot = blockIdx.x % nkb;
        for (int i = wave; i < nkb; i += WAVES) {
            int kb = i + rot;
            kb = kb >= nkb ? kb - nkb : kb;
            __builtin_amdgcn_global_load_lds(Epanel + static_cast<size_t>(ks0) * 256 + kb * 64 + lane, panel + kb * 64, 16,
                                             0, 0);
        }
        for (int e = nkb * 64 + tid; e < steps * 256; e += THREADS) panel[e] = make_uint4(0, 0, 0, 0);
    };
    // A reduction that fits in LDS is staged once, and its copies are issued first of all so that
    // they fly while the first tile's addresses and row sums are worked out.
    bool staged = false;
    if (nchunks == 1 && mt_first < g.n_mtiles) stage_panel(kbeg, kend, (kend - kbeg + kPrefetch - 1) / kPrefetch * kPrefetch);
    for (int mt = mt_first; mt < g.n_mtiles; mt += mt_step) {
        const int m_base = mt * MTILE + wave * 64;
        int pixoff[2], mypix = 0;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int m = min(m_base + i * 32 + (lane & 31), g.M - 1);
            const int b = fdiv(m, g.d_HoWo);
            const int r = m - b * g.HoWo;
            const int oy = fdiv(r, g.d_Wo);
            const int ox = r - oy * g.Wo;
            const int pix = (b * g.Hp + oy * g.sh) * g.Wp + ox * g.sw;
            pixoff[i] = pix * 16 + (lane >> 5) * g.plane;
            if (i == (lane >> 5)) mypix = pix;                         // lane l owns row l of the 64 for the row sums
        }
        // sA of this lane's row: box sum of the per-pixel sums over the filter window (the first T
        // entries of the k-step table are the window's pixel offsets, times 16).  Thirty-two loads at a
        // time (a 5x5 window is one round trip); the result is needed only after the reduction loop.
        float rowsum = 0.0f;
        if (MODE != kOutSplit) {
            int sum = 0;
            for (int t0 = 0; t0 < g.T; t0 += 32) {
                int v[32];
#pragma unroll
                for (int u = 0; u < 32; ++u) v[u] = pixsum[mypix + (ktab[min(t0 + u, g.T - 1)] >> 4)];
#pragma unroll
                for (int u = 0; u < 32; ++u) sum += t0 + u < g.T ? v[u] : 0;
            }
            rowsum = static_cast<float>(sum);
        }
        v16f acc[2][4];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;

        for (int chunk = 0; chunk < nchunks; ++chunk) {
            const int ks0 = kbeg + chunk * g.kchunk;
            const int ks1 = min(kend, ks0 + g.kchunk);
            // panel entries of this chunk rounded up to a queue round; the extra k-steps multiply
            // zero B fragments (and read some valid A fragment), so the loop has no tail
            const int steps = (ks1 - ks0 + kPrefetch - 1) / kPrefetch * kPrefetch;
            if (nchunks > 1) {
                __syncthreads();                                   // previous users of the panel are done
                stage_panel(ks0, ks1, steps);
            }
            // A fragments: a queue of kPrefetch k-steps per row block, refilled as it drains.  The byte
            // offset of a k-step comes from the table the prepare kernel wrote (four per scalar
            // load); steps past the end read a valid fragment against zero B fragments.
            auto load_a = [&](int i, int poff) -> v4i {
                const auto v = __builtin_amdgcn_raw_buffer_load_b128(a4rsrc, pixoff[i], poff, 0);
                return v4i{static_cast<int>(v[0]), static_cast<int>(v[1]), static_cast<int>(v[2]), static_cast<int>(v[3])};
            };
            // Slot d of the queue holds the fragments of step st + d; the slot emptied by the previous
            // step is refilled during this one (kPrefetch - 1 steps ahead), so a register is never live as
            // both a pending load and an operand and the loop carries no copies.  The first
            // fragments are requested before the wait for the panel, so both latencies overlap.
            const int* kt = ktab + ks0;
            v4i abuf[kPrefetch][2];
#pragma unroll
            for (int d = 0; d < kPrefetch - 1; ++d) {
                const int p = kt[d];
#pragma unroll
                for (int i = 0; i < 2; ++i) abuf[d][i] = load_a(i, p);
            }
            if (nchunks > 1) {
                __builtin_amdgcn_s_waitcnt(0);                     // every counter to zero: the copies have landed
                __syncthreads();
            } else if (!staged) {
                // the copies were issued before the first tile's address work and row sums
                __builtin_amdgcn_s_waitcnt(0);
                __syncthreads();
                staged = true;
            }
            const uint4* bp = panel + lane;
            uint4 bq[2][4];
#pragma unroll
            for (int j = 0; j < 4; ++j) bq[0][j] = bp[j * 64];
            for (int st = 0; st < steps; st += kPrefetch) {
#pragma unroll
                for (int d = 0; d < kPrefetch; ++d) {
                    constexpr int kAhead = kPrefetch - 1;
                    // B fragments of the next step are read while this one multiplies
                    const uint4* bn = bp + static_cast<size_t>(min(st + d + 1, steps - 1)) * 256;
#pragma unroll
                    for (int j = 0; j < 4; ++j) bq[(d + 1) & 1][j] = bn[j * 64];
                    const int p = kt[st + d + kAhead];
                    abuf[(d + kAhead) % kPrefetch][0] = load_a(0, p);
                    abuf[(d + kAhead) % kPrefetch][1] = load_a(1, p);
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const uint4 bu = bq[d & 1][j];
                        const v4i bv = {static_cast<int>(bu.x), static_cast<int>(bu.y), static_cast<int>(bu.z),
                                        static_cast<int>(bu.w)};
                        acc[0][j] = mfma_fp4(abuf[d][0], bv, acc[0][j]);
                        acc[1][j] = mfma_fp4(abuf[d][1], bv, acc[1][j]);
                    }
                    // issue order of this k-step: every memory instruction in the shadow of an MFMA
                    DAB_SLOT_DS(); DAB_SLOT_DS(); DAB_SLOT_DS(); DAB_SLOT_DS();
                    DAB_SLOT_VMEM(); DAB_SLOT_NONE(); DAB_SLOT_VMEM(); DAB_SLOT_NONE();
                }
            }
        }

        // ---- epilogue.  Register v of a 32x32 block is row (v/4)*8 + (lane/32)*4 + v%4,
        // column lane%32, so the 32 lanes of a half-wavefront touch 128 contiguous bytes of one
        // output row.  Direct mode: y = (alpha - beta)*s1 + beta*sA; interior tiles store
        // without any predicate, so nothing orders one store behind another.  Split mode: the
        // exact partial s1 goes to this split's slice of the workspace.
        const bool interior = m_base + 64 <= g.M && f0 + kNTile <= g.F;
        float4 s4[2][4];
        if (MODE != kOutSplit) sA_lds[wave][lane] = rowsum;
        // (the wavefront reads back only what it wrote itself: no workgroup barrier needed)
        if (MODE != kOutSplit) {
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    s4[i][q] = *reinterpret_cast<const float4*>(&sA_lds[wave][i * 32 + q * 8 + (lane >> 5) * 4]);
        }
        if (MODE == kOutBits) {
            // Re-binarized output: bit = [y >= tau_f] with y evaluated exactly as in the fp32 output.
            // The ballot of one accumulator register is the 32-filter word of two rows (lanes 0..31 and
            // 32..63); lane l collects the four words of row l and stores them side by side.
            int wb[4] = {0, 0, 0, 0};
#pragma unroll
            for (int i = 0; i < 2; ++i) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float sv[4] = {s4[i][q].x, s4[i][q].y, s4[i][q].z, s4[i][q].w};
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        const int r0 = i * 32 + q * 8 + t;             // row of lanes 0..31; lanes 32..63 hold r0 + 4
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            const float y = fmaf(dcol[j], acc[i][j][q * 4 + t], bcol[j] * sv[t]);
                            const bool bit = f0 + j * 32 + (lane & 31) < g.F && y >= tcol[j];
                            const unsigned long long mask = __ballot(bit);
                            // the two halves of the (wavefront-uniform) mask go to lanes r0 and r0 + 4
                            // The mask is written by a vector compare.  On this ISA a vector instruction that reads a scalar
                            // register needs two wait states behind the vector instruction that wrote it; the compiler
                            // inserts them for its own instructions but does not look into inline assembly (without them the
                            // lane write took the register's previous content, the compare before the F mask: bits past F set).
                            asm volatile("s_nop 1\n\tv_writelane_b32 %0, %1, %2"
                                         : "+v"(wb[j]) : "s"(static_cast<uint32_t>(mask)), "n"(r0));
                            asm volatile("v_writelane_b32 %0, %1, %2"
                                         : "+v"(wb[j]) : "s"(static_cast<uint32_t>(mask >> 32)), "n"(r0 + 4));
                        }
                    }
                }
            }
            const int row = m_base + lane;
            const int Fw = (g.F + 31) >> 5;
            if (row < g.M) {
                uint32_t* dst = out_bits + static_cast<size_t>(row) * Fw + ntile * 4;
                if ((Fw & 3) == 0) {
                    *reinterpret_cast<int4*>(dst) = make_int4(wb[0], wb[1], wb[2], wb[3]);
                } else {
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        if (ntile * 4 + j < Fw) dst[j] = static_cast<uint32_t>(wb[j]);
                }
            }
            continue;
        }
        float* out = MODE == kOutSplit ? ws_s1 + static_cast<size_t>(ksplit_id) * g.M * g.F : Y;
        if (interior) {
            // no predicate anywhere: nothing orders one store behind another
#pragma unroll
            for (int i = 0; i < 2; ++i) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float sv[4] = {s4[i][q].x, s4[i][q].y, s4[i][q].z, s4[i][q].w};
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        const int row = m_base + i * 32 + q * 8 + (lane >> 5) * 4 + t;
                        const size_t o = static_cast<size_t>(row) * g.F + f0 + (lane & 31);
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            const float s1 = acc[i][j][q * 4 + t];
                            // written once and not read again by this kernel: streaming stores
                            __builtin_nontemporal_store(MODE == kOutSplit ? s1 : fmaf(dcol[j], s1, bcol[j] * sv[t]),
                                                        out + o + j * 32);
                            if (MODE == kOutYDebug) dbg_s1[o + j * 32] = static_cast<int>(s1);
                        }
                    }
                }
            }
        } else {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float sv[4] = {s4[i][q].x, s4[i][q].y, s4[i][q].z, s4[i][q].w};
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        const int row = m_base + i * 32 + q * 8 + (lane >> 5) * 4 + t;
                        const size_t o = static_cast<size_t>(row) * g.F + f0 + (lane & 31);
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            const float s1 = acc[i][j][q * 4 + t];
                            if (row < g.M && f0 + j * 32 + (lane & 31) < g.F) {
                                out[o + j * 32] = MODE == kOutSplit ? s1 : fmaf(dcol[j], s1, bcol[j] * sv[t]);
                                if (MODE == kOutYDebug) dbg_s1[o + j * 32] = static_cast<int>(s1);
                            }
                        }
                    }
                }
            }
        }
    }
}

// ---------------------------------------------------------------- small products
// Layers with a few hundred 32x32 output blocks at most (conv6 and fc7 of the Sketch-A-Net trunk,
// the late stages of a ResNet at small batch) are latency problems: the persistent kernel above
// would run on a handful of compute units or need a split reduction with partial sums in memory.
// Here one workgroup owns one 32-pixel x 32-filter block; its WAVES wavefronts take consecutive
// shares of the reduction, each reading both fragments straight from global memory (L2) through
// two eight-step register sets, and add their integer partial sums (exact in fp32) through LDS.
// sA comes from the prepare kernel's per-pixel pass.
constexpr int kSmallDepth = 8;

template <int MODE, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void binconv_small_kernel(
    const MfmaGeom g, const char* __restrict__ A4, const uint4* __restrict__ E4, const float* __restrict__ alpha,
    const float* __restrict__ beta, float* __restrict__ Y, int32_t* __restrict__ dbg_s1, const float* __restrict__ sA,
    const int32_t* __restrict__ ktab, const float* __restrict__ tau_out, uint32_t* __restrict__ out_bits) {
    __shared__ float red[WAVES][16][64];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int mb = fdiv(blockIdx.x, g.d_fblocks);
    const int fb = blockIdx.x - mb * g.n_fblocks;                   // neighbouring workgroups share the pixel rows
    const uint4* Eb = E4 + static_cast<size_t>(fb >> 2) * g.nk * 256 + (fb & 3) * 64 + lane;
    const __amdgpu_buffer_rsrc_t a4rsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(A4), 0, 2 * g.KB * g.plane, 0x00020000);
    int pixoff;
    {
        const int m = min(mb * 32 + (lane & 31), g.M - 1);
        const int b = fdiv(m, g.d_HoWo);
        const int r = m - b * g.HoWo;
        const int oy = fdiv(r, g.d_Wo);
        const int ox = r - oy * g.Wo;
        pixoff = ((b * g.Hp + oy * g.sh) * g.Wp + ox * g.sw) * 16 + (lane >> 5) * g.plane;
    }
    // column constants of this thread's outputs (every element it finishes has column lane % 32)
    const int f = min(fb * 32 + (lane & 31), g.F - 1);
    const float al = alpha[f], be = beta[f];
    const float tcol = (MODE == kOutBits && tau_out) ? tau_out[f] : 0.0f;

    auto load_a = [&](int poff) -> v4i {
        const auto v = __builtin_amdgcn_raw_buffer_load_b128(a4rsrc, pixoff, poff, 0);
        return v4i{static_cast<int>(v[0]), static_cast<int>(v[1]), static_cast<int>(v[2]), static_cast<int>(v[3])};
    };
    v16f acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.0f;
    // This wavefront's steps [k0, k1), taken in groups of kSmallDepth with two register sets: the
    // loads of the next group are issued back to back before the products of the current one.
    // Consecutive steps are neighbouring taps, i.e. neighbouring 16-byte pieces of the same cache
    // lines, so a burst finds the lines its first load brought in (issued one per step instead,
    // the eight wavefronts evict each other's lines and nearly every load goes to L2).  Fetches
    // past k1 repeat its last step.
    const int per = (g.nk + WAVES - 1) / WAVES;
    const int k0 = min(wave * per, g.nk), k1 = min(k0 + per, g.nk);
    const int klast = max(k1 - 1, 0);
    v4i aq[2][kSmallDepth];
    uint4 bq[2][kSmallDepth];
    auto fetch = [&](int set, int first) {
#pragma unroll
        for (int d = 0; d < kSmallDepth; ++d) aq[set][d] = load_a(ktab[min(first + d, klast)]);
#pragma unroll
        for (int d = 0; d < kSmallDepth; ++d) bq[set][d] = Eb[static_cast<size_t>(min(first + d, klast)) * 256];
    };
    auto multiply = [&](int set, int first) {
#pragma unroll
        for (int d = 0; d < kSmallDepth; ++d) {
            if (first + d < k1) {
                const uint4 bu = bq[set][d];
                const v4i bv = {static_cast<int>(bu.x), static_cast<int>(bu.y), static_cast<int>(bu.z),
                                static_cast<int>(bu.w)};
                acc = mfma_fp4(aq[set][d], bv, acc);
            }
        }
    };
    fetch(0, k0);
    for (int st = k0; st < k1; st += 2 * kSmallDepth) {
        fetch(1, st + kSmallDepth);
        multiply(0, st);
        fetch(0, st + 2 * kSmallDepth);
        multiply(1, st + kSmallDepth);
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) red[wave][v][lane] = acc[v];
    __syncthreads();

    // register v of lane l is row (v/4)*8 + (l/32)*4 + v%4 of the block, column l%32; wavefront w
    // finishes registers w, w + WAVES, ...
    const bool fvalid = fb * 32 + (lane & 31) < g.F;
    const float dcol = al - be;
    const int Fw = (g.F + 31) >> 5;
#pragma unroll
    for (int v = wave; v < 16; v += WAVES) {
        const int rl = (v >> 2) * 8 + (lane >> 5) * 4 + (v & 3);
        const int row = mb * 32 + rl;
        const float sv = sA[min(row, g.M - 1)];
        float s1 = 0.0f;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) s1 += red[w][v][lane];
        const float y = fmaf(dcol, s1, be * sv);
        if (MODE == kOutBits) {
            const unsigned long long mask = __ballot(fvalid && y >= tcol);
            const uint32_t word = static_cast<uint32_t>(lane < 32 ? mask : mask >> 32);
            if ((lane & 31) == 0 && row < g.M) out_bits[static_cast<size_t>(row) * Fw + fb] = word;
        } else if (row < g.M && fvalid) {
            const size_t o = static_cast<size_t>(row) * g.F + fb * 32 + (lane & 31);
            Y[o] = y;
            if (MODE == kOutYDebug) dbg_s1[o] = static_cast<int>(s1);
        }
    }
}

// ---------------------------------------------------------------- finish (split launches)
__global__ __launch_bounds__(256) void binconv_finish_kernel(const float* __restrict__ ws_s1,
                                                             const float* __restrict__ ws_sA,
                                                             const float* __restrict__ alpha,
                                                             const float* __restrict__ beta, float* __restrict__ Y,
                                                             int32_t* __restrict__ dbg_s1, int M, int F, int ksplit) {
    const size_t i = static_cast<size_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    const size_t total = static_cast<size_t>(M) * F;
    if (i >= total) return;
    const int m = static_cast<int>(i / F);
    const int f = static_cast<int>(i - static_cast<size_t>(m) * F);
    float s1 = 0.f;                                 // integer-valued, exact in any order
    int k = 0;
    for (; k + 8 <= ksplit; k += 8) {               // eight partials in flight
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = ws_s1[static_cast<size_t>(k + u) * total + i];
#pragma unroll
        for (int u = 0; u < 8; ++u) s1 += v[u];
    }
    for (; k < ksplit; ++k) s1 += ws_s1[static_cast<size_t>(k) * total + i];
    const float sA = ws_sA[m];
    const float al = alpha[f], be = beta[f];
    Y[i] = fmaf(al - be, s1, be * sA);
    if (dbg_s1) dbg_s1[i] = static_cast<int>(s1);
}

// Split launches with re-binarized output: one wavefront per (pixel, 64 filters); the ballot of the
// compare is the two packed words.
__global__ __launch_bounds__(256) void binconv_finish_bits_kernel(const float* __restrict__ ws_s1,
                                                                  const float* __restrict__ ws_sA,
                                                                  const float* __restrict__ alpha,
                                                                  const float* __restrict__ beta,
                                                                  const float* __restrict__ tau_out,
                                                                  uint32_t* __restrict__ out_bits, int M, int F,
                                                                  int ksplit) {
    const int lane = threadIdx.x & 63;
    const int F64 = (F + 63) >> 6, Fw = (F + 31) >> 5;
    const long long item = 1ll * blockIdx.x * 4 + (threadIdx.x >> 6);
    if (item >= 1ll * M * F64) return;
    const int m = static_cast<int>(item / F64);
    const int f = static_cast<int>(item - 1ll * m * F64) * 64 + lane;
    const size_t total = static_cast<size_t>(M) * F;
    bool bit = false;
    if (f < F) {
        float s1 = 0.f;
        const float* p = ws_s1 + static_cast<size_t>(m) * F + f;
        int k = 0;
        for (; k + 8 <= ksplit; k += 8) {           // eight partials in flight
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = p[static_cast<size_t>(k + u) * total];
#pragma unroll
            for (int u = 0; u < 8; ++u) s1 += v[u];
        }
        for (; k < ksplit; ++k) s1 += p[static_cast<size_t>(k) * total];
        const float al = alpha[f], be = beta[f];
        bit = fmaf(al - be, s1, be * ws_sA[m]) >= (tau_out ? tau_out[f] : 0.0f);
    }
    const unsigned long long mask = __ballot(bit);
    const int w = (f - lane) >> 5;
    if (lane == 0) out_bits[static_cast<size_t>(m) * Fw + w] = static_cast<uint32_t>(mask);
    if (lane == 32 && w + 1 < Fw) out_bits[static_cast<size_t>(m) * Fw + w + 1] = static_cast<uint32_t>(mask >> 32);
}

// ------------------------------------------------------------------ host side

struct MfmaPlan {
    MfmaGeom g;
    int waves;
    bool split, small;
    size_t a4_bytes, e4_bytes, sa_bytes, s1_bytes, ws_bytes, lds_bytes;
    unsigned grid;
};

static size_t round256(size_t x) { return (x + 255) & ~static_cast<size_t>(255); }

static int plan_binconv(const dab_conv_desc& d, MfmaPlan* pl) {
    MfmaGeom& g = pl->g;
    g = MfmaGeom{};
    g.B = d.B; g.H = d.H; g.W = d.W; g.F = d.F; g.kh = d.kh; g.kw = d.kw;
    g.ph = d.pad_h; g.pw = d.pad_w; g.sh = d.stride_h; g.sw = d.stride_w;
    g.C = d.C; g.Cw = ceil_div(d.C, 32);
    // k-blocks per tap: 64 channels of fp4
    g.KB = ceil_div(d.C, 64);
    g.Ho = (d.H + 2 * d.pad_h - d.kh) / d.stride_h + 1;
    g.Wo = (d.W + 2 * d.pad_w - d.kw) / d.stride_w + 1;
    g.HoWo = g.Ho * g.Wo;
    g.Hp = d.H + 2 * d.pad_h; g.Wp = d.W + 2 * d.pad_w;
    g.Fp = 64 * ceil_div(d.F, 64);
    const long long M = 1ll * d.B * g.HoWo;
    const long long a4 = 1ll * d.B * g.Hp * g.Wp * g.KB * 32;
    const long long nk = 1ll * d.kh * d.kw * g.KB;
    if (M >= (1ll << 30) || a4 >= (1ll << 31) || nk >= (1 << 20) || 1ll * M * d.F >= (1ll << 40)) return DAB_ERR_UNSUPPORTED;
    if (1ll * d.C * d.kh * d.kw >= (1ll << 24)) return DAB_ERR_UNSUPPORTED;   // |s1| must stay exact in fp32
    g.M = static_cast<int>(M);
    g.nk = static_cast<int>(nk);
    g.n_ntiles = ceil_div(d.F, kNTile);
    if (1ll * g.n_ntiles * g.nk >= (1ll << 22)) return DAB_ERR_UNSUPPORTED;

    // Workgroup shape and split.  Eight wavefronts (two per SIMD, 512 pixels per tile) overlap
    // one wavefront's stores with another's multiplies and win on large layers; four keep more
    // compute units busy on mid-sized ones.  When even 256-pixel tiles leave most compute
    // units idle, the reduction is split until about one unit per compute unit exists.
    const int tiles256 = ceil_div(g.M, 256) * g.n_ntiles;
    pl->waves = 1ll * ceil_div(g.M, 512) * g.n_ntiles >= kNumCU * 3 / 4 ? 8 : 4;
    g.ksplit = 1;
    if (tiles256 * 2 <= kNumCU) {
        g.ksplit = kNumCU / tiles256;
        const int max_split = g.nk / (2 * kPrefetch);              // at least two prefetch groups per split
        if (g.ksplit > max_split) g.ksplit = max_split;
        if (g.ksplit < 1) g.ksplit = 1;
    }
    g.split_steps = ceil_div(g.nk, g.ksplit);
    g.ksplit = ceil_div(g.nk, g.split_steps);
    pl->split = g.ksplit > 1;
    if (pl->split) pl->waves = 4;
    // A layer that would need the split and has at most 512 output blocks of 32 x 32 runs one
    // workgroup per block over the whole reduction instead (no partial sums in memory, no finish kernel).
    g.n_fblocks = ceil_div(d.F, 32);
    g.d_fblocks = make_fastdiv(g.n_fblocks);
    pl->small = tiles256 * 2 <= kNumCU && 1ll * ceil_div(g.M, 32) * g.n_fblocks <= 512;
    if (pl->small) {
        pl->split = false;
        g.ksplit = 1;
        g.split_steps = g.nk;
    }
    // chunks of the LDS panel
    const int span = pl->split ? g.split_steps : g.nk;
    const int nchunks = ceil_div(span, kMaxChunk);
    g.kchunk = ceil_div(ceil_div(span, nchunks), kPrefetch) * kPrefetch;
    g.n_mtiles = ceil_div(g.M, 64 * pl->waves);
    g.wg_per_ntile = kNumCU / g.n_ntiles;
    if (g.wg_per_ntile < 1) g.wg_per_ntile = 1;
    if (g.wg_per_ntile > g.n_mtiles) g.wg_per_ntile = g.n_mtiles;
    pl->grid = pl->split ? static_cast<unsigned>(g.n_ntiles * g.n_mtiles * g.ksplit)
                         : static_cast<unsigned>(g.wg_per_ntile * g.n_ntiles);

    g.T = d.kh * d.kw; g.npix = d.B * g.Hp * g.Wp; g.plane = g.npix * 16;
    g.d_HoWo = make_fastdiv(g.HoWo); g.d_Wo = make_fastdiv(g.Wo);
    g.d_Wp = make_fastdiv(g.Wp); g.d_HpWp = make_fastdiv(g.Hp * g.Wp);
    g.d_T = make_fastdiv(g.T); g.d_kw = make_fastdiv(g.kw); g.d_Cw = make_fastdiv(g.Cw);
    g.d_nk = make_fastdiv(g.nk); g.d_mtiles = make_fastdiv(g.n_mtiles); g.d_ksplit = make_fastdiv(g.ksplit);

    pl->a4_bytes = round256(static_cast<size_t>(a4));
    pl->e4_bytes = static_cast<size_t>(g.n_ntiles) * g.nk * 4096;
    pl->sa_bytes = round256(static_cast<size_t>(g.M) * 4) + round256(static_cast<size_t>(g.npix) * 4) +
                   round256(static_cast<size_t>(g.nk + kTabPad + g.T) * 4);
    pl->s1_bytes = pl->split ? round256(static_cast<size_t>(g.ksplit) * g.M * d.F * 4) : 0;
    pl->ws_bytes = pl->a4_bytes + pl->e4_bytes + pl->sa_bytes + pl->s1_bytes;
    pl->lds_bytes = static_cast<size_t>(g.kchunk) * 4096;

    g.act_w = 2 * g.KB >= 8 ? 8 : 2 * g.KB;                      // 2, 4, 6 (-> 4 x 64 would not divide) ...
    while (256 % g.act_w) --g.act_w;
    g.act_p = 256 / g.act_w;
    g.act_wt = ceil_div(2 * g.KB, g.act_w);
    g.d_act_wt = make_fastdiv(g.act_wt);
    g.blk_act = static_cast<unsigned>(ceil_div(g.npix, g.act_p)) * g.act_wt;
    g.sum_shift = 0;
    while (g.sum_shift < 6 && (4 << g.sum_shift) < g.Cw) ++g.sum_shift;       // about four words per lane
    g.blk_wgt = static_cast<unsigned>((1ll * g.n_ntiles * g.nk * 256 + 255) / 256);
    g.blk_sum = static_cast<unsigned>((1ll * g.npix * (1 << g.sum_shift) + 255) / 256);
    g.blk_tab = static_cast<unsigned>((g.nk + kTabPad + 255) / 256);
    g.blk_sa = (pl->split || pl->small) ? static_cast<unsigned>((g.M + 3) / 4) : 0u;
    return DAB_OK;
}

template <int WAVES, int MODE>
static int launch_main(const MfmaPlan& pl, hipStream_t st, const char* a4, const uint4* e4, float* sa,
                       const float* alpha, const float* beta, float* Y, int32_t* dbg_s1, float* ws_s1,
                       const int32_t* pixsum, const int32_t* ktab, const float* tau_out, uint32_t* out_bits) {
    return launch(binconv_mfma_kernel<WAVES, MODE>, dim3(pl.grid), dim3(64 * WAVES), pl.lds_bytes, st, pl.g, a4, e4,
                  alpha, beta, Y, dbg_s1, ws_s1, sa, pixsum, ktab, tau_out, out_bits);
}

// One-time set-up on the current device: the panel of the main kernel takes up to kMaxChunk * 4 KB
// of dynamic LDS, above the default limit of a launch.
template <int WAVES, int MODE>
static int raise_lds_limit() {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&binconv_mfma_kernel<WAVES, MODE>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, kMaxChunk * 4096);
    return e == hipSuccess ? static_cast<int>(DAB_OK) : hip_failed(e);
}
int init_binconv() {
    if (int rc = raise_lds_limit<8, kOutY>()) return rc;
    if (int rc = raise_lds_limit<8, kOutYDebug>()) return rc;
    if (int rc = raise_lds_limit<8, kOutBits>()) return rc;
    if (int rc = raise_lds_limit<4, kOutY>()) return rc;
    if (int rc = raise_lds_limit<4, kOutYDebug>()) return rc;
    if (int rc = raise_lds_limit<4, kOutBits>()) return rc;
    return raise_lds_limit<4, kOutSplit>();
}

// Estimated time of the launches that go through the workspace: operands written (a4, e4) at 2.9 TB/s, then per tile of a
// workgroup the k-steps of eight or four wavefronts, the output beside the multiplies of others at 14.2 TB/s, or at 6.4
// where the stores are of single values; with the reduction split, the partial sums twice through memory.  (Fitted to
// the layers that plan_product names; rms error 7 %.)
static double expanded_us(const MfmaPlan& pl, bool bits) {
    const MfmaGeom& g = pl.g;
    const double out = 1.0 * g.M * g.F;
    const long long units = 1ll * g.n_ntiles * g.n_mtiles * g.ksplit;
    const long long tiles = pl.split ? (units + kNumCU - 1) / kNumCU
                                     : 1ll * ceil_div(g.n_mtiles, g.wg_per_ntile) * ceil_div(g.n_ntiles, kNumCU);
    double us = 9.9 + static_cast<double>(pl.a4_bytes + pl.e4_bytes) / 2.9e6 +
                static_cast<double>(tiles) * (ceil_div(g.nk, g.ksplit) * (pl.waves == 8 ? 0.31 : 0.207) + 5.3);
    if (!bits) us += 4.0 * out / (g.F % 4 ? 6.4e6 : 14.2e6);
    if (pl.split) us += 3.2 + 8.0 * g.ksplit * out / 5.5e6;
    return us;
}

// Estimated times (us) of the kernels that read bits, for reductions of at most 36 k-steps.  Fitted to random layers of more
// than 256 blocks, both outputs, every kernel timed on each (persistent and blocks 573 layers, rms error 12 and 9 %; split 2100
// layers, 9 %).
static double short_out(const DirectGeom& g, bool bits, double whole, double part) {
    return bits ? 0.0 : 4.0e-6 * g.M * g.F * (g.F % 4 ? part : whole);    // rows of whole 16-byte stores, other rows
}
static double short_direct_us(const DirectPlan& pl, bool bits) {
    const DirectGeom& g = pl.g;
    const int n_ntiles = ceil_div(g.F, kNTile), tiles = ceil_div(g.n_mtiles, g.wg_per_ntile) * ceil_div(n_ntiles, kNumCU);
    const double step = (pl.waves == 4 ? 0.114 : 0.151) * (pl.pad ? 1.485 : 1.0) * (pl.lw == 1 ? 1.477 : pl.lw == 2 ? 1.062 : 1.0);
    return 3.64 + 0.0385 * g.n_ent + tiles * ((g.n_ent - 1) * step + (pl.waves == 4 ? 2.08 : 3.72)) + short_out(g, bits, 0.033, 0.12);
}
static double short_block_us(const BlockPlan& pl, bool bits) {
    const DirectGeom& g = pl.g;
    const double per_cu = static_cast<double>(pl.grid) / kNumCU;
    const double step = pl.lw == 4 ? (g.T > 1 ? 0.0099 : 0.0061) : (g.T > 1 ? 0.0186 : 0.0239);
    const int share = ceil_div(g.nk, pl.waves * pl.lw) * pl.lw, steps = ceil_div(share, pl.depth) * pl.depth;
    return 4.04 + (per_cu + 0.435) * ((pl.pad ? 0.243 : 0.182) + pl.waves * steps * step) + short_out(g, bits, 0.095, 0.141);
}
static double short_split_us(const SplitPlan& pl, bool bits) {
    const DirectGeom& g = pl.g;
    const double step = (pl.lw == 1 ? 0.381 : pl.lw == 2 ? 0.276 : 0.165) + (pl.pad ? 0.108 : 0.0) + 0.074 / g.T + 0.231 * pl.filled;
    return 4.86 + pl.rounds * (pl.sg.log_ks ? -0.06 : 1.43) + pl.rounds * pl.steps_run * step + short_out(g, bits, 0.064, 0.121);
}

// Which kernel computes a layer, with its plan.
struct ProductPlans {
    BlockPlan block;
    DirectPlan direct;
    SplitPlan split;
    MfmaPlan expanded;
    bool needs_ws;          // the caller has to bring the workspace of `expanded`, whichever kernel is taken
};
static int plan_product(const dab_conv_desc& d, bool bits, ProductPlans* p, Product* which) {
    p->needs_ws = false;
    // layers of a few hundred output blocks: one workgroup per block, straight from the bits, no workspace
    *which = Product::kBlock;
    if (plan_block(d, &p->block, false)) return DAB_OK;
    // A reduction whose B fragments fit in LDS: the persistent kernel, which builds them once per workgroup.  With too few
    // tiles for the compute units, a workgroup per 32 x 32 block or the split kernel are faster: taken where their estimates
    // are under 0.95 and 0.85 of the persistent one's, the split kernel's also under 0.9 of the blocks' (from
    // eight k-steps and up to two rounds of workgroups, as far as it was timed).  Over 2137 random layers the form taken
    // is 0.7 % slower than the fastest in the geometric mean.  (us, persistent | blocks | split, fp32:) 7290 pixels x 18
    // steps x 519 filters 10.7 | 16.6 | 12.4, 52200 x 20 x 88 11.6 | 21.1 | 14.3; 864 x 25 x 382 12.6 | 4.9 | 7.3, 16473 x 12 x 19
    // 7.8 | 4.0 | 7.3; 3648 x 25 x 487 14.0 | 11.0 | 8.6, 12544 x 36 x 115 13.0 | 9.9 | 7.7.
    if ((bits || d.F <= kDirMaxFilters) && plan_direct(d, &p->direct)) {
        *which = Product::kDirect;
        const double direct = short_direct_us(p->direct, bits);
        double best = direct;
        if (plan_block(d, &p->block, true) && short_block_us(p->block, bits) < 0.95 * direct) {
            best = short_block_us(p->block, bits);
            *which = Product::kBlock;
        }
        if (p->direct.g.nk >= 8 && plan_split(d, &p->split) && p->split.sg.units <= 2 * kNumCU) {
            const double split = short_split_us(p->split, bits);
            if (split < (*which == Product::kBlock ? 0.9 * best : 0.85 * direct) && split < 0.85 * direct) *which = Product::kSplit;
        }
        return DAB_OK;
    }
    // Longer reductions: shares of it per wavefront over blocks of 64 x 128 where that is the faster form.  Otherwise a
    // workgroup per 32 x 32 block up to a few thousand blocks, and past those the operands expanded into the workspace:
    // a multiply has less work beside it there (nothing is expanded again for each filter tile and tap), which pays for
    // the launch and the bytes more on large layers.  Chosen by estimated times, which are within 9 % (blocks), 7 %
    // (split) and 7 % rms (workspace) of the measured ones over random layers of 37 to 1100 k-steps, both outputs;
    // over 1900 others the form taken is 0.5 % slower than the fastest one in the geometric mean.  (Split where its estimate
    // is 5 % below the blocks', up to 3 % above the workspace's: of the factors 0.9 to 1.1 these made the best choices.)
    // (us, split | blocks | workspace, fp32 output:) 5819 pixels x 66 steps x 542 filters 15.2 |
    // 39.3 | 42.4, 19044 x 50 x 290 19.7 | 35.9 | 25.8; 5408 x 50 x 40 9.5 | 6.0 | -, 624 x 60 x 446 9.3 | 5.8 | 13.4;
    // 58190 x 117 x 144 71.9 | - | 57.7, 98315 x 325 x 35 152 | - | 120.
    // (The workspace is asked for, as dab_binconv2d_workspace_bytes says, whichever of split and workspace is taken.)
    const bool few_blocks = plan_block(d, &p->block, true);
    if (!few_blocks) {
        if (int rc = plan_binconv(d, &p->expanded)) return rc;
        p->needs_ws = true;
    }
    const bool splits = plan_split(d, &p->split);
    const double other_us = few_blocks ? p->block.us : expanded_us(p->expanded, bits);
    if (splits && (bits ? p->split.us_bits : p->split.us) < (few_blocks ? 0.95 : 1.03) * other_us) *which = Product::kSplit;
    else *which = few_blocks ? Product::kBlock : Product::kExpanded;
    return DAB_OK;
}
int product_of(const dab_conv_desc& d, bool bits, Product* which) {
    ProductPlans p;
    return plan_product(d, bits, &p, which);
}

// Y != nullptr: fp32 output (and optional dbg_s1); Y == nullptr: re-binarized output into out_bits.
static int run_binconv(const dab_conv_desc& d, const uint32_t* A, const uint32_t* E, const float* alpha,
                       const float* beta, float* Y, int32_t* dbg_s1, const float* tau_out, uint32_t* out_bits,
                       void* ws, size_t ws_bytes, hipStream_t st) {
    ProductPlans p;
    Product which;
    if (int rc = plan_product(d, Y == nullptr, &p, &which)) return rc;
    const MfmaPlan& pl = p.expanded;
    if (p.needs_ws && (!ws || ws_bytes < pl.ws_bytes || misaligned(ws, 256))) return DAB_ERR_WORKSPACE;
    if (which == Product::kBlock) return launch_block(p.block, st, A, E, alpha, beta, Y, dbg_s1, tau_out, out_bits);
    if (int rc = ensure_device_ready()) return rc;
    if (which == Product::kDirect) return launch_direct(p.direct, st, A, E, alpha, beta, Y, dbg_s1, tau_out, out_bits);
    if (which == Product::kSplit) return launch_split(p.split, st, A, E, alpha, beta, Y, dbg_s1, tau_out, out_bits);
    char* a4 = static_cast<char*>(ws);
    uint4* e4 = reinterpret_cast<uint4*>(a4 + pl.a4_bytes);
    float* sa = reinterpret_cast<float*>(a4 + pl.a4_bytes + pl.e4_bytes);
    float* s1 = reinterpret_cast<float*>(a4 + pl.a4_bytes + pl.e4_bytes + pl.sa_bytes);
    const MfmaGeom& g = pl.g;

    int32_t* pixsum = reinterpret_cast<int32_t*>(reinterpret_cast<char*>(sa) + round256(static_cast<size_t>(g.M) * 4));
    int32_t* ktab = reinterpret_cast<int32_t*>(reinterpret_cast<char*>(pixsum) + round256(static_cast<size_t>(g.npix) * 4));
    if (int rc = launch(binconv_prepare_kernel, dim3(g.blk_act + g.blk_wgt + g.blk_sum + g.blk_tab + g.blk_sa), dim3(256), 0,
                        st, g, A, E, reinterpret_cast<uint4*>(a4), e4, pixsum, ktab, sa))
        return rc;

    if (pl.small) {
        const unsigned blocks = static_cast<unsigned>(ceil_div(g.M, 32) * g.n_fblocks);
        auto small = [&](auto kernel, int waves) {
            return launch(kernel, dim3(blocks), dim3(64 * waves), 0, st, g, a4, e4, alpha, beta, Y, dbg_s1, sa, ktab, tau_out,
                          out_bits);
        };
        // enough wavefronts per block that each keeps a few steps of the reduction
        if (g.nk >= 32) {
            if (!Y) return small(binconv_small_kernel<kOutBits, 8>, 8);
            if (dbg_s1) return small(binconv_small_kernel<kOutYDebug, 8>, 8);
            return small(binconv_small_kernel<kOutY, 8>, 8);
        }
        if (!Y) return small(binconv_small_kernel<kOutBits, 2>, 2);
        if (dbg_s1) return small(binconv_small_kernel<kOutYDebug, 2>, 2);
        return small(binconv_small_kernel<kOutY, 2>, 2);
    }
    if (pl.split) {
        if (int rc = launch_main<4, kOutSplit>(pl, st, a4, e4, sa, alpha, beta, Y, dbg_s1, s1, pixsum, ktab, tau_out, out_bits)) return rc;
        const size_t total = static_cast<size_t>(g.M) * d.F;
        if (!Y) {
            const long long items = 1ll * g.M * ceil_div(d.F, 64);
            return launch(binconv_finish_bits_kernel, dim3(static_cast<unsigned>((items + 3) / 4)), dim3(256), 0, st, s1, sa,
                          alpha, beta, tau_out, out_bits, g.M, d.F, g.ksplit);
        }
        return launch(binconv_finish_kernel, dim3(static_cast<unsigned>((total + 255) / 256)), dim3(256), 0, st, s1, sa, alpha,
                      beta, Y, dbg_s1, g.M, d.F, g.ksplit);
    }
    if (!Y)
        return pl.waves == 8 ? launch_main<8, kOutBits>(pl, st, a4, e4, sa, alpha, beta, Y, dbg_s1, s1, pixsum, ktab, tau_out, out_bits)
                             : launch_main<4, kOutBits>(pl, st, a4, e4, sa, alpha, beta, Y, dbg_s1, s1, pixsum, ktab, tau_out, out_bits);
    if (pl.waves == 8)
        return dbg_s1 ? launch_main<8, kOutYDebug>(pl, st, a4, e4, sa, alpha, beta, Y, dbg_s1, s1, pixsum, ktab, tau_out, out_bits)
                      : launch_main<8, kOutY>(pl, st, a4, e4, sa, alpha, beta, Y, dbg_s1, s1, pixsum, ktab, tau_out, out_bits);
    return dbg_s1 ? launch_main<4, kOutYDebug>(pl, st, a4, e4, sa, alpha, beta, Y, dbg_s1, s1, pixsum, ktab, tau_out, out_bits)
                  : launch_main<4, kOutY>(pl, st, a4, e4, sa, alpha, beta, Y, dbg_s1, s1, pixsum, ktab, tau_out, out_bits);
}

// The weights-only layer (wbin.hip).
static int run_wbin(const dab_conv_desc& d, const float* X, const uint32_t* E, const float* alpha, const float* beta,
                    float* Y, void* ws, size_t ws_bytes, hipStream_t st) {
    size_t need = 0;
    if (int rc = wbin_workspace(d, &need)) return rc;
    if (!ws || ws_bytes < need || misaligned(ws, 256)) return DAB_ERR_WORKSPACE;
    if (int rc = ensure_device_ready()) return rc;
    WbinPlan pl;
    plan_wbin(d, &pl);
    return launch_wbin(pl, st, X, E, alpha, beta, Y);
}

static int check_common(const void* A, const void* E, const void* alpha, const void* beta, const void* Y,
                        const void* dbg) {
    if (!A || !E || !alpha || !beta || !Y) return DAB_ERR_NULL;
    if (misaligned(A, 16) || misaligned(E, 64) || misaligned(Y, 16) || misaligned(alpha, 4) ||
        misaligned(beta, 4) || (dbg && misaligned(dbg, 16)))
        return DAB_ERR_ALIGN;
    return DAB_OK;
}

static int check_desc(const dab_conv_desc* d) {
    if (d->B < 1 || d->C < 1 || d->H < 1 || d->W < 1 || d->F < 1 || d->kh < 1 || d->kw < 1 ||
        d->pad_h < 0 || d->pad_w < 0 || d->stride_h < 1 || d->stride_w < 1)
        return DAB_ERR_SHAPE;
    if (d->H + 2 * d->pad_h < d->kh || d->W + 2 * d->pad_w < d->kw) return DAB_ERR_SHAPE;
    if (1ll * d->C * d->kh * d->kw < 2) return DAB_ERR_SHAPE;
    // (pad >= kernel extent: windows entirely in the border are allowed; they give s1 = sA = 0)
    return DAB_OK;
}

}  // namespace dab

extern "C" {

size_t dab_binconv2d_workspace_bytes(const dab_conv_desc* d) {
    dab::MfmaPlan pl;
    dab::DirectPlan dp;
    if (!d || dab::check_desc(d) != DAB_OK) return 0;
    dab::BlockPlan bp;
    if (dab::plan_block(*d, &bp, false) || (d->F <= dab::kDirMaxFilters && dab::plan_direct(*d, &dp)) || dab::plan_block(*d, &bp, true)) return 0;
    if (dab::plan_binconv(*d, &pl) != DAB_OK) return 0;
    return pl.ws_bytes;
}

size_t dab_binfc_workspace_bytes(int32_t B, int32_t Kin, int32_t F) {
    if (B < 1 || Kin < 2 || F < 1) return 0;
    const dab_conv_desc d{B, Kin, 1, 1, F, 1, 1, 0, 0, 1, 1};
    return dab_binconv2d_workspace_bytes(&d);
}

int dab_binconv2d(const dab_conv_desc* d, const uint32_t* A_packed, const uint32_t* E_packed,
                  const float* alpha, const float* beta, float* Y, int32_t* dbg_s1,
                  void* ws, size_t ws_bytes, void* stream) {
    if (!d) return DAB_ERR_NULL;
    if (int rc = dab::check_common(A_packed, E_packed, alpha, beta, Y, dbg_s1)) return rc;
    if (int rc = dab::check_desc(d)) return rc;
    return dab::run_binconv(*d, A_packed, E_packed, alpha, beta, Y, dbg_s1, nullptr, nullptr, ws, ws_bytes,
                            static_cast<hipStream_t>(stream));
}

int dab_binfc(int32_t B, int32_t Kin, int32_t F, const uint32_t* A_packed, const uint32_t* E_packed,
              const float* alpha, const float* beta, float* Y, int32_t* dbg_s1,
              void* ws, size_t ws_bytes, void* stream) {
    if (int rc = dab::check_common(A_packed, E_packed, alpha, beta, Y, dbg_s1)) return rc;
    if (B < 1 || Kin < 2 || F < 1) return DAB_ERR_SHAPE;
    const dab_conv_desc d{B, Kin, 1, 1, F, 1, 1, 0, 0, 1, 1};
    return dab::run_binconv(d, A_packed, E_packed, alpha, beta, Y, dbg_s1, nullptr, nullptr, ws, ws_bytes,
                            static_cast<hipStream_t>(stream));
}

size_t dab_wbin_conv2d_workspace_bytes(const dab_conv_desc* d) {
    size_t need = 0;
    return d && dab::check_desc(d) == DAB_OK && dab::wbin_workspace(*d, &need) == DAB_OK ? need : 0;
}

size_t dab_wbin_fc_workspace_bytes(int32_t B, int32_t Kin, int32_t F) {
    if (B < 1 || Kin < 2 || F < 1) return 0;
    const dab_conv_desc d{B, Kin, 1, 1, F, 1, 1, 0, 0, 1, 1};
    return dab_wbin_conv2d_workspace_bytes(&d);
}

int dab_wbin_conv2d(const dab_conv_desc* d, const float* X, const uint32_t* E_packed, const float* alpha,
                    const float* beta, float* Y, void* ws, size_t ws_bytes, void* stream) {
    if (!d) return DAB_ERR_NULL;
    if (int rc = dab::check_common(X, E_packed, alpha, beta, Y, nullptr)) return rc;
    if (int rc = dab::check_desc(d)) return rc;
    return dab::run_wbin(*d, X, E_packed, alpha, beta, Y, ws, ws_bytes, static_cast<hipStream_t>(stream));
}

int dab_wbin_fc(int32_t B, int32_t Kin, int32_t F, const float* X, const uint32_t* E_packed, const float* alpha,
                const float* beta, float* Y, void* ws, size_t ws_bytes, void* stream) {
    if (int rc = dab::check_common(X, E_packed, alpha, beta, Y, nullptr)) return rc;
    if (B < 1 || Kin < 2 || F < 1) return DAB_ERR_SHAPE;
    const dab_conv_desc d{B, Kin, 1, 1, F, 1, 1, 0, 0, 1, 1};
    return dab::run_wbin(d, X, E_packed, alpha, beta, Y, ws, ws_bytes, static_cast<hipStream_t>(stream));
}

int dab_binconv2d_bits(const dab_conv_desc* d, const uint32_t* A_packed, const uint32_t* E_packed,
                       const float* alpha, const float* beta, const float* tau_out, uint32_t* A_next,
                       void* ws, size_t ws_bytes, void* stream) {
    if (!d) return DAB_ERR_NULL;
    if (!A_packed || !E_packed || !alpha || !beta || !A_next) return DAB_ERR_NULL;
    if (dab::misaligned(A_packed, 16) || dab::misaligned(E_packed, 64) || dab::misaligned(A_next, 16) ||
        dab::misaligned(alpha, 4) || dab::misaligned(beta, 4) || (tau_out && dab::misaligned(tau_out, 4)))
        return DAB_ERR_ALIGN;
    if (int rc = dab::check_desc(d)) return rc;
    return dab::run_binconv(*d, A_packed, E_packed, alpha, beta, nullptr, nullptr, tau_out, A_next, ws, ws_bytes,
                            static_cast<hipStream_t>(stream));
}

int dab_binfc_bits(int32_t B, int32_t Kin, int32_t F, const uint32_t* A_packed, const uint32_t* E_packed,
                   const float* alpha, const float* beta, const float* tau_out, uint32_t* A_next,
                   void* ws, size_t ws_bytes, void* stream) {
    if (!A_packed || !E_packed || !alpha || !beta || !A_next) return DAB_ERR_NULL;
    if (dab::misaligned(A_packed, 16) || dab::misaligned(E_packed, 64) || dab::misaligned(A_next, 16) ||
        dab::misaligned(alpha, 4) || dab::misaligned(beta, 4) || (tau_out && dab::misaligned(tau_out, 4)))
        return DAB_ERR_ALIGN;
    if (B < 1 || Kin < 2 || F < 1) return DAB_ERR_SHAPE;
    const dab_conv_desc d{B, Kin, 1, 1, F, 1, 1, 0, 0, 1, 1};
    return dab::run_binconv(d, A_packed, E_packed, alpha, beta, nullptr, nullptr, tau_out, A_next, ws, ws_bytes,
                            static_cast<hipStream_t>(stream));
}

}  // extern "C"
