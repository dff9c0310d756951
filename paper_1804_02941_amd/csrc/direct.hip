// Binarized convolution / fully-connected product straight from the packed bits, one launch (gfx950).
//
// Section 4.3.2 of arXiv 1804.02941: the layer output is the ordinary convolution of the +1/-1
// input with the two-valued filter W~ = alpha*e + beta*(1-e) (Section 4.1), i.e.
//   y = alpha*s1 + beta*s2,  s1 = sum_i a_i e_i,  s1 + s2 = sA = sum_i a_i   (taps inside the image).
// s1 is a dense contraction and runs on the matrix cores on 4-bit floats (E2M1), which represent
// +1, -1 and 0 exactly; fp32 accumulation of at most 2^24 such products is exact.
//
// Both operands stay bits in memory and are expanded to fp4 on the way into the multiply:
//   weights      a workgroup owns 128 filters.  It reads their bit words once (word-major rows of
//                E, 128 bytes per row and wavefront half), expands them (mask bit 1 -> 1.0 = 0x2,
//                0 -> 0) and keeps the B fragments of the whole reduction in LDS;
//   activations  a lane owns one output pixel and one half of the channel words of a tap.  It
//                loads those words as they are packed (one, two or four per load, whole cache
//                lines per wavefront), expands each 32-bit word to the sixteen bytes of an A
//                fragment in seven vector instructions, and counts its ones for sA on the way.
//                Taps outside the image load nothing (buffer range check) and expand to zeros.
// The reduction is order-free, so a word's 32 channels may sit anywhere inside a k-step as long as
// both operands agree: bit 4i + d of a word goes to nibble i of dword d, which is a shift, a mask
// and an or per dword.  The sign bit of the fp4 code is the activation bit itself, so the
// accumulators hold -s1 (bit 1 = -1.0); the epilogue multiplies by (beta - alpha) instead.
//
// A wavefront computes 64 pixels x 128 filters per tile, workgroups are persistent and walk over pixel
// tiles; the loop over tiles has no barrier, the wavefronts of a workgroup drift apart and one's stores
// overlap another's multiplies.
#include "dab_internal.h"
#include "mfma_tools.h"

#include <type_traits>

namespace dab {

constexpr int kDirNTile = 128;              // filters per workgroup
constexpr int kDirGroupTable = 64;          // >= load groups of a tile (36) + two rounds of lookahead

// bit 4i + d of x -> sign bit of nibble i of dword d, magnitude 1.0: the A fragment of 32 channels.
// m8 / m2 are 0x88888888 / 0x22222222, or zero for a tap outside the image.
__device__ __forceinline__ v4i expand_a(uint32_t x, uint32_t m8, uint32_t m2) {
    v4i r;
    r.x = static_cast<int>(((x << 3) & m8) | m2);
    r.y = static_cast<int>(((x << 2) & m8) | m2);
    r.z = static_cast<int>(((x << 1) & m8) | m2);
    r.w = static_cast<int>((x & m8) | m2);
    return r;
}
// the same positions for the mask bits: 1 -> 1.0 (0x2), 0 -> 0
__device__ __forceinline__ uint4 expand_e(uint32_t x) {
    return make_uint4((x << 1) & 0x22222222u, x & 0x22222222u, (x >> 1) & 0x22222222u, (x >> 2) & 0x22222222u);
}

// The kernels that expand the mask words beside the multiplies are bound by that, so their codes leave out two of three
// shifts: mask bit 1 stands for 0.5, 1, 2 (0x1, 0x2, 0x4: the bit where it lies) and, shifted, 1 in the four dwords, and the
// activation's magnitude for 2, 1, 0.5 and 1, so that every product is 1 (exact, as before).  Five vector instructions a word
// instead of seven: 1024 x 9216 x 4096 21.4 -> 20.6 us, small batches of such layers up to 4 % (padded 3 x 3 layers unchanged).
__device__ __forceinline__ uint4 expand_e_in_place(uint32_t x) {
    return make_uint4(x & 0x11111111u, x & 0x22222222u, x & 0x44444444u, (x >> 2) & 0x22222222u);
}
// The masks of the expansion, or zeros for a tap outside the image: the sign bits, and magnitudes 2, 1 and 0.5.
struct SignMasks {
    uint32_t s, m2, m1, mh;
};
// In registers (as literals they would split the and-or in two).
__device__ __forceinline__ SignMasks sign_masks() {
    SignMasks m;
    asm volatile("s_mov_b32 %0, 0x88888888" : "=s"(m.s));
    asm volatile("v_mov_b32 %0, 0x44444444" : "=v"(m.m2));
    asm volatile("v_mov_b32 %0, 0x22222222" : "=v"(m.m1));
    asm volatile("v_mov_b32 %0, 0x11111111" : "=v"(m.mh));
    return m;
}
__device__ __forceinline__ SignMasks masks_where(bool in, const SignMasks& m) {
    return SignMasks{in ? m.s : 0u, in ? m.m2 : 0u, in ? m.m1 : 0u, in ? m.mh : 0u};
}
__device__ __forceinline__ v4i expand_a_in_place(uint32_t x, const SignMasks& m) {
    v4i r;
    r.x = static_cast<int>(((x << 3) & m.s) | m.m2);
    r.y = static_cast<int>(((x << 2) & m.s) | m.m1);
    r.z = static_cast<int>(((x << 1) & m.s) | m.mh);
    r.w = static_cast<int>((x & m.s) | m.m1);
    return r;
}

// Output stores as inline assembly.  Loads and stores share one counter (vmcnt) on this ISA and may
// complete out of order with respect to each other, so a compiler that sees both pending waits for
// the counter to reach zero before every use of a loaded activation word, once per round of the
// reduction loop: the prefetch distance is gone and the loop runs at memory latency.  With the
// stores out of its sight it counts the loads alone, which is safe wherever the stores lie: loads complete
// in order among themselves, so while the awaited load is pending, so are the n loads requested behind it,
// and more than n operations are outstanding.  Stores in flight only make a wait longer: the first loads of a
// tile are requested in front of the stores of the tile before, so its first wait is also one for all but a few
// of those stores.  Stores read their operands when they issue;
// a store of more than eight bytes is followed by a wait state before its data may be overwritten.
typedef int v4s __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));
// f(integral_constant<int, 0>) ... f(integral_constant<int, N - 1>): a loop whose index is a constant expression
template <int N, int J = 0, typename Fn>
__device__ __forceinline__ void for_each_column(Fn&& f) {
    if constexpr (J < N) {
        f(std::integral_constant<int, J>{});
        for_each_column<N, J + 1>(f);
    }
}
// Cache policy of the output stores (measured on MI355X; a policy changes only where the data waits
// on its way to memory).  Streaming ("nt") for outputs above 96 MB in whole lines of 128 bytes: they reach memory while the
// multiplies leave it idle, and leave the memory-side cache to the operands.  Smaller ones are read from that cache by what comes
// behind the layer, which streaming takes away.  (us, written through | streamed; the product alone over outputs in turn, over
// one output, with packing of the output behind it, with an in-place ReLU: 56 MB of 256 filters 21.4 | 22.5, 18.9 | 22.4,
// 29.4 | 32.0, 37.9 | 43.7; 80 MB of 64 25.8 | 25.3, 22.0 | 22.7, 35.8 | 37.1, 52.0 | 56.9; 128 MB of 64 38.7 | 36.0, 31.5 | 32.2,
// 51.0 | 52.9, 77.5 | 83.4; 160 MB of 128 48.3 | 44.0, 39.8 | 39.5, 63.7 | 66.4, 100.5 | 104.2.  The six layers of the Sketch-A-Net
// trunk at batch 256, outputs of 59 and 126 MB, with their weight sides, streamed above 48 MB | above 96 MB | never: outputs in
// turn 154.7 | 158.9 | 161.9, one set of them 153.8 | 147.9 | 159.2, each packed 209.4 | 203.9 | 202.9, behind a ReLU 284 | 266 | 261.)
// Device-scope write-through ("sc1") for the smaller ones, which the memory-side cache absorbs: their stores otherwise pile up
// behind the end of the kernel (12 to 16 % with the default policy at 15 to 60 MB).  Rows that are not whole
// lines leave both ends of a tile's row in parts: streamed, such outputs above 96 MB took 1.2 to 1.9 times as long as with
// the default policy, written through 0.9 to 1.2 times; where the stores are not even aligned to their 16 bytes, writing
// through takes up to 4 times as long, so those keep the default (1286 random layers).
template <int POLICY>
__device__ __forceinline__ void store_buffer_x4(v4f v, uint32_t voff, v4s rsrc, uint32_t soff) {
    if constexpr (POLICY == kStoreStream) {
        asm volatile("buffer_store_dwordx4 %0, %1, %2, %3 offen nt\n\ts_nop 1" : : "v"(v), "v"(voff), "s"(rsrc), "s"(soff) : "memory");
    } else if constexpr (POLICY == kStoreThrough) {
        asm volatile("buffer_store_dwordx4 %0, %1, %2, %3 offen sc1\n\ts_nop 1" : : "v"(v), "v"(voff), "s"(rsrc), "s"(soff) : "memory");
    } else {
        asm volatile("buffer_store_dwordx4 %0, %1, %2, %3 offen\n\ts_nop 1" : : "v"(v), "v"(voff), "s"(rsrc), "s"(soff) : "memory");
    }
}
__device__ __forceinline__ void store_buffer(float v, uint32_t voff, v4s rsrc, uint32_t soff) {
    asm volatile("buffer_store_dword %0, %1, %2, %3 offen" : : "v"(v), "v"(voff), "s"(rsrc), "s"(soff) : "memory");
}
__device__ __forceinline__ void store_u32(uint32_t* ptr, uint32_t v) {
    asm volatile("global_store_dword %0, %1, off" : : "v"(ptr), "v"(v) : "memory");
}
typedef uint32_t v2u __attribute__((ext_vector_type(2)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void store_u32x4(uint32_t* ptr, v4u v) {
    asm volatile("global_store_dwordx4 %0, %1, off\n\ts_nop 1" : : "v"(ptr), "v"(v) : "memory");
}

// Activation loads and the waits for them are inline assembly as well: the compiler orders
// independent loads as it likes and then waits for all of them, while the queue below relies on
// "the oldest group has landed once at most n younger loads are outstanding".  A load's result
// registers must not be touched before wait_words() has named them.
// The LW words of one load as one register tuple, so that nothing splits them before the wait.
template <int LW> struct WordsOf;
template <> struct WordsOf<1> { typedef uint32_t type; };
template <> struct WordsOf<2> { typedef v2u type; };
template <> struct WordsOf<4> { typedef v4u type; };
template <int LW>
__device__ __forceinline__ void load_words(typename WordsOf<LW>::type& dst, v4s rsrc, uint32_t voff) {
    if constexpr (LW == 1) {
        asm volatile("buffer_load_dword %0, %1, %2, 0 offen" : "=v"(dst) : "v"(voff), "s"(rsrc));
    } else if constexpr (LW == 2) {
        asm volatile("buffer_load_dwordx2 %0, %1, %2, 0 offen" : "=v"(dst) : "v"(voff), "s"(rsrc));
    } else {
        asm volatile("buffer_load_dwordx4 %0, %1, %2, 0 offen" : "=v"(dst) : "v"(voff), "s"(rsrc));
    }
}
// Waits until at most N vector-memory operations are outstanding; the words are operands so that
// every use of them stays behind the wait.
template <int N, typename T>
__device__ __forceinline__ void wait_words(T& a, T& b) {
    asm volatile("s_waitcnt vmcnt(%2)" : "+v"(a), "+v"(b) : "n"(N));
}
// a = 4 a + 2 [a0 >= t0] + [a1 >= t1], and b likewise: a compare and an add with carry per bit.  (In C++ the compiler makes a
// select, half a shift and half an or of every bit.)  A carry is read three instructions behind its compare; two are required.
__device__ __forceinline__ void append_bits(uint32_t& a, uint32_t& b, float a0, float b0, float t0, float a1, float b1, float t1) {
    unsigned long long c0, c1, c2, c3;
    asm("v_cmp_ge_f32_e64 %2, %6, %8\n\tv_cmp_ge_f32_e64 %3, %7, %8\n\tv_cmp_ge_f32_e64 %4, %9, %11\n\tv_cmp_ge_f32_e64 %5, %10, %11\n\t"
        "v_addc_co_u32_e64 %0, vcc, %0, %0, %2\n\tv_addc_co_u32_e64 %1, vcc, %1, %1, %3\n\t"
        "v_addc_co_u32_e64 %0, vcc, %0, %0, %4\n\tv_addc_co_u32_e64 %1, vcc, %1, %1, %5"
        : "+v"(a), "+v"(b), "=&s"(c0), "=&s"(c1), "=&s"(c2), "=&s"(c3)
        : "v"(a0), "v"(b0), "v"(t0), "v"(a1), "v"(b1), "v"(t1)
        : "vcc");
}
template <int LW>
__device__ __forceinline__ uint32_t word_of(const typename WordsOf<LW>::type& x, int u) {
    if constexpr (LW == 1) return x;
    else return x[u];
}

// Where a lane's N pixels (row blocks of 32 from m_base on) have their windows: byte offset of the
// first word of its half (half_bytes from the pixel's first), and a bit per tap that lies inside the image.
template <bool PAD, int N>
__device__ __forceinline__ void locate_windows(const DirectGeom& g, int m_base, int p, int half_bytes, uint32_t (&base)[N],
                                               uint32_t (&tbits)[N]) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int m = min(m_base + i * 32 + p, g.M - 1);
        const int b = fdiv(m, g.d_HoWo);
        const int r = m - b * g.HoWo;
        const int oy = fdiv(r, g.d_Wo);
        const int ox = r - oy * g.Wo;
        const int iy0 = oy * g.sh - g.ph, ix0 = ox * g.sw - g.pw;
        base[i] = static_cast<uint32_t>(((b * g.H + iy0) * g.W + ix0) * g.pix_bytes + half_bytes);
        tbits[i] = 0xFFFFFFFFu;
        if (PAD) {
            // bit t: tap t of the window lies inside the image (at most 32 taps, checked on the host): a run
            // of columns, the same for every window row inside
            const int x_lo = max(0, -ix0), n_in = min(g.kw, g.W - ix0) - x_lo;
            const uint32_t cols = n_in > 0 ? (0xFFFFFFFFu >> (32 - n_in)) << x_lo : 0u;
            uint32_t bitsv = 0;
            for (int ky = 0; ky < g.kh; ++ky)
                bitsv |= (static_cast<unsigned>(iy0 + ky) < static_cast<unsigned>(g.H) ? cols : 0u) << (ky * g.kw);
            tbits[i] = bitsv;
        }
    }
}

// LW    words per activation load (1, 2 or 4: the words of a half must divide into such loads)
// PF    load groups in the queue = groups per round of the reduction loop (the host picks one that
//       divides the number of groups where it can: a round past the end multiplies zeros)
// PAD   the layer has zero padding: taps are tested against the image per lane
// BITS  re-binarized output (packed signs) instead of fp32
template <int LW, int PF, bool PAD, bool BITS>
__global__ __launch_bounds__(512) void binconv_direct_kernel(const uint32_t* __restrict__ E, const uint32_t* __restrict__ A,
                                                             const float* __restrict__ alpha,
                                                             const float* __restrict__ beta,
                                                             const float* __restrict__ tau_out, const FastDiv d_wgs,
                                                             const DirectGeom g, float* __restrict__ Y,
                                                             int32_t* __restrict__ dbg_s1, uint32_t* __restrict__ out_bits) {
    constexpr int NFP = 4;                                         // 32-filter column blocks of a tile
    extern __shared__ __align__(16) uint4 panel[];                 // [n_ent][4][64 lanes] 16-byte groups; entries from nk on are zero
    __shared__ __align__(16) float sA_lds[8][64];                  // row sums of each wavefront's 64 pixels
    __shared__ __align__(16) float col_lds[3][kDirNTile];                        // beta - alpha, beta, tau of the tile's columns
    // The load groups of a tile in order: .x byte offset of the group inside the window (kOob past
    // the last one), .y its tap, and bit 8 where the upper half's word does not exist (the last group
    // of a tap with an odd number of words).  Read one group ahead by every lane (same address: a
    // broadcast), in place of a cursor of five scalar registers advanced by selects at every load.
    __shared__ uint2 gtab[kDirGroupTable];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int waves = static_cast<int>(blockDim.x >> 6);
    const int p = lane & 31, h = lane >> 5;
    const int ntile = fdiv(static_cast<int>(blockIdx.x), d_wgs);
    const int mt_first = static_cast<int>(blockIdx.x) - ntile * g.wg_per_ntile;
    const int f0 = ntile * kDirNTile;

    // ---- the B panel: bits -> fp4, once per workgroup.  Which filter sits in column n of column
    // block j is free to choose; it is filter 4n + j.  With fp32 output a lane then holds four
    // neighbouring filters of an output row in its four blocks and writes them with one 16-byte
    // store, a half-wavefront a whole 512-byte row segment; with bit output it holds sixteen neighbouring
    // bits of each of a pixel's words.  Item = (k-step, half): lane n reads the mask words of its four
    // filters, sixteen contiguous bytes.
    // Five entries of a wavefront at a time: their loads are in flight together (with eight
    // wavefronts that is the whole panel in one round trip).  The first five are requested before anything else is
    // worked out.
    constexpr int kBatch = 5;
    const int n_items = g.n_ent;
    uint32_t bits[kBatch][4];
    auto request_masks = [&](int ks0) {
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const int ks = ks0 + u * waves;
            const int tap = fdiv(min(ks, n_items - 1), g.d_WH);
            const int wd = h * g.WH + (ks - tap * g.WH);
#pragma unroll
            for (int j = 0; j < 4; ++j) bits[u][j] = 0u;
            if (ks < g.nk && wd < g.Cw && f0 + 4 * p < g.Fp) {       // (Fp is a multiple of 64: all four or none)
                const uint4 v = *reinterpret_cast<const uint4*>(E + static_cast<size_t>(tap * g.Cw + wd) * g.Fp + f0 + 4 * p);
                bits[u][0] = v.x; bits[u][1] = v.y; bits[u][2] = v.z; bits[u][3] = v.w;
            }
        }
    };
    auto expand_masks = [&](int ks0) {
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const int ks = ks0 + u * waves;
            if (ks < n_items) {
#pragma unroll
                for (int j = 0; j < 4; ++j) panel[(ks * 4 + j) * 64 + lane] = expand_e(bits[u][j]);
            }
        }
    };
    request_masks(wave);
    // scalars of the tile's 128 columns
    const int f_col = min(f0 + (tid & (kDirNTile - 1)), g.F - 1);
    const float al = alpha[f_col], be = beta[f_col], ta = BITS && tau_out ? tau_out[f_col] : 0.0f;
    __builtin_amdgcn_sched_barrier(0);

    // the packed activations as a raw buffer: offsets past its end read as zero
    const uint64_t a_addr = reinterpret_cast<uint64_t>(A);
    const v4s arsrc = {static_cast<int>(static_cast<uint32_t>(a_addr)), static_cast<int>(static_cast<uint32_t>(a_addr >> 32) & 0xFFFFu),
                       static_cast<int>(g.a_bytes), 0x00020000};
    // Load cursor: the windows whose words are being requested, and a group's two loads into a slot of the queue.
    // off, tap: where the group lies in the window; last_odd: its upper half's word does not exist (the last
    // group of a tap with an odd number of words per pixel)
    uint32_t base[2], tbits[2];
    locate_windows<PAD>(g, (mt_first * waves + wave) * 64, p, h * g.WH * 4, base, tbits);
    typename WordsOf<LW>::type xq[PF][2];
    auto request = [&](int slot, uint32_t off, uint32_t tap, bool last_odd) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            uint32_t voff = base[i] + off;
            if (PAD) voff = ((tbits[i] >> (tap & 31u)) & 1u) ? voff : kOob;
            if (LW == 1) voff = (h == 1 && last_odd) ? kOob : voff;
            load_words<LW>(xq[slot][i], arsrc, voff);
        }
    };
    // The first tile's first groups are requested before the panel is built, and every later tile's before the epilogue
    // of the tile in front, so that no tile begins with a round trip of its loads (with fp32 output its first wait counts
    // the stores of that epilogue too, so the gain there is small).  With the mask words requested before
    // the windows are worked out and the sums cleared in front of the barrier, what comes before the first multiply went from
    // 3.9 to 3.2 us: with the epilogue below, the six layers that hand bits on, batch 256, 102.7 -> 97.1 us, with fp32 output
    // 165.6 -> 163.8, 64 x 56 x 56 x 64 -> 64, 3 x 3, 25.6 -> 25.1.
    {
        int jg = 0, kx = 0;
        uint32_t tap = 0, off = 0, row = 0;                        // row: offset of the window row's first tap
#pragma unroll
        for (int d = 0; d < PF - 1; ++d) {
            request(d, d < g.NG ? off : kOob, tap, g.odd && jg == g.G - 1);
            const bool next_tap = ++jg == g.G;
            jg = next_tap ? 0 : jg;
            tap += next_tap ? 1 : 0;
            kx += next_tap ? 1 : 0;
            const bool next_row = kx == g.kw;
            kx = next_row ? 0 : kx;
            row += next_row ? static_cast<uint32_t>(g.W * g.pix_bytes) : 0u;
            off = row + static_cast<uint32_t>(kx * g.pix_bytes + jg * LW * 4);
        }
    }

    if (tid < kDirGroupTable) {
        uint2 e = make_uint2(kOob, 0u);
        if (tid < g.NG) {
            const int tap = tid / g.G, jg = tid - tap * g.G;
            const int ky = tap / g.kw, kx = tap - ky * g.kw;
            e.x = static_cast<uint32_t>(((ky * g.W + kx) * g.Cw + jg * LW) * 4);
            e.y = static_cast<uint32_t>(tap) | ((g.odd && jg == g.G - 1) ? 256u : 0u);
        }
        gtab[tid] = e;
    }
    expand_masks(wave);
    for (int ks0 = wave + kBatch * waves; ks0 < n_items; ks0 += kBatch * waves) {
        request_masks(ks0);
        expand_masks(ks0);
    }
    // the columns' scalars are kept in LDS (not in registers through the reduction loop), in filter order; the epilogues
    // index accordingly
    if (tid < kDirNTile) {
        col_lds[0][tid] = be - al;                                 // the accumulators hold -s1
        col_lds[1][tid] = be;
        col_lds[2][tid] = f0 + tid >= g.F ? __builtin_nanf("") : ta;
    }
    // the outputs as raw buffers (stores past their end are dropped)
    auto as_buffer = [](const void* ptr, uint32_t bytes) {
        const uint64_t a = reinterpret_cast<uint64_t>(ptr);
        return v4s{static_cast<int>(static_cast<uint32_t>(a)), static_cast<int>(static_cast<uint32_t>(a >> 32) & 0xFFFFu),
                   static_cast<int>(bytes), 0x00020000};
    };
    const v4s yrsrc = as_buffer(Y, g.y_bytes);
    const v4s drsrc = as_buffer(dbg_s1, dbg_s1 ? g.y_bytes : 0u);
    // the first tile's sums start before the barrier, every later tile's behind the epilogue of the tile in front
    v16f acc[2][NFP];
    auto clear = [&]() {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < NFP; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;
    };
    clear();
    __syncthreads();                                               // the panel is complete

    // the two masks of the expansion in registers (as literals they would split the and-or in two)
    uint32_t k8, k2;
    asm volatile("s_mov_b32 %0, 0x88888888" : "=s"(k8));
    asm volatile("v_mov_b32 %0, 0x22222222" : "=v"(k2));
    const uint4* bp = panel + lane;
    for (int mt = mt_first; mt < g.n_mtiles; mt += g.wg_per_ntile) {
        const int m_base = (mt * waves + wave) * 64;
        if (m_base >= g.M) break;                                  // (nor has a later tile pixels for this wavefront)
        int ones[2] = {0, 0};
        {
            // ---- the reduction.  Load groups run over (tap, word group); group gi covers k-steps
            // gi*LW .. gi*LW + LW-1.  PF groups are in flight (the first PF - 1 of a tile when it begins);
            // the slot emptied by the previous group is refilled during this one.  Groups between the last one and
            // the end of the round load nothing (zeros) and meet zero entries of the panel.  Where a group
            // lies comes from the table in LDS; the consume cursor is wavefront-uniform and advances by
            // selects, so a round of PF groups is one basic block.
            int l_g = PF - 1;
            uint2 nxt = gtab[l_g];                                 // the entry of group l_g
            auto issue = [&](int slot) {
                request(slot, nxt.x, nxt.y, (nxt.y & 256u) != 0u);
                ++l_g;
                nxt = gtab[l_g];
            };
            const uint4* bptr = bp;                                // B fragments of the round's first k-step
            // B fragments: one register set; a fragment is reloaded for the next k-step right behind the
            // two multiplies that read it, a whole k-step before its next use
            uint4 bq[NFP];
#pragma unroll
            for (int j = 0; j < NFP; ++j) bq[j] = bptr[j * 64];
            int c_tap = 0, c_jg = 0;                               // consume cursor
            // masks of a group's taps (zero for a tap outside the image)
            auto tap_masks = [&](uint32_t (&m8)[2], uint32_t (&m2)[2]) {
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const bool in = !PAD || ((tbits[i] >> (c_tap & 31)) & 1u);
                    m8[i] = in ? k8 : 0u;
                    m2[i] = in ? k2 : 0u;
                }
                ++c_jg;
                const bool cwrap = c_jg == g.G;
                c_jg = cwrap ? 0 : c_jg;
                c_tap += cwrap ? 1 : 0;
            };
            // The A fragments of a k-step are expanded during the k-step before it.
            uint32_t m8[2], m2[2];
            v4i an[2];
            tap_masks(m8, m2);
            {
                // the first group's words: PF - 2 younger groups are in flight
                wait_words<2 * (PF - 2)>(xq[0][0], xq[0][1]);
                const uint32_t x0 = word_of<LW>(xq[0][0], 0), x1 = word_of<LW>(xq[0][1], 0);
                ones[0] += __builtin_popcount(x0);
                ones[1] += __builtin_popcount(x1);
                an[0] = expand_a(x0, m8[0], m2[0]);
                an[1] = expand_a(x1, m8[1], m2[1]);
            }
            for (int g0 = 0; g0 < g.NG; g0 += PF, bptr += PF * LW * 256) {
#pragma unroll
                for (int d = 0; d < PF; ++d) {
#pragma unroll
                    for (int u = 0; u < LW; ++u) {
                        const int q = d * LW + u;                  // k-step of the round
                        const v4i a0 = an[0], a1 = an[1];
                        // the next k-step's words: the next word of this group, or the first of the
                        // next group (of the next round's first slot at the end of a round)
                        const int un = u + 1 < LW ? u + 1 : 0;
                        const int dn = u + 1 < LW ? d : (d + 1) % PF;
                        uint32_t x0 = 0, x1 = 0;
                        // Two multiplies, the reload of the fragment they have read and a quarter of the
                        // next step's vector work at a time; nothing moves across the fences between
                        // them.  (Left to the scheduler's own groups the reload ended up right in front
                        // of its use.  This order alone: six layers that hand bits on, batch 256, 103.2 ->
                        // 101.0 us, with fp32 output 174.7 -> 173.3, 64 x 56 x 56 x 64 -> 64 25.9 -> 25.7.)
                        for_each_column<NFP>([&](auto jc) {
                            constexpr int j = decltype(jc)::value;
                            const uint4 bu = bq[j];
                            const v4i bv = {static_cast<int>(bu.x), static_cast<int>(bu.y), static_cast<int>(bu.z),
                                            static_cast<int>(bu.w)};
                            // packed signs: the blocks transposed, so that a lane holds one pixel's filters
                            acc[0][j] = BITS ? mfma_fp4(bv, a0, acc[0][j]) : mfma_fp4(a0, bv, acc[0][j]);
                            acc[1][j] = BITS ? mfma_fp4(bv, a1, acc[1][j]) : mfma_fp4(a1, bv, acc[1][j]);
                            // (the panel ends with one entry more than the loop multiplies)
                            bq[j] = bptr[(q + 1) * 256 + j * 64];
                            if constexpr (j == 0) {
                                // the slot the previous group emptied is refilled PF - 1 groups ahead
                                if (u == 0) issue((d + PF - 1) % PF);
                            } else if constexpr (j == 1) {
                                if (un == 0) {
                                    tap_masks(m8, m2);
                                    wait_words<2 * (PF - 2)>(xq[dn][0], xq[dn][1]);   // PF - 2 younger groups are in flight
                                }
                                x0 = word_of<LW>(xq[dn][0], un);
                                x1 = word_of<LW>(xq[dn][1], un);
                                ones[0] += __builtin_popcount(x0);
                                ones[1] += __builtin_popcount(x1);
                            } else if constexpr (j == 2) {
                                an[0] = expand_a(x0, m8[0], m2[0]);
                            } else {
                                an[1] = expand_a(x1, m8[1], m2[1]);
                            }
                            __builtin_amdgcn_sched_barrier(0);
                        });
                    }
                }
            }

            // The loop leaves PF - 1 groups in flight (past the end: they load nothing, but their result
            // registers are written when they return): wait for them before those registers get another use.
#pragma unroll
            for (int d = 0; d < PF; ++d) asm volatile("s_waitcnt vmcnt(0)" : "+v"(xq[d][0]), "+v"(xq[d][1]));
            // ---- sA of this lane's rows: ones of both halves of a pixel, taps inside the image
            float sAv[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int both = ones[i] + __shfl_xor(ones[i], 32, 64);
                const int taps = PAD ? __builtin_popcount(tbits[i]) : g.T;
                sAv[i] = static_cast<float>(2 * both - taps * g.C);
            }
            // lane l holds row l of the 64 (row block l / 32, pixel l % 32); a wavefront reads back only
            // what it wrote itself: no workgroup barrier needed
            if (!BITS) sA_lds[wave][lane] = h ? sAv[1] : sAv[0];
            const int m_next = ((mt + g.wg_per_ntile) * waves + wave) * 64;
            if (mt + g.wg_per_ntile < g.n_mtiles && m_next < g.M) {
                locate_windows<PAD>(g, m_next, p, h * g.WH * 4, base, tbits);
#pragma unroll
                for (int d = 0; d < PF - 1; ++d) {
                    const uint2 e = gtab[d];
                    request(d, e.x, e.y, (e.y & 256u) != 0u);
                }
            }

            // ---- epilogue.  Register v of a 32x32 block is row (v/4)*8 + (lane/32)*4 + v%4, column
            // lane%32.  y = (beta - alpha)*(-s1) + beta*sA.
            if constexpr (BITS) {
                // The blocks are transposed here: register 4q + t of block j is filter 4(8q + 4(lane/32) + t) + j, which
                // is bit 16(lane/32) + 4t + j of word q, and the lane's pixel is column lane%32.  So a lane gathers
                // half of each word by itself, a bit a time from the highest down (the compare's carry is added to twice
                // the bits so far), and an exchange with the lane that has the same pixel's other filters completes
                // the words.  What bounds this is vector instructions, four a value.  (Pixels in rows, a ballot per register
                // and two lane writes to drop it into its row took 3.3-4.3 us per tile, more than a third of the
                // reduction; a select and an or per bit, a word's bits scattered over the lane's nibbles, 2.2-3.1; this
                // form 1.8-2.5.)  Columns past F compare against NaN.
                uint32_t half[2][NFP];
#pragma unroll
                for (int q = 0; q < NFP; ++q) {
                    half[0][q] = half[1][q] = 0u;
#pragma unroll
                    for (int t = 3; t >= 0; --t) {
                        const int c0 = q * 32 + h * 16 + t * 4;
                        const float4 d4 = *reinterpret_cast<const float4*>(&col_lds[0][c0]);
                        const float4 b4 = *reinterpret_cast<const float4*>(&col_lds[1][c0]);
                        const float4 t4 = *reinterpret_cast<const float4*>(&col_lds[2][c0]);
                        const float dv[4] = {d4.x, d4.y, d4.z, d4.w}, bv[4] = {b4.x, b4.y, b4.z, b4.w}, tv[4] = {t4.x, t4.y, t4.z, t4.w};
#pragma unroll
                        for (int j = 3; j >= 0; j -= 2) {
                            float y[2][2];
#pragma unroll
                            for (int i = 0; i < 2; ++i)
#pragma unroll
                                for (int k = 0; k < 2; ++k) y[i][k] = fmaf(dv[j - k], acc[i][j - k][q * 4 + t], bv[j - k] * sAv[i]);
                            append_bits(half[0][q], half[1][q], y[0][0], y[1][0], tv[j], y[0][1], y[1][1], tv[j - 1]);
                        }
                    }
                }
                // lane l stores row l of the 64: block i = h of its own pixel; two halves of words per exchange
                uint32_t wb[NFP];
#pragma unroll
                for (int q = 0; q < NFP; q += 2) {
                    const uint32_t gives = (h ? half[0][q] : half[1][q]) | ((h ? half[0][q + 1] : half[1][q + 1]) << 16);
                    const uint32_t gets = static_cast<uint32_t>(__shfl_xor(static_cast<int>(gives), 32, 64));
#pragma unroll
                    for (int k = 0; k < 2; ++k) {
                        const uint32_t mine = h ? half[1][q + k] : half[0][q + k], other = k ? gets >> 16 : gets & 0xFFFFu;
                        wb[q + k] = h ? other | (mine << 16) : mine | (other << 16);
                    }
                }
                const int row = m_base + lane;
                const int Fw = (g.F + 31) >> 5;
                if (row < g.M) {
                    uint32_t* dst = out_bits + static_cast<size_t>(row) * Fw + (f0 >> 5);
                    if ((Fw & 3) == 0) {
                        store_u32x4(dst, v4u{wb[0], wb[1], wb[2], wb[3]});
                    } else {
#pragma unroll
                        for (int j = 0; j < NFP; ++j)
                            if ((f0 >> 5) + j < Fw) store_u32(dst + j, wb[j]);
                    }
                }
                clear();
                continue;
            }
            // fp32 output.  Column n of block j is filter 4n + j, so the four
            // blocks of a register index are four neighbouring filters of one output row: one
            // 16-byte store per lane, 512 contiguous bytes per half-wavefront, two rows per
            // instruction.  Y (and the optional integer dump) are raw buffers: the lane's offset
            // (first row of its half, its four filters) plus a scalar row offset; rows past M fall
            // outside the buffer and are dropped by the range check.
            static_assert(NFP == 4, "the epilogues store all four column blocks of a row together");
            float4 s4[2][4];
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    s4[i][q] = *reinterpret_cast<const float4*>(&sA_lds[wave][i * 32 + q * 8 + h * 4]);
            const float4 d4 = *reinterpret_cast<const float4*>(&col_lds[0][4 * p]);
            const float4 b4 = *reinterpret_cast<const float4*>(&col_lds[1][4 * p]);
            const float dv[4] = {d4.x, d4.y, d4.z, d4.w}, bv[4] = {b4.x, b4.y, b4.z, b4.w};
            const int fl = f0 + 4 * p;                             // first of this lane's four filters
            const uint32_t lane_off = static_cast<uint32_t>(((m_base + h * 4) * g.F + fl) * 4);
            // Offsets of the lane's stores, kept in registers (worked out again in front of every store, into a register that
            // the store before it still reads, they slowed narrow tiles by up to 13 %): of the four values together, and, in
            // the one lane whose four filters the last one is among, of each by itself.  A 16-byte store needs 4-byte alignment
            // only, so rows of any number of filters take it.  (As single
            // values: 111475 pixels x 9 steps x 175 filters 44.0 us, now 23.0; 78608 x 18 x 182 45.7 and 23.7.)
            uint32_t off4 = fl + 4 <= g.F ? lane_off : kOobStore, off1[3];
            asm volatile("" : "+v"(off4));
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                off1[j] = fl + 4 > g.F && fl + j < g.F ? lane_off + 4 * j : kOobStore;
                asm volatile("" : "+v"(off1[j]));
            }
            const bool tail = (g.F & 3) != 0 && f0 + kDirNTile > g.F;
            auto store_tile = [&](auto policy) {
#pragma unroll
                for (int i = 0; i < 2; ++i) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const float sv[4] = {s4[i][q].x, s4[i][q].y, s4[i][q].z, s4[i][q].w};
#pragma unroll
                        for (int t = 0; t < 4; ++t) {
                            const uint32_t row_off = static_cast<uint32_t>((i * 32 + q * 8 + t) * g.F * 4);   // scalar
                            float y[4];
#pragma unroll
                            for (int j = 0; j < 4; ++j) y[j] = fmaf(dv[j], acc[i][j][q * 4 + t], bv[j] * sv[t]);
                            store_buffer_x4<decltype(policy)::value>(v4f{y[0], y[1], y[2], y[3]}, off4, yrsrc, row_off);
                            if constexpr (decltype(policy)::value == kStorePlain) {
                                if (tail) {
#pragma unroll
                                    for (int j = 0; j < 3; ++j) store_buffer(y[j], off1[j], yrsrc, row_off);
                                }
                                if (dbg_s1) {
                                    float n[4];
#pragma unroll
                                    for (int j = 0; j < 4; ++j) n[j] = __int_as_float(-static_cast<int>(acc[i][j][q * 4 + t]));
                                    store_buffer_x4<kStorePlain>(v4f{n[0], n[1], n[2], n[3]}, off4, drsrc, row_off);
#pragma unroll
                                    for (int j = 0; j < 3; ++j) store_buffer(n[j], off1[j], drsrc, row_off);
                                }
                            }
                        }
                    }
                }
            };
            // (rows of whole 16-byte stores, and nothing else to store, outside the default policy)
            if (g.store_policy == kStoreStream && !dbg_s1) store_tile(std::integral_constant<int, kStoreStream>{});
            else if (g.store_policy == kStoreThrough && !dbg_s1) store_tile(std::integral_constant<int, kStoreThrough>{});
            else store_tile(std::integral_constant<int, kStorePlain>{});
            clear();
        }
    }
    // (a wavefront without a tile leaves with its first requests answered)
#pragma unroll
    for (int d = 0; d < PF - 1; ++d) asm volatile("s_waitcnt vmcnt(0)" : "+v"(xq[d][0]), "+v"(xq[d][1]));
}

// ---------------------------------------------------------------- small products
// Layers with a few hundred 32 x 32 output blocks at most (the last layers of the Sketch-A-Net
// trunk, a late ResNet stage at small batch) are latency problems: too few tiles for the
// persistent kernel above.  Here one workgroup owns one 32-pixel x 32-filter block and its
// wavefronts take consecutive shares of the reduction.  Both operands are read as packed bits
// straight from memory (L2), DEPTH k-steps per burst into two register sets, expanded in
// registers and multiplied; the wavefronts' exact partial sums (and their counts of ones for
// sA) are added through LDS.  Workgroups that share a block of filters are neighbours on an XCD, so
// the filter words are fetched into few L2s.

template <bool PAD, bool BITS, int WAVES, int DEPTH, int LW>
__global__ __launch_bounds__(64 * WAVES) void binconv_block_kernel(const DirectGeom g, const BlockGeom bg,
                                                                   const uint32_t* __restrict__ A,
                                                                   const uint32_t* __restrict__ E,
                                                                   const float* __restrict__ alpha,
                                                                   const float* __restrict__ beta, float* __restrict__ Y,
                                                                   int32_t* __restrict__ dbg_s1,
                                                                   const float* __restrict__ tau_out,
                                                                   uint32_t* __restrict__ out_bits) {
    __shared__ float red[WAVES][16][64];
    __shared__ int ones_lds[WAVES][64];
    DAB_RESERVE_VGPRS();
    const int lane = threadIdx.x & 63, p = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // Block of this workgroup: consecutive workgroups go to consecutive XCDs, and an XCD takes a contiguous run of blocks,
    // pixel blocks of one filter block next to each other.  (A filter block to one XCD left XCDs without work where
    // there are fewer than eight, or not a multiple of eight: 14175 pixels x 144 steps x 21 59 us, now
    // 12.3; 13454 x 95 x 20 41 and 9.0.)
    const int unit = static_cast<int>(blockIdx.x % kNumXCD) * bg.per_xcd + static_cast<int>(blockIdx.x / kNumXCD);
    if (unit >= bg.units) return;                                  // (the whole workgroup)
    const int fb = fdiv(unit, bg.d_mblocks);
    const int mb = unit - fb * bg.n_mblocks;

    const __amdgpu_buffer_rsrc_t arsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(A), 0, static_cast<int>(g.a_bytes), 0x00020000);
    const __amdgpu_buffer_rsrc_t ersrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(E), 0, static_cast<int>(bg.e_bytes), 0x00020000);
    const int fcol = fb * 32 + p;                                  // this lane's filter (as the B operand's column)
    const uint32_t ecol = fcol < g.Fp ? static_cast<uint32_t>(fcol * 4) : kOob;
    // the filter's scalars, which the epilogue would otherwise wait for behind the barrier (with the mask words requested
    // before the windows are worked out and one barrier in place of two: conv4 of the sketch network, one image, 4.4 -> 4.0 us)
    const int f = min(fcol, g.F - 1);
    const float al = alpha[f], be = beta[f], tcol = (BITS && tau_out) ? tau_out[f] : 0.0f;

    // this wavefront's k-steps [k0, k1): k-step ks = tap * WH + j multiplies word h*WH + j of the tap.
    // A lane's activation words of a tap are neighbours in memory: with LW = 4 (WH a multiple of four)
    // one 16-byte load brings four k-steps, and a wavefront's load touches a quarter of the cache
    // lines per k-step (its lanes read different pixels, a line each).
    static_assert((LW == 1 || LW == 4) && DEPTH % LW == 0, "whole loads per burst");
    constexpr int NL = DEPTH / LW;
    const int per = (g.nk + WAVES * LW - 1) / (WAVES * LW) * LW;
    const int k0 = min(wave * per, g.nk), k1 = min(k0 + per, g.nk);
    typename WordsOf<LW>::type xa[2][NL];
    uint32_t xe[2][DEPTH];
    bool va[2][NL];
    uint32_t base1[1], tbits1[1];
    auto fetch = [&](int set, int first, bool masks, bool words) {
#pragma unroll
        for (int l = 0; l < NL; ++l) {
            const int ks = first + l * LW;                         // (wavefront-uniform; a multiple of LW)
            const int tap = fdiv(min(ks, g.nk - 1), g.d_WH);
            const int j = min(ks, g.nk - LW) - tap * g.WH;
            const int ky = fdiv(tap, bg.d_kw);
            const int kx = tap - ky * g.kw;
            const int wd = h * g.WH + j;
            const bool live = ks < k1 && wd < g.Cw;                // (LW = 4: Cw = 2 WH, all four words or none)
            if (masks) {
#pragma unroll
                for (int u = 0; u < LW; ++u) {
                    const uint32_t eoff = ecol + static_cast<uint32_t>((tap * g.Cw + wd + u) * g.Fp * 4);
                    xe[set][l * LW + u] = __builtin_amdgcn_raw_buffer_load_b32(ersrc, static_cast<int>(live ? eoff : kOob), 0, 0);
                }
            }
            if (!words) continue;
            const uint32_t base = base1[0], tbits = tbits1[0];
            const bool in = live && (!PAD || ((tbits >> (tap & 31)) & 1u));
            const uint32_t aoff = base + static_cast<uint32_t>(((ky * g.W + kx) * g.Cw + j) * 4);
            if constexpr (LW == 1) {
                xa[set][l] = __builtin_amdgcn_raw_buffer_load_b32(arsrc, static_cast<int>(in ? aoff : kOob), 0, 0);
            } else {
                xa[set][l] = __builtin_bit_cast(v4u, __builtin_amdgcn_raw_buffer_load_b128(arsrc, static_cast<int>(in ? aoff : kOob), 0, 0));
            }
            va[set][l] = in;
        }
    };
    const SignMasks masks = sign_masks();
    v16f acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.0f;
    int ones = 0;
    auto multiply = [&](int set) {
#pragma unroll
        for (int d = 0; d < DEPTH; ++d) {
            const uint32_t x = word_of<LW>(xa[set][d / LW], d % LW);
            ones += __builtin_popcount(x);                         // (words that were not loaded are zero)
            const v4i a = expand_a_in_place(x, masks_where(va[set][d / LW], masks));
            const uint4 e = expand_e_in_place(xe[set][d]);
            const v4i bv = {static_cast<int>(e.x), static_cast<int>(e.y), static_cast<int>(e.z), static_cast<int>(e.w)};
            acc = mfma_fp4<true>(a, bv, acc);                      // (a k-step past k1 multiplies zeros)
        }
    };
    // the first mask words are requested before the windows are worked out: byte offset of word h*WH of the window's
    // first tap, taps inside the image
    fetch(0, k0, true, false);
    locate_windows<PAD>(g, mb * 32, p, h * g.WH * 4, base1, tbits1);
    fetch(0, k0, false, true);
    for (int st = k0; st < k1; st += 2 * DEPTH) {
        fetch(1, st + DEPTH, true, true);
        multiply(0);
        fetch(0, st + 2 * DEPTH, true, true);
        multiply(1);
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) red[wave][v][lane] = acc[v];
    ones_lds[wave][lane] = ones;
    __syncthreads();
    // sA of pixel p, in every wavefront: ones of both halves and all wavefronts, taps inside the image
    int both = 0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) both += ones_lds[w][lane];
    both += __shfl_xor(both, 32, 64);
    const int taps = PAD ? __builtin_popcount(tbits1[0]) : g.T;
    const float sA = static_cast<float>(2 * both - taps * g.C);

    // register v of lane l is row (v/4)*8 + (l/32)*4 + v%4 of the block, column l%32; wavefront w
    // finishes registers w, w + WAVES, ...  The accumulators hold -s1.
    const bool fvalid = fcol < g.F;
    const float dcol = be - al;
    const int Fw = (g.F + 31) >> 5;
#pragma unroll
    for (int v = wave; v < 16; v += WAVES) {
        const int rl = (v >> 2) * 8 + h * 4 + (v & 3);
        const int row = mb * 32 + rl;
        float ns1 = 0.0f;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) ns1 += red[w][v][lane];
        const float y = fmaf(dcol, ns1, be * __shfl(sA, rl, 64));
        if (BITS) {
            const unsigned long long mask = __ballot(fvalid && y >= tcol);
            const uint32_t word = static_cast<uint32_t>(lane < 32 ? mask : mask >> 32);
            if (p == 0 && row < g.M) out_bits[static_cast<size_t>(row) * Fw + fb] = word;
        } else if (row < g.M && fvalid) {
            const size_t o = static_cast<size_t>(row) * g.F + fcol;
            Y[o] = y;
            if (dbg_s1) dbg_s1[o] = -static_cast<int>(ns1);
        }
    }
}

// ---------------------------------------------------------------- long reductions
// Reductions whose B fragments do not fit in LDS (more than kDirMaxSteps k-steps) over more blocks
// than the small kernel above is for: the wide fully-connected layers at a training batch, large
// windows over many channels.  A wavefront computes 64 pixels x 128 filters over a share of the
// reduction, with both operands read as packed bits and expanded in registers: per k-step 34 vector
// instructions beside eight multiplies, which hide them (two wavefronts per SIMD: the multiplies are
// 65 % of the issue time).  The eight wavefronts of a workgroup are 8 / KS pixel blocks x KS shares of
// the reduction; the shares' exact partial sums are added through LDS, each wavefront finishing a
// KS-th of the rows.  Nothing is staged, no workspace, one launch; the only barrier is that of the
// exchange.  (The form it replaces expanded both operands into a workspace, multiplied from there and
// added the shares in a third launch: 1024 x 9216 x 4096 took 9.8 + 29.5 + 18.5 us.)
constexpr int kSplitWaves = 8;
constexpr int kSplitLds = kSplitWaves * 16 * 64 * 16;              // bytes of the exchange between the shares

template <int LW, bool PAD, bool BITS>
__global__ __launch_bounds__(64 * kSplitWaves) void binconv_split_kernel(const DirectGeom g, const SplitGeom sg,
                                                                        const uint32_t* __restrict__ A,
                                                                        const uint32_t* __restrict__ E,
                                                                        const float* __restrict__ alpha,
                                                                        const float* __restrict__ beta,
                                                                        float* __restrict__ Y, int32_t* __restrict__ dbg_s1,
                                                                        const float* __restrict__ tau_out,
                                                                        uint32_t* __restrict__ out_bits) {
    constexpr int NFP = 4;
    constexpr int STEPS = 8;                                       // k-steps per round, and weight loads in the queue
    constexpr int PF = STEPS / LW;                                 // activation load groups per round and in the queue
    extern __shared__ __align__(16) float4 red[];                  // [wave][register row e of a block row][lane]: the exchange
    uint4* const red16 = reinterpret_cast<uint4*>(red);            // the same of both block rows, 16 bits a sum
    __shared__ int ones_lds[2][kSplitWaves][64];
    __shared__ __align__(16) float sA_lds[kSplitWaves][64];
    __shared__ __align__(16) float col_lds[3][kDirNTile];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int p = lane & 31, h = lane >> 5;
    // an XCD takes a contiguous run of tiles, pixel tiles of one filter tile next to each other
    const int unit = static_cast<int>(blockIdx.x % kNumXCD) * sg.per_xcd + static_cast<int>(blockIdx.x / kNumXCD);
    if (unit >= sg.units) return;                                  // (the whole workgroup)
    const int ntile = fdiv(unit, sg.d_mtiles);
    const int mt = unit - ntile * sg.n_mtiles;
    const int f0 = ntile * kDirNTile;
    const int share = wave & ((1 << sg.log_ks) - 1), mw = wave >> sg.log_ks;
    const int m_base = (mt * (kSplitWaves >> sg.log_ks) + mw) * 64;
    // the load groups of this wavefront (none for a block past the last pixel)
    const int g_first = min(share * sg.groups_per_share, g.NG);
    const int g_end = m_base < g.M ? min(g_first + sg.groups_per_share, g.NG) : g_first;

    // scalars of the tile's columns: requested in front of the operands and put into LDS behind the operands' requests
    const int f_col = min(f0 + (tid & (kDirNTile - 1)), g.F - 1);
    const float al = alpha[f_col], be = beta[f_col], ta = BITS && tau_out ? tau_out[f_col] : 0.0f;
    auto keep_columns = [&]() {
        __builtin_amdgcn_sched_barrier(0);
        if (tid < kDirNTile) {
            col_lds[0][tid] = be - al;                             // the accumulators hold -s1
            col_lds[1][tid] = be;
            col_lds[2][tid] = f0 + tid >= g.F ? __builtin_nanf("") : ta;
        }
    };
    const __amdgpu_buffer_rsrc_t arsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(A), 0, static_cast<int>(g.a_bytes), 0x00020000);
    const __amdgpu_buffer_rsrc_t ersrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(E), 0, static_cast<int>(sg.e_bytes), 0x00020000);
    // The halves of a tap's words alternate by load: words [2 LW jg, + LW) of group jg belong to lanes 0..31,
    // the next LW to lanes 32..63, so a load takes 2 LW neighbouring words of every pixel (with the halves
    // WH words apart a long row's load touched twice the cache lines).
    uint32_t base[2], tbits[2];
    locate_windows<PAD>(g, m_base, p, h * LW * 4, base, tbits);

    // ---- load cursors (wavefront-uniform).  Offsets past the end are kOob: such loads return zeros, a
    // zero mask word multiplies to nothing and a zero activation word counts no ones.
    const int tap0 = fdiv(min(g_first, g.NG - 1), sg.d_G);
    int a_left = g_end - g_first;                                  // activation groups still to request
    int a_jg = min(g_first, g.NG - 1) - tap0 * g.G, a_tap = tap0;
    int a_kx = tap0 - fdiv(tap0, sg.d_kw) * g.kw;
    uint32_t a_off = static_cast<uint32_t>(((fdiv(tap0, sg.d_kw) * g.W + a_kx) * g.Cw + a_jg * 2 * LW) * 4);
    typename WordsOf<LW>::type xa[PF][2];
    auto request_a = [&](int slot) {
        const bool live = a_left > 0;
        const uint32_t off = live ? a_off : kOob;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            uint32_t voff = base[i] + off;
            if (PAD) voff = ((tbits[i] >> (a_tap & 31)) & (live ? 1u : 0u)) ? voff : kOob;
            // an odd number of words per pixel: the upper half's last word does not exist
            if (LW == 1) voff = (h == 1 && g.odd && a_jg == g.G - 1) ? kOob : voff;
            if constexpr (LW == 1) xa[slot][i] = __builtin_amdgcn_raw_buffer_load_b32(arsrc, static_cast<int>(voff), 0, 0);
            else if constexpr (LW == 2) xa[slot][i] = __builtin_bit_cast(v2u, __builtin_amdgcn_raw_buffer_load_b64(arsrc, static_cast<int>(voff), 0, 0));
            else xa[slot][i] = __builtin_bit_cast(v4u, __builtin_amdgcn_raw_buffer_load_b128(arsrc, static_cast<int>(voff), 0, 0));
        }
        --a_left;
        const bool next_tap = ++a_jg == g.G;
        a_jg = next_tap ? 0 : a_jg;
        a_tap += next_tap ? 1 : 0;
        a_kx += next_tap ? 1 : 0;
        const bool next_row = a_kx == g.kw;
        a_kx = next_row ? 0 : a_kx;
        a_off += next_row ? g.step_ky : (next_tap ? g.step_kx : static_cast<uint32_t>(2 * LW * 4));
    };
    int b_left = (g_end - g_first) * LW;                           // weight steps still to request
    int b_jg = min(g_first, g.NG - 1) - tap0 * g.G;
    uint32_t b_off = static_cast<uint32_t>((tap0 * g.Cw + b_jg * 2 * LW) * g.Fp * 4);
    // lane n takes the sixteen bytes of filters 4n .. 4n+3 of a row of E
    const uint32_t b_lane = f0 + 4 * p < g.Fp ? static_cast<uint32_t>((h * LW * g.Fp + f0 + 4 * p) * 4) : kOob;
    v4u xb[STEPS];
    auto request_b = [&](int slot, bool last_of_group) {
        uint32_t voff = b_lane + (b_left > 0 ? b_off : kOob);
        if (LW == 1) voff = (h == 1 && g.odd && b_jg == g.G - 1) ? kOob : voff;
        xb[slot] = __builtin_bit_cast(v4u, __builtin_amdgcn_raw_buffer_load_b128(ersrc, static_cast<int>(voff), 0, 0));
        --b_left;
        // rows of a group's upper half lie between its own and the next group's (an odd tap ends without one)
        if (last_of_group) {
            const bool next_tap = ++b_jg == g.G;
            b_jg = next_tap ? 0 : b_jg;
            b_off += static_cast<uint32_t>((LW == 1 && next_tap && g.odd ? 1 : LW + 1) * g.Fp * 4);
        } else {
            b_off += static_cast<uint32_t>(g.Fp * 4);
        }
    };

    // Partial sums that the shares exchange as 16-bit numbers count from 1.5 * 2^23: the low half of such a float is the
    // sum's, modulo 2^16.  (Register by register: eight equal initial values in C++ are made by copying one tuple, which
    // costs scratch memory here.)
    const float start = sg.narrow ? 12582912.0f : 0.0f;
    v16f acc[2][NFP];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < NFP; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) asm volatile("v_mov_b32 %0, %1" : "=v"(acc[i][j][v]) : "s"(start));
    int ones[2] = {0, 0};

    if (g_first < g_end) {
        // requests in the order of their use, a whole round of them in flight
        for_each_column<STEPS>([&](auto qc) {
            constexpr int q = decltype(qc)::value;
            if constexpr (q % LW == 0) request_a(q / LW);
            request_b(q, q % LW == LW - 1);
        });
        keep_columns();
        const SignMasks masks = sign_masks();
        int c_tap = tap0, c_jg = min(g_first, g.NG - 1) - tap0 * g.G;       // consume cursor
        SignMasks m[2];
        auto tap_masks = [&]() {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                m[i] = masks_where(!PAD || ((tbits[i] >> (c_tap & 31)) & 1u), masks);
            }
            const bool next_tap = ++c_jg == g.G;
            c_jg = next_tap ? 0 : c_jg;
            c_tap += next_tap ? 1 : 0;
        };
        tap_masks();
        v4i an[2];
        {
            const uint32_t x0 = word_of<LW>(xa[0][0], 0), x1 = word_of<LW>(xa[0][1], 0);
            ones[0] += __builtin_popcount(x0);
            ones[1] += __builtin_popcount(x1);
            an[0] = expand_a_in_place(x0, m[0]);
            an[1] = expand_a_in_place(x1, m[1]);
        }
        uint4 bn = expand_e_in_place(xb[0][0]);
        // One k-step: two multiplies, the expansion of the next column block's weights and a quarter of the
        // next step's activations at a time, in this order (fences between them).  A queue slot is
        // requested again as soon as its last word has been expanded, a round ahead of its use.
        auto step = [&](auto qc, auto more) {
            constexpr int q = decltype(qc)::value, qn = (q + 1) % STEPS;
            constexpr int u = q % LW, d = q / LW, un = qn % LW, dn = qn / LW;
            const v4i a0 = an[0], a1 = an[1];
            uint32_t x0 = 0, x1 = 0;
            for_each_column<NFP>([&](auto jc) {
                constexpr int j = decltype(jc)::value;
                const v4i bv = {static_cast<int>(bn.x), static_cast<int>(bn.y), static_cast<int>(bn.z), static_cast<int>(bn.w)};
                acc[0][j] = mfma_fp4(a0, bv, acc[0][j]);
                acc[1][j] = mfma_fp4(a1, bv, acc[1][j]);
                bn = expand_e_in_place(j + 1 < NFP ? xb[q][(j + 1) % NFP] : xb[qn][0]);
                if constexpr (j == 0) {
                    if constexpr (u == LW - 1 && decltype(more)::value) request_a(d);
                    if constexpr (un == 0) tap_masks();
                } else if constexpr (j == 1) {
                    x0 = word_of<LW>(xa[dn][0], un);
                    x1 = word_of<LW>(xa[dn][1], un);
                    ones[0] += __builtin_popcount(x0);
                    ones[1] += __builtin_popcount(x1);
                } else if constexpr (j == 2) {
                    an[0] = expand_a_in_place(x0, m[0]);
                } else {
                    an[1] = expand_a_in_place(x1, m[1]);
                    if constexpr (decltype(more)::value) request_b(q, u == LW - 1);
                }
                __builtin_amdgcn_sched_barrier(0);
            });
        };
        // whole rounds, then half a round where that is enough (steps past the end multiply zeros; a loop
        // left in the middle of a round lets the compiler sink the requests behind the exits)
        const int steps = (g_end - g_first) * LW;
        int left = steps;
        for (; left > STEPS / 2; left -= STEPS) for_each_column<STEPS>([&](auto qc) { step(qc, std::true_type{}); });
        if (left > 0) for_each_column<STEPS / 2>([&](auto qc) { step(qc, std::false_type{}); });
    } else {
        keep_columns();
    }

    // ---- what the workgroup's wavefronts hand each other: counts of ones and, in 16-bit numbers, the sums
    ones_lds[0][wave][lane] = ones[0];
    ones_lds[1][wave][lane] = ones[1];
    // ---- epilogue.  Register row e = 4q + t of block row i is output row i*32 + q*8 + (lane/32)*4 + t,
    // column n of block j is filter 4n + j.  y = (beta - alpha)*(-s1) + beta*sA.
    float4 d4, b4, t4;
    auto read_columns = [&]() {                                    // (behind a barrier)
        d4 = *reinterpret_cast<const float4*>(&col_lds[0][4 * p]);
        b4 = *reinterpret_cast<const float4*>(&col_lds[1][4 * p]);
        t4 = *reinterpret_cast<const float4*>(&col_lds[2][4 * p]);
    };
    const int fl = f0 + 4 * p;
    const int Fw = (g.F + 31) >> 5;
    auto finish = [&](int i, int e, float4 ns1) {
        const int rl = i * 32 + (e >> 2) * 8 + h * 4 + (e & 3);
        const int row = m_base + rl;
        const float sv = sA_lds[wave][rl];
        const float y[4] = {fmaf(d4.x, ns1.x, b4.x * sv), fmaf(d4.y, ns1.y, b4.y * sv), fmaf(d4.z, ns1.z, b4.z * sv),
                            fmaf(d4.w, ns1.w, b4.w * sv)};
        if constexpr (BITS) {
            // the ballot of block j holds filters 4n + j of both rows; lane w < 4 of a half interleaves
            // the four bytes that make up word w of its row
            const unsigned long long b[4] = {__ballot(y[0] >= t4.x), __ballot(y[1] >= t4.y), __ballot(y[2] >= t4.z), __ballot(y[3] >= t4.w)};
            uint32_t word = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                uint32_t x = (static_cast<uint32_t>(h ? b[j] >> 32 : b[j]) >> (8 * (p & 3))) & 0xFFu;
                x = (x | (x << 12)) & 0x000F000Fu;
                x = (x | (x << 6)) & 0x03030303u;
                x = (x | (x << 3)) & 0x11111111u;
                word |= x << j;
            }
            if (p < 4 && row < g.M && (f0 >> 5) + p < Fw) out_bits[static_cast<size_t>(row) * Fw + (f0 >> 5) + p] = word;
        } else if (row < g.M) {
            // (rows of any number of filters: a 16-byte store needs 4-byte alignment only; 10300 x 25 x 202 16.4 -> 14.0 us)
            typedef float v4f_any __attribute__((ext_vector_type(4), aligned(4)));
            const size_t o = static_cast<size_t>(row) * g.F + fl;
            if ((g.F & 3) == 0 && !dbg_s1) {
                if (fl < g.F) *reinterpret_cast<float4*>(Y + o) = make_float4(y[0], y[1], y[2], y[3]);
            } else if (fl + 4 <= g.F && !dbg_s1) {
                *reinterpret_cast<v4f_any*>(Y + o) = v4f_any{y[0], y[1], y[2], y[3]};
            } else {
                const float n[4] = {ns1.x, ns1.y, ns1.z, ns1.w};
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (fl + j < g.F) {
                        Y[o + j] = y[j];
                        if (dbg_s1) dbg_s1[o + j] = -static_cast<int>(n[j]);
                    }
            }
        }
    };
    // ones of a pixel: both halves, all shares.  lane l: row l of the block (read back by this wavefront only)
    auto row_sums = [&](int both) {
        const int taps = PAD ? __builtin_popcount(h ? tbits[1] : tbits[0]) : g.T;
        sA_lds[wave][lane] = static_cast<float>(2 * both - taps * g.C);
    };
    // Sums of 16-bit numbers: the exact sum of at most 2^15 - 1 terms is what it is modulo 2^16, whatever the shares' own.
    // Half the bytes of an exchange of fp32 sums, so both block rows fit in LDS at once, one barrier in place of
    // four, and with the number of shares known all reads of a wavefront are in flight together.  With the columns'
    // scalars requested instead of waited for in front of the operands: 7200 pixels x 36 steps x 256, eight shares, 10.4 ->
    // 7.5 us, 12312 x 50 x 150 (signs), four shares, 15.7 -> 13.6, 1024 x 9216 x 4096, four shares, 23.7 -> 21.6.
    auto exchange16 = [&](auto lk) {
        constexpr int KS = 1 << decltype(lk)::value, PER = 16 / KS;
        int both = 0;
#pragma unroll
        for (int k = 0; k < KS; ++k) both += ones_lds[h][mw * KS + k][p] + ones_lds[h][mw * KS + k][p + 32];
        row_sums(both);
        typedef short v2s __attribute__((ext_vector_type(2)));
        v2s s[PER][4];
#pragma unroll
        for (int n = 0; n < PER; ++n)
#pragma unroll
            for (int k = 0; k < KS; ++k) {
                const uint4 v = red16[((mw * KS + k) * 16 + share * PER + n) * 64 + lane];
                const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const v2s t = __builtin_bit_cast(v2s, w[c]);
                    s[n][c] = k ? s[n][c] + t : t;
                }
            }
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int n = 0; n < PER; ++n) {
                finish(i, share * PER + n, make_float4(s[n][2 * i].x, s[n][2 * i].y, s[n][2 * i + 1].x, s[n][2 * i + 1].y));
                __builtin_amdgcn_sched_barrier(0);
            }
    };
    if (sg.narrow) {
        // low halves of two registers in a word
        auto low_halves = [](float lo, float hi) { return __builtin_amdgcn_perm(__float_as_uint(hi), __float_as_uint(lo), 0x05040100u); };
#pragma unroll
        for (int e = 0; e < 16; ++e)
            red16[(wave * 16 + e) * 64 + lane] =
                make_uint4(low_halves(acc[0][0][e], acc[0][1][e]), low_halves(acc[0][2][e], acc[0][3][e]),
                           low_halves(acc[1][0][e], acc[1][1][e]), low_halves(acc[1][2][e], acc[1][3][e]));
        __syncthreads();
        read_columns();
        if (sg.log_ks == 3) exchange16(std::integral_constant<int, 3>{});
        else if (sg.log_ks == 2) exchange16(std::integral_constant<int, 2>{});
        else exchange16(std::integral_constant<int, 1>{});
        return;
    }
    // One share, or sums that 16 bits do not hold.
    __syncthreads();
    read_columns();
    const int ks = 1 << sg.log_ks;
    int both = 0;
    for (int k = 0; k < ks; ++k) both += ones_lds[h][mw * ks + k][p] + ones_lds[h][mw * ks + k][p + 32];
    row_sums(both);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        if (ks == 1) {
#pragma unroll
            for (int e = 0; e < 16; ++e) finish(i, e, make_float4(acc[i][0][e], acc[i][1][e], acc[i][2][e], acc[i][3][e]));
            continue;
        }
        if (i == 1) __syncthreads();                               // the first block row's sums have been read
#pragma unroll
        for (int e = 0; e < 16; ++e)
            red[(wave * 16 + e) * 64 + lane] = make_float4(acc[i][0][e], acc[i][1][e], acc[i][2][e], acc[i][3][e]);
        __syncthreads();
        const int per = 16 >> sg.log_ks;
        for (int e = share * per; e < (share + 1) * per; ++e) {
            float4 s = red[(mw * ks * 16 + e) * 64 + lane];
            for (int k = 1; k < ks; ++k) {
                const float4 v = red[((mw * ks + k) * 16 + e) * 64 + lane];
                s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;    // (exact: whole numbers below 2^24)
            }
            finish(i, e, s);
        }
    }
}

// ------------------------------------------------------------------ host side

// Whether the direct kernel covers the layer, and its geometry.  It needs the B fragments of the
// whole reduction in LDS (at most kDirMaxSteps k-steps) and, for padded layers, a window of at
// most 32 taps (one validity bit per tap and lane).
constexpr int kDirMaxSteps = 36;

// The layer's geometry for the kernels that read packed bits through 64-pixel blocks; false where their
// offsets (30 bits) or tap masks (32 taps of a padded window) do not reach.
static bool describe(const dab_conv_desc& d, DirectGeom* pg, bool* pad, int* lw) {
    DirectGeom& g = *pg;
    g = DirectGeom{};
    g.H = d.H; g.W = d.W; g.C = d.C; g.F = d.F; g.kh = d.kh; g.kw = d.kw;
    g.ph = d.pad_h; g.pw = d.pad_w; g.sh = d.stride_h; g.sw = d.stride_w;
    g.Cw = ceil_div(d.C, 32);
    g.WH = (g.Cw + 1) / 2;
    g.Fp = 64 * ceil_div(d.F, 64);
    const int Ho = (d.H + 2 * d.pad_h - d.kh) / d.stride_h + 1;
    g.Wo = (d.W + 2 * d.pad_w - d.kw) / d.stride_w + 1;
    g.HoWo = Ho * g.Wo;
    g.T = d.kh * d.kw;
    const long long M = 1ll * d.B * g.HoWo;
    const long long a_bytes = 1ll * d.B * d.H * d.W * g.Cw * 4;
    const long long nk = 1ll * g.T * g.WH;
    if (M >= (1ll << 30) || a_bytes >= (1ll << 30) || nk >= (1 << 20) || 1ll * M * d.F >= (1ll << 29)) return false;
    *pad = d.pad_h > 0 || d.pad_w > 0;
    if (*pad && g.T > 32) return false;
    g.M = static_cast<int>(M);
    g.a_bytes = static_cast<uint32_t>(a_bytes);
    g.y_bytes = static_cast<uint32_t>(M * d.F * 4);
    g.store_policy = d.F % 4 ? kStorePlain : (g.y_bytes > (96u << 20) && d.F % 32 == 0 ? kStoreStream : kStoreThrough);
    g.pix_bytes = g.Cw * 4;
    g.nk = static_cast<int>(nk);
    g.odd = g.Cw & 1;
    *lw = g.odd ? 1 : (g.WH % 4 == 0 ? 4 : (g.WH % 2 == 0 ? 2 : 1));
    g.G = g.WH / *lw;
    g.NG = g.T * g.G;
    g.d_HoWo = make_fastdiv(g.HoWo); g.d_Wo = make_fastdiv(g.Wo); g.d_WH = make_fastdiv(g.WH);
    return true;
}

bool plan_direct(const dab_conv_desc& d, DirectPlan* pl) {
    DirectGeom& g = pl->g;
    if (!describe(d, &g, &pl->pad, &pl->lw) || g.nk > kDirMaxSteps) return false;
    // The loop runs whole rounds of PF groups and reads one B entry ahead.  Of the two queue depths
    // built per load width, the one that wastes fewer groups in the last round (the deeper on a tie).
    const int deep = pl->lw == 1 ? 6 : (pl->lw == 2 ? 4 : 3), shallow = deep - 1;
    const int waste_deep = ceil_div(g.NG, deep) * deep - g.NG, waste_shallow = ceil_div(g.NG, shallow) * shallow - g.NG;
    pl->pf = waste_shallow < waste_deep ? shallow : deep;
    g.n_ent = ceil_div(g.NG, pl->pf) * pl->pf * pl->lw + 1;
    if (g.n_ent > kDirMaxSteps + 1) return false;
    // eight wavefronts (512 pixels per tile) when that still gives most compute units a tile, else four
    // (layers with fewer tiles than compute units leave some idle, and are still done in one launch)
    const int n_ntiles = ceil_div(d.F, kDirNTile);
    pl->waves = 1ll * ceil_div(g.M, 512) * n_ntiles >= kNumCU * 3 / 4 ? 8 : 4;
    g.n_mtiles = ceil_div(g.M, 64 * pl->waves);
    g.wg_per_ntile = kNumCU / n_ntiles;
    if (g.wg_per_ntile < 1) g.wg_per_ntile = 1;
    if (g.wg_per_ntile > g.n_mtiles) g.wg_per_ntile = g.n_mtiles;
    pl->grid = static_cast<unsigned>(g.wg_per_ntile * n_ntiles);
    pl->lds_bytes = static_cast<size_t>(g.n_ent) * 4096;
    return true;
}

// Layers for the block kernel.  Small ones (at most 512 blocks of 32 x 32 and too few tiles to give
// half the compute units one of the persistent kernel's): it is the fastest form.  With `large`, up
// to 8192 blocks and 400 000 block k-steps (well past where the kernel for long reductions is the faster
// one), and an estimate of the time to compare with that kernel's.
bool plan_block(const dab_conv_desc& d, BlockPlan* pl, bool large) {
    DirectGeom& g = pl->g;
    g = DirectGeom{};
    g.H = d.H; g.W = d.W; g.C = d.C; g.F = d.F; g.kh = d.kh; g.kw = d.kw;
    g.ph = d.pad_h; g.pw = d.pad_w; g.sh = d.stride_h; g.sw = d.stride_w;
    g.Cw = ceil_div(d.C, 32);
    g.WH = (g.Cw + 1) / 2;
    g.Fp = 64 * ceil_div(d.F, 64);
    const int Ho = (d.H + 2 * d.pad_h - d.kh) / d.stride_h + 1;
    g.Wo = (d.W + 2 * d.pad_w - d.kw) / d.stride_w + 1;
    g.HoWo = Ho * g.Wo;
    g.T = d.kh * d.kw;
    const long long M = 1ll * d.B * g.HoWo;
    const long long a_bytes = 1ll * d.B * d.H * d.W * g.Cw * 4;
    const long long e_bytes = 1ll * g.T * g.Cw * g.Fp * 4;
    const long long nk = 1ll * g.T * g.WH;
    if (M >= (1ll << 30) || a_bytes >= (1ll << 30) || e_bytes >= (1ll << 30) || nk >= (1 << 20)) return false;
    if (1ll * d.C * g.T >= (1ll << 24)) return false;             // |s1| must stay exact in fp32
    pl->pad = d.pad_h > 0 || d.pad_w > 0;
    if (pl->pad && g.T > 32) return false;
    g.M = static_cast<int>(M);
    g.a_bytes = static_cast<uint32_t>(a_bytes);
    g.pix_bytes = g.Cw * 4;
    g.nk = static_cast<int>(nk);
    g.d_HoWo = make_fastdiv(g.HoWo); g.d_Wo = make_fastdiv(g.Wo); g.d_WH = make_fastdiv(g.WH);
    BlockGeom& bg = pl->bg;
    bg.n_mblocks = ceil_div(g.M, 32);
    bg.d_mblocks = make_fastdiv(bg.n_mblocks);
    bg.e_bytes = static_cast<uint32_t>(e_bytes);
    bg.d_kw = make_fastdiv(d.kw);
    const long long blocks = 1ll * bg.n_mblocks * ceil_div(d.F, 32);
    const int tiles256 = ceil_div(g.M, 256) * ceil_div(d.F, kDirNTile);
    if (large ? (blocks > 8192 || blocks * nk > 400000) : (tiles256 * 2 > kNumCU || blocks > 512)) return false;
    bg.units = static_cast<int>(blocks);
    bg.per_xcd = ceil_div(bg.units, kNumXCD);
    pl->grid = static_cast<unsigned>(bg.per_xcd * kNumXCD);
    // enough wavefronts per block that each keeps a few k-steps of the reduction; the burst such that
    // two of them hold a wavefront's whole share where that is short (one round trip to memory).  From 17 k-steps four
    // wavefronts are faster than two for any number of blocks, below that while a compute unit has two of them at most (us,
    // two | four wavefronts, 300 random layers: 126 blocks x 25 steps 5.9 | 4.3, 306 x 18 6.2 | 4.4, 1568 x 18 10.9 | 10.1,
    // 480 x 9 4.9 | 4.6; 728 x 9 5.8 | 6.2, 2044 x 8 6.9 | 9.7).  Sixteen instead of eight gain 3 % at most and lose up to half.
    pl->waves = g.nk >= 32 ? 8 : (g.nk >= 17 || pl->grid <= 2 * kNumCU ? 4 : 2);
    pl->lw = (g.Cw % 2 == 0 && g.WH % 4 == 0) ? 4 : 1;
    const int share = ceil_div(g.nk, pl->waves * pl->lw) * pl->lw;
    if (pl->lw == 4) pl->depth = share <= 8 ? 4 : (share > 16 && share <= 32 ? 16 : 8);
    else pl->depth = share <= 8 ? 4 : (share > 16 && share <= 26 ? 13 : 8);
    // Time of a launch, fitted to random layers of more than 36 k-steps (rms error 9 %): workgroups per compute unit (they are
    // dealt evenly over the XCDs), and in each the k-steps of its wavefronts in whole bursts, at
    // sixteen and four bytes of a pixel per load; dearer where neighbouring taps share no cache lines.
    const double per_cu = static_cast<double>(pl->grid) / kNumCU;
    const double step_us = pl->lw == 4 ? (g.T > 1 ? 0.0081 : 0.0093) : (g.T > 1 ? 0.015 : 0.0165);
    pl->us = 1.9 + (per_cu + 1.65) * ((pl->pad ? 0.57 : 0.42) + pl->waves * ceil_div(share, pl->depth) * pl->depth * step_us);
    return true;
}

template <bool PAD, bool BITS, int WAVES, int DEPTH, int LW>
static int launch_block_as(const BlockPlan& pl, hipStream_t st, const uint32_t* A, const uint32_t* E, const float* alpha,
                           const float* beta, float* Y, int32_t* dbg_s1, const float* tau_out, uint32_t* out_bits) {
    return launch(binconv_block_kernel<PAD, BITS, WAVES, DEPTH, LW>, dim3(pl.grid), dim3(64 * WAVES), 0, st, pl.g, pl.bg, A, E, alpha,
                  beta, Y, dbg_s1, tau_out, out_bits);
}

int launch_block(const BlockPlan& pl, hipStream_t st, const uint32_t* A, const uint32_t* E, const float* alpha,
                 const float* beta, float* Y, int32_t* dbg_s1, const float* tau_out, uint32_t* out_bits) {
    const bool bits = Y == nullptr;
#define DAB_X(WAVES, DEPTH, LW)                                                                                              \
    if (pl.waves == WAVES && pl.depth == DEPTH && pl.lw == LW) {                                                             \
        if (pl.pad)                                                                                                          \
            return bits ? launch_block_as<true, true, WAVES, DEPTH, LW>(pl, st, A, E, alpha, beta, Y, dbg_s1, tau_out, out_bits)   \
                        : launch_block_as<true, false, WAVES, DEPTH, LW>(pl, st, A, E, alpha, beta, Y, dbg_s1, tau_out, out_bits); \
        return bits ? launch_block_as<false, true, WAVES, DEPTH, LW>(pl, st, A, E, alpha, beta, Y, dbg_s1, tau_out, out_bits)      \
                    : launch_block_as<false, false, WAVES, DEPTH, LW>(pl, st, A, E, alpha, beta, Y, dbg_s1, tau_out, out_bits);    \
    }
    DAB_X(8, 4, 1) DAB_X(8, 8, 1) DAB_X(8, 13, 1) DAB_X(4, 4, 1) DAB_X(2, 4, 1)
    DAB_X(8, 4, 4) DAB_X(8, 8, 4) DAB_X(8, 16, 4) DAB_X(4, 4, 4) DAB_X(2, 4, 4)
#undef DAB_X
    return DAB_ERR_UNSUPPORTED;
}

// Layers whose reduction is too long for the persistent kernel's panel and that have more blocks than
// the small-product kernel is for.
bool plan_split(const dab_conv_desc& d, SplitPlan* pl) {
    DirectGeom& g = pl->g;
    if (!describe(d, &g, &pl->pad, &pl->lw)) return false;
    const long long e_bytes = 1ll * g.T * g.Cw * g.Fp * 4;
    if (e_bytes >= (1ll << 30) || 1ll * d.C * g.T >= (1ll << 24)) return false;      // |s1| must stay exact in fp32
    SplitGeom& sg = pl->sg;
    sg.e_bytes = static_cast<uint32_t>(e_bytes);
    // byte steps of the load cursor: to the next tap of a window row, to the next row of the window
    g.step_kx = static_cast<uint32_t>((g.Cw - (g.G - 1) * 2 * pl->lw) * 4);
    g.step_ky = static_cast<uint32_t>(((d.W - (d.kw - 1)) * g.Cw - (g.G - 1) * 2 * pl->lw) * 4);
    sg.d_G = make_fastdiv(g.G);
    sg.d_kw = make_fastdiv(d.kw);
    // Shares of the reduction per pixel block: the number that minimises rounds of workgroups times the
    // time of one: 0.4 us a k-step of two wavefronts per SIMD, set-up and epilogue 4.5, the exchange 0.5 (2.5 in fp32).
    // (Over 3587 random layers for which this is the kernel, 0.4 % slower than the best number of shares.)
    const bool narrow = 1ll * d.C * g.T < (1 << 15);
    const int n_ntiles = ceil_div(d.F, kDirNTile);
    double best = 0.0;
    for (int lk = 0; lk <= 3; ++lk) {
        const int per = ceil_div(g.NG, 1 << lk);
        const long long units = 1ll * ceil_div(g.M, 64 * (kSplitWaves >> lk)) * n_ntiles;
        const double us = static_cast<double>((units + kNumCU - 1) / kNumCU) * (per * pl->lw * 0.4 + 4.5 + (lk ? (narrow ? 0.5 : 2.5) : 0.0));
        if (lk == 0 || us < best) {
            best = us;
            sg.log_ks = lk;
            sg.groups_per_share = per;
        }
    }
    sg.n_mtiles = ceil_div(g.M, 64 * (kSplitWaves >> sg.log_ks));
    const long long units = 1ll * sg.n_mtiles * n_ntiles;
    if (units >= (1ll << 30)) return false;
    // Time of a launch, to compare with the other kernels' (fitted to 1900 random layers with the shares chosen above,
    // rms error 7 %): per round of workgroups the k-steps, which come in whole and then half rounds of eight, by the
    // words per load; dearer with padding, with fewer taps that share their cache lines and with more compute units at
    // work.  What the fp32 stores add is more where rows are no whole number of 16-byte stores.
    const int steps = sg.groups_per_share * pl->lw;
    pl->steps_run = steps % 8 == 0 ? steps : steps / 8 * 8 + (steps % 8 <= 4 ? 4 : 8);
    pl->rounds = static_cast<int>((units + kNumCU - 1) / kNumCU);
    pl->filled = static_cast<double>(units) / (1.0 * pl->rounds * kNumCU);
    const double step_us = (pl->lw == 1 ? 0.334 : (pl->lw == 2 ? 0.23 : 0.189)) + (pl->pad ? 0.078 : 0.0) + 0.088 / g.T + 0.112 * pl->filled;
    pl->us_bits = 2.75 + pl->rounds * (3.62 + (sg.log_ks ? (narrow ? -0.85 : 1.75) : 0.0) + pl->steps_run * step_us);
    pl->us = pl->us_bits + (d.F % 4 ? 0.14 : 0.057) * 4.0e-6 * g.M * d.F;
    sg.units = static_cast<int>(units);
    sg.per_xcd = ceil_div(sg.units, kNumXCD);
    sg.d_mtiles = make_fastdiv(sg.n_mtiles);
    pl->grid = static_cast<unsigned>(sg.per_xcd * kNumXCD);
    pl->lds_bytes = sg.log_ks ? kSplitLds : 0;
    sg.narrow = sg.log_ks && narrow ? 1 : 0;
    return true;
}

template <int LW>
static int launch_split_as(const SplitPlan& pl, hipStream_t st, const uint32_t* A, const uint32_t* E, const float* alpha,
                           const float* beta, float* Y, int32_t* dbg_s1, const float* tau_out, uint32_t* out_bits) {
    const bool bits = Y == nullptr;
    auto go = [&](auto kernel) {
        return launch(kernel, dim3(pl.grid), dim3(64 * kSplitWaves), pl.lds_bytes, st, pl.g, pl.sg, A, E, alpha, beta, Y, dbg_s1, tau_out,
                      out_bits);
    };
    if (pl.pad) return bits ? go(binconv_split_kernel<LW, true, true>) : go(binconv_split_kernel<LW, true, false>);
    return bits ? go(binconv_split_kernel<LW, false, true>) : go(binconv_split_kernel<LW, false, false>);
}
int launch_split(const SplitPlan& pl, hipStream_t st, const uint32_t* A, const uint32_t* E, const float* alpha, const float* beta,
                 float* Y, int32_t* dbg_s1, const float* tau_out, uint32_t* out_bits) {
    if (pl.lw == 4) return launch_split_as<4>(pl, st, A, E, alpha, beta, Y, dbg_s1, tau_out, out_bits);
    if (pl.lw == 2) return launch_split_as<2>(pl, st, A, E, alpha, beta, Y, dbg_s1, tau_out, out_bits);
    return launch_split_as<1>(pl, st, A, E, alpha, beta, Y, dbg_s1, tau_out, out_bits);
}

template <int LW, int PF, bool PAD, bool BITS>
static int launch_direct_as(const DirectPlan& pl, hipStream_t st, const uint32_t* A, const uint32_t* E, const float* alpha,
                            const float* beta, float* Y, int32_t* dbg_s1, const float* tau_out, uint32_t* out_bits) {
    return launch(binconv_direct_kernel<LW, PF, PAD, BITS>, dim3(pl.grid), dim3(64 * pl.waves), pl.lds_bytes, st, E, A, alpha, beta,
                  tau_out, make_fastdiv(pl.g.wg_per_ntile), pl.g, Y, dbg_s1, out_bits);
}

// The instantiations in use: (words per load, groups per round) x padding x (fp32 | bits).
#define DAB_DIRECT_VARIANTS(X) X(1, 5) X(1, 6) X(2, 3) X(2, 4) X(4, 2) X(4, 3)

int launch_direct(const DirectPlan& pl, hipStream_t st, const uint32_t* A, const uint32_t* E, const float* alpha,
                  const float* beta, float* Y, int32_t* dbg_s1, const float* tau_out, uint32_t* out_bits) {
    const bool bits = Y == nullptr;
#define DAB_X(LW, PF)                                                                                              \
    if (pl.lw == LW && pl.pf == PF) {                                                                              \
        if (pl.pad)                                                                                                \
            return bits ? launch_direct_as<LW, PF, true, true>(pl, st, A, E, alpha, beta, Y, dbg_s1, tau_out, out_bits) \
                        : launch_direct_as<LW, PF, true, false>(pl, st, A, E, alpha, beta, Y, dbg_s1, tau_out, out_bits); \
        return bits ? launch_direct_as<LW, PF, false, true>(pl, st, A, E, alpha, beta, Y, dbg_s1, tau_out, out_bits) \
                    : launch_direct_as<LW, PF, false, false>(pl, st, A, E, alpha, beta, Y, dbg_s1, tau_out, out_bits); \
    }
    DAB_DIRECT_VARIANTS(DAB_X)
#undef DAB_X
    return DAB_ERR_UNSUPPORTED;
}

// One-time set-up on the current device: the panel takes up to (kDirMaxSteps + 1) * 4 KB of dynamic LDS.
template <int LW, int PF, bool PAD, bool BITS>
static int raise_direct_limit() {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&binconv_direct_kernel<LW, PF, PAD, BITS>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (kDirMaxSteps + 1) * 4096);
    return e == hipSuccess ? static_cast<int>(DAB_OK) : hip_failed(e);
}
template <int LW>
static int raise_split_limit() {
    for (const void* k : {reinterpret_cast<const void*>(&binconv_split_kernel<LW, false, false>),
                          reinterpret_cast<const void*>(&binconv_split_kernel<LW, false, true>),
                          reinterpret_cast<const void*>(&binconv_split_kernel<LW, true, false>),
                          reinterpret_cast<const void*>(&binconv_split_kernel<LW, true, true>)})
        if (const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, kSplitLds); e != hipSuccess)
            return hip_failed(e);
    return DAB_OK;
}
int init_direct() {
    if (int rc = raise_split_limit<1>()) return rc;
    if (int rc = raise_split_limit<2>()) return rc;
    if (int rc = raise_split_limit<4>()) return rc;
#define DAB_X(LW, PF)                                                   \
    if (int rc = raise_direct_limit<LW, PF, false, false>()) return rc; \
    if (int rc = raise_direct_limit<LW, PF, false, true>()) return rc;  \
    if (int rc = raise_direct_limit<LW, PF, true, false>()) return rc;  \
    if (int rc = raise_direct_limit<LW, PF, true, true>()) return rc;
    DAB_DIRECT_VARIANTS(DAB_X)
#undef DAB_X
    return DAB_OK;
}

}  // namespace dab
