// Weight-side steps of a training iteration (Algorithm 2): MeanCenter + Clamp of the real weights,
// W~ = alpha e + beta (1 - e) from the split descriptor, and the element-wise gradient factor of
// Theorem 4.  All three stream the weights and are bound by memory, the short rows by the latency of
// one trip to it.  Where a row's sums are needed first, one workgroup owns the row and keeps it in
// registers; every call may run in place.
#include "dab_internal.h"

#include "estimate_rows.h"

namespace dab {

constexpr int kTrainThreads = 256;

// Sum of one double per thread over the workgroup, returned to every thread (s_part: one slot per wavefront).
__device__ __forceinline__ double block_sum(double v, double* s_part) {
    for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
    const int wave = threadIdx.x >> 6;
    __syncthreads();                                       // the previous use of s_part is over
    if ((threadIdx.x & 63) == 0) s_part[wave] = v;
    __syncthreads();
    double t = 0.0;
    for (int w = 0; w < static_cast<int>(blockDim.x >> 6); ++w) t += s_part[w];
    return t;
}

__device__ __forceinline__ float center_clamp(float w, double mean, float lo, float hi) {
    const double c = static_cast<double>(w) - mean;
    return static_cast<float>(fmin(fmax(c, static_cast<double>(lo)), static_cast<double>(hi)));
}

// ---------------------------------------------------------------- rows held in registers
// Rows of up to 16384 weights are read once: N elements per thread, every load in flight before the first sum, and
// the sums of a row are exchanged once (data-parallel-primitive moves inside a wavefront, one LDS barrier between them).
// VEC 4: 16-byte pieces (rows of a multiple of four weights, 16-byte aligned); VEC 1: single weights, any row.
// (Three sums by shuffles, two barriers each, and the upstream gradient fetched behind them: the gradient factor of config 3's
// layers took 6.2, 6.2, 7.1, 7.1, 24.8 and 5.7 us; now 4.4, 4.3, 4.9, 4.9, 18.8 and 3.7.)
template <int THREADS, int N, int VEC>
struct Row {
    float v[N];
    static __device__ __forceinline__ int index(int j) {
        const int tid = threadIdx.x;
        return VEC == 4 ? 4 * (tid + j / 4 * THREADS) + j % 4 : tid + j * THREADS;
    }
    // (positions past the end hold `past`)
    __device__ __forceinline__ void load(const float* __restrict__ row, int n, float past) {
        if constexpr (VEC == 4) {
#pragma unroll
            for (int j = 0; j < N; j += 4) {
                const int i = index(j);
                const float4 q = i < n ? *reinterpret_cast<const float4*>(row + i) : make_float4(past, past, past, past);
                v[j] = q.x; v[j + 1] = q.y; v[j + 2] = q.z; v[j + 3] = q.w;
            }
        } else {
            const RowWindow win = row_window(row, n);
#pragma unroll
            for (int j = 0; j < N; ++j) {
                if (j * THREADS >= n) v[j] = past;
                else v[j] = load_from(win, index(j) * 4, 0);
                if ((j + 1) * THREADS > n && index(j) >= n) v[j] = past;
            }
        }
    }
    __device__ __forceinline__ void store(float* row, int n) const {
        if constexpr (VEC == 4) {
#pragma unroll
            for (int j = 0; j < N; j += 4)
                if (index(j) < n) *reinterpret_cast<float4*>(row + index(j)) = make_float4(v[j], v[j + 1], v[j + 2], v[j + 3]);
        } else {
#pragma unroll
            for (int j = 0; j < N; ++j)
                if (index(j) < n) row[index(j)] = v[j];
        }
    }
};

// Sums over the workgroup, returned to every thread.  (Once per kernel: the array is not used again.)
template <int THREADS, int M>
__device__ __forceinline__ void row_sums(double (&s)[M]) {
    constexpr int NW = THREADS / 64;
    __shared__ double part[M][NW];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int m = 0; m < M; ++m) s[m] = wave_inclusive_scan_f64(s[m]);
    if (NW == 1) {
#pragma unroll
        for (int m = 0; m < M; ++m) s[m] = lane_of(s[m], 63);
        return;
    }
    if (lane == 63) {
#pragma unroll
        for (int m = 0; m < M; ++m) part[m][wave] = s[m];
    }
    lds_barrier();
#pragma unroll
    for (int m = 0; m < M; ++m) {
        double t = part[m][0];
#pragma unroll
        for (int w = 1; w < NW; ++w) t += part[m][w];
        s[m] = t;
    }
}

template <int THREADS, int N, int VEC>
__global__ __launch_bounds__(THREADS) void center_row_kernel(const float* W, int n, float lo, float hi, float* out) {
    DAB_RESERVE_VGPRS();
    const size_t at = static_cast<size_t>(blockIdx.x) * n;
    Row<THREADS, N, VEC> x;
    x.load(W + at, n, 0.0f);
    double s[1] = {0.0};
#pragma unroll
    for (int j = 0; j < N; j += 2) s[0] += static_cast<double>(x.v[j]) + static_cast<double>(x.v[j + 1]);
    row_sums<THREADS>(s);
    const double mean = s[0] / static_cast<double>(n);
#pragma unroll
    for (int j = 0; j < N; ++j) x.v[j] = center_clamp(x.v[j], mean, lo, hi);
    x.store(out + at, n);
}

// Membership of element i in the alpha group, from the estimator's split descriptor.
__device__ __forceinline__ bool in_alpha_group(float w, int i, float tv, int ti, bool upper) {
    const bool lower = w < tv || (w == tv && i <= ti);
    return lower != upper;
}

// Theorem 4, element-wise: with e the mask, T_k = W o e and R = W - T_k,
//   G~_i = e_i / K + (||T_k||_1 / K) T_k^i [|W_i| <= 1] + (1 - e_i) / (n - K) + (||R||_1 / (n - K)) R^i [|W_i| <= 1],
// optionally times the upstream gradient.  K and the two l1 norms, in double, come first; an empty
// group (a descriptor with K = 0 or K = n, which the estimator never returns) contributes nothing.
struct GradientTerms {
    double inv_a, inv_b, sa, sb;
};
__device__ __forceinline__ GradientTerms gradient_terms(double la, double lb, double K, int n) {
    const double nK = static_cast<double>(n) - K;
    GradientTerms t;
    t.inv_a = K > 0.0 ? 1.0 / K : 0.0;
    t.inv_b = nK > 0.0 ? 1.0 / nK : 0.0;
    t.sa = la * t.inv_a;
    t.sb = lb * t.inv_b;
    return t;
}
__device__ __forceinline__ double gradient_of(float w, bool in, const GradientTerms& t) {
    const double ste = fabsf(w) <= 1.0f ? static_cast<double>(w) : 0.0;
    return in ? t.inv_a + t.sa * ste : t.inv_b + t.sb * ste;
}

template <int THREADS, int N, int VEC>
__global__ __launch_bounds__(THREADS) void gradient_row_kernel(const float* W, int n, const float* __restrict__ thr_val,
                                                               const int32_t* __restrict__ thr_idx,
                                                               const uint8_t* __restrict__ alpha_is_upper,
                                                               const float* upstream, float* out) {
    DAB_RESERVE_VGPRS();
    const int f = blockIdx.x;
    const size_t at = static_cast<size_t>(f) * n;
    Row<THREADS, N, VEC> x, u;
    x.load(W + at, n, 0.0f);
    if (upstream) u.load(upstream + at, n, 0.0f);
    const float tv = thr_val[f];
    const int ti = thr_idx[f];
    const bool upper = alpha_is_upper[f] != 0;
    double s[3] = {0.0, 0.0, 0.0};
    uint32_t member = 0, count = 0;                        // bit j: element j is in the alpha group
#pragma unroll
    for (int j = 0; j < N; ++j) {
        const int i = x.index(j);
        const bool in = (i < n) & in_alpha_group(x.v[j], i, tv, ti, upper);
        const float a = fabsf(x.v[j]);                                 // (zero past the end)
        s[0] += static_cast<double>(in ? a : 0.0f);
        s[1] += static_cast<double>(in ? 0.0f : a);                    // (no difference: an infinite weight stays with its group)
        member |= in ? 1u << j : 0u;
    }
    count = static_cast<uint32_t>(__popc(member));
    s[2] = static_cast<double>(count);                     // exact: a count below 2^31
    row_sums<THREADS>(s);
    const GradientTerms t = gradient_terms(s[0], s[1], s[2], n);
#pragma unroll
    for (int j = 0; j < N; ++j) {
        double g = gradient_of(x.v[j], (member >> j) & 1u, t);
        if (upstream) g *= static_cast<double>(u.v[j]);
        x.v[j] = static_cast<float>(g);
    }
    x.store(out + at, n);
}

// ---------------------------------------------------------------- any row
// MeanCenter over the n = C*T weights of a filter, then Clamp.
__global__ __launch_bounds__(kTrainThreads) void center_filter_kernel(const float* W, int n, float lo, float hi,
                                                                      float* out) {
    DAB_RESERVE_VGPRS();
    __shared__ double s_part[16];
    const float* row = W + static_cast<size_t>(blockIdx.x) * n;
    float* orow = out + static_cast<size_t>(blockIdx.x) * n;
    double s = 0.0;
    for (int i = threadIdx.x; i < n; i += kTrainThreads) s += static_cast<double>(row[i]);
    const double mean = block_sum(s, s_part) / static_cast<double>(n);
    for (int i = threadIdx.x; i < n; i += kTrainThreads) orow[i] = center_clamp(row[i], mean, lo, hi);
}

// MeanCenter over the C input channels of every (filter, tap), then Clamp.  A workgroup takes one
// filter; its threads are laid out as Tt taps x CL channel lanes (Tt = min(T, 256)), so loads run
// along the taps, which are contiguous in memory.
__global__ __launch_bounds__(kTrainThreads) void center_channel_kernel(const float* W, int C, int T, float lo,
                                                                       float hi, float* out) {
    DAB_RESERVE_VGPRS();
    __shared__ double s_sum[kTrainThreads];
    const float* row = W + static_cast<size_t>(blockIdx.x) * C * T;
    float* orow = out + static_cast<size_t>(blockIdx.x) * C * T;
    const int Tt = min(T, kTrainThreads);
    const int CL = kTrainThreads / Tt;
    const int tl = threadIdx.x % Tt, cl = threadIdx.x / Tt;
    const bool active = cl < CL;
    for (int t0 = 0; t0 < T; t0 += Tt) {
        const int t = t0 + tl;
        double s = 0.0;
        if (active && t < T)
            for (int c = cl; c < C; c += CL) s += static_cast<double>(row[static_cast<size_t>(c) * T + t]);
        __syncthreads();                                   // the previous tile's sums have been read
        s_sum[threadIdx.x] = s;
        __syncthreads();
        double tot = 0.0;
        for (int k = 0; k < CL; ++k) tot += s_sum[k * Tt + tl];
        const double mean = tot / static_cast<double>(C);
        if (active && t < T)
            for (int c = cl; c < C; c += CL) {
                const size_t o = static_cast<size_t>(c) * T + t;
                orow[o] = center_clamp(row[o], mean, lo, hi);
            }
    }
}

// W~ of Algorithm 2: alpha on the mask, beta off it.  Nothing of a row is needed but its descriptor: a row is cut into
// chunks of four pieces per thread, blockIdx.y + y0 says which.
constexpr int kTildePieces = 4;
template <int VEC>
__global__ __launch_bounds__(kTrainThreads) void binarized_weights_kernel(
    const float* W, int n, const float* __restrict__ alpha, const float* __restrict__ beta, const float* __restrict__ thr_val,
    const int32_t* __restrict__ thr_idx, const uint8_t* __restrict__ alpha_is_upper, float* out, int y0) {
    constexpr int kChunk = kTildePieces * kTrainThreads * VEC;
    const int f = blockIdx.x;
    const int c0 = (static_cast<int>(blockIdx.y) + y0) * kChunk, left = n - c0;     // (c0 < n < 2^31)
    const float* src = W + static_cast<size_t>(f) * n + c0;
    float* dst = out + static_cast<size_t>(f) * n + c0;
    float w[kTildePieces][VEC];
#pragma unroll
    for (int k = 0; k < kTildePieces; ++k) {
        const int i = (threadIdx.x + k * kTrainThreads) * VEC;
        if (i < left) {
            if constexpr (VEC == 4) {
                const float4 q = *reinterpret_cast<const float4*>(src + i);
                w[k][0] = q.x; w[k][1] = q.y; w[k][2] = q.z; w[k][3] = q.w;
            } else {
                w[k][0] = src[i];
            }
        }
    }
    const float al = alpha[f], be = beta[f], tv = thr_val[f];
    const int ti = thr_idx[f];
    const bool upper = alpha_is_upper[f] != 0;
#pragma unroll
    for (int k = 0; k < kTildePieces; ++k) {
        const int i = (threadIdx.x + k * kTrainThreads) * VEC;
        if (i < left) {
            float r[VEC];
#pragma unroll
            for (int c = 0; c < VEC; ++c) r[c] = in_alpha_group(w[k][c], c0 + i + c, tv, ti, upper) ? al : be;
            if constexpr (VEC == 4) *reinterpret_cast<float4*>(dst + i) = make_float4(r[0], r[1], r[2], r[3]);
            else dst[i] = r[0];
        }
    }
}

// The gradient factor of a row that does not fit in registers: read twice.
__global__ __launch_bounds__(kTrainThreads) void weight_gradient_kernel(
    const float* __restrict__ W, int n, const float* __restrict__ thr_val, const int32_t* __restrict__ thr_idx,
    const uint8_t* __restrict__ alpha_is_upper, const float* __restrict__ upstream, float* __restrict__ out) {
    DAB_RESERVE_VGPRS();
    __shared__ double s_part[16];
    const int f = blockIdx.x;
    const float* row = W + static_cast<size_t>(f) * n;
    const float tv = thr_val[f];
    const int ti = thr_idx[f];
    const bool upper = alpha_is_upper[f] != 0;
    double la = 0.0, lb = 0.0, cnt = 0.0;
    for (int i = threadIdx.x; i < n; i += kTrainThreads) {
        const float w = row[i];
        const double a = fabs(static_cast<double>(w));
        if (in_alpha_group(w, i, tv, ti, upper)) {
            la += a;
            cnt += 1.0;
        } else {
            lb += a;
        }
    }
    la = block_sum(la, s_part);
    lb = block_sum(lb, s_part);
    const GradientTerms t = gradient_terms(la, lb, block_sum(cnt, s_part), n);
    const float* up = upstream ? upstream + static_cast<size_t>(f) * n : nullptr;
    float* orow = out + static_cast<size_t>(f) * n;
    for (int i = threadIdx.x; i < n; i += kTrainThreads) {
        const float w = row[i];
        double g = gradient_of(w, in_alpha_group(w, i, tv, ti, upper), t);
        if (up) g *= static_cast<double>(up[i]);
        orow[i] = static_cast<float>(g);
    }
}

// ---------------------------------------------------------------- host side
inline bool whole_pieces(const void* a, const void* b, const void* c, int n) {
    return n % 4 == 0 && !misaligned(a, 16) && !misaligned(b, 16) && !(c && misaligned(c, 16));
}
constexpr int kRowMaxN = 1024 * 16;

// DO(threads, elements per thread) for the smallest workgroup that holds a row of n <= kRowMaxN weights.  (Eight
// wavefronts for the long rows: two or three rows share a compute unit; with sixteen it was one at a time.)
#define DAB_ROW_CLASSES(DO) \
    if (n <= 512) DO(128, 4); \
    if (n <= 1024) DO(256, 4); \
    if (n <= 2048) DO(256, 8); \
    if (n <= 4096) DO(512, 8); \
    if (n <= 8192) DO(512, 16); \
    if (n <= 14336) DO(512, 28); \
    DO(1024, 16)

static int center_rows(const float* W, int F, int n, float lo, float hi, float* out, hipStream_t st) {
#define DAB_CENTER(T, N) \
    return vec ? launch(center_row_kernel<T, N, 4>, dim3(F), dim3(T), 0, st, W, n, lo, hi, out) \
               : launch(center_row_kernel<T, N, 1>, dim3(F), dim3(T), 0, st, W, n, lo, hi, out)
    const bool vec = whole_pieces(W, out, nullptr, n);
    DAB_ROW_CLASSES(DAB_CENTER);
#undef DAB_CENTER
}

static int gradient_rows(const float* W, int F, int n, const float* thr_val, const int32_t* thr_idx, const uint8_t* aiu,
                         const float* upstream, float* out, hipStream_t st) {
#define DAB_GRADIENT(T, N) \
    return vec ? launch(gradient_row_kernel<T, N, 4>, dim3(F), dim3(T), 0, st, W, n, thr_val, thr_idx, aiu, upstream, out) \
               : launch(gradient_row_kernel<T, N, 1>, dim3(F), dim3(T), 0, st, W, n, thr_val, thr_idx, aiu, upstream, out)
    const bool vec = whole_pieces(W, out, upstream, n);
    DAB_ROW_CLASSES(DAB_GRADIENT);
#undef DAB_GRADIENT
}
#undef DAB_ROW_CLASSES

}  // namespace dab

extern "C" {

int dab_mean_center_clamp(const float* W, int32_t F, int32_t C, int32_t T, int32_t axis, float lo, float hi, float* W_out,
                          void* stream) {
    using namespace dab;
    if (!W || !W_out) return DAB_ERR_NULL;
    if (F < 1 || C < 1 || T < 1 || 1ll * C * T > 0x7fffffffll || !(lo <= hi)) return DAB_ERR_SHAPE;
    if (axis != DAB_CENTER_FILTER && axis != DAB_CENTER_CHANNEL) return DAB_ERR_UNSUPPORTED;
    if (misaligned(W, 4) || misaligned(W_out, 4)) return DAB_ERR_ALIGN;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (axis == DAB_CENTER_FILTER && C * T <= kRowMaxN) return center_rows(W, F, C * T, lo, hi, W_out, st);
    if (axis == DAB_CENTER_FILTER)
        return launch(center_filter_kernel, dim3(F), dim3(kTrainThreads), 0, st, W, C * T, lo, hi, W_out);
    else
        return launch(center_channel_kernel, dim3(F), dim3(kTrainThreads), 0, st, W, C, T, lo, hi, W_out);
}

int dab_binarized_weights(const float* W, int32_t F, int32_t n, const float* alpha, const float* beta, const float* thr_val,
                          const int32_t* thr_idx, const uint8_t* alpha_is_upper, float* W_tilde, void* stream) {
    using namespace dab;
    if (!W || !alpha || !beta || !thr_val || !thr_idx || !alpha_is_upper || !W_tilde) return DAB_ERR_NULL;
    if (F < 1 || n < 1) return DAB_ERR_SHAPE;
    if (misaligned(W, 4) || misaligned(alpha, 4) || misaligned(beta, 4) || misaligned(thr_val, 4) ||
        misaligned(thr_idx, 4) || misaligned(W_tilde, 4))
        return DAB_ERR_ALIGN;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const bool vec = whole_pieces(W, W_tilde, nullptr, n);
    const int chunks = (n - 1) / (kTildePieces * kTrainThreads * (vec ? 4 : 1)) + 1;
    for (int y0 = 0; y0 < chunks; y0 += 32768) {              // (a launch's grid.y ends at 65535)
        const dim3 grid(F, chunks - y0 < 32768 ? chunks - y0 : 32768);
        const int rc = vec ? launch(binarized_weights_kernel<4>, grid, dim3(kTrainThreads), 0, st, W, n, alpha, beta, thr_val, thr_idx,
                                    alpha_is_upper, W_tilde, y0)
                           : launch(binarized_weights_kernel<1>, grid, dim3(kTrainThreads), 0, st, W, n, alpha, beta, thr_val, thr_idx,
                                    alpha_is_upper, W_tilde, y0);
        if (rc) return rc;
    }
    return DAB_OK;
}

int dab_weight_gradient(const float* W, int32_t F, int32_t n, const float* thr_val, const int32_t* thr_idx,
                        const uint8_t* alpha_is_upper, const float* upstream, float* G_out, void* stream) {
    using namespace dab;
    if (!W || !thr_val || !thr_idx || !alpha_is_upper || !G_out) return DAB_ERR_NULL;
    if (F < 1 || n < 2) return DAB_ERR_SHAPE;
    if (misaligned(W, 4) || misaligned(thr_val, 4) || misaligned(thr_idx, 4) || misaligned(G_out, 4) ||
        (upstream && misaligned(upstream, 4)))
        return DAB_ERR_ALIGN;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (n <= kRowMaxN) return gradient_rows(W, F, n, thr_val, thr_idx, alpha_is_upper, upstream, G_out, st);
    return launch(weight_gradient_kernel, dim3(F), dim3(kTrainThreads), 0, st, W, n, thr_val, thr_idx, alpha_is_upper, upstream,
                  G_out);
}

}  // extern "C"
