// Scale machinery of sections 3.1 and 4.1: the two scale-gradient sums of one tensor
// (STE-based and MSE-based) and percentile calibration of an activation step.  All are
// streaming reductions over the tensor, bound by HBM bandwidth (one read of x per pass).
#include "mkq_internal.h"

namespace mkq {

__device__ __forceinline__ double wave_sum_f64(double v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

constexpr int CAL_THREADS = 1024;
// Threads per workgroup of the gradient sums: a tensor that 64 small workgroups cover takes small ones, which spread it over
// more CUs (128 x 768 binary32 7.3 -> 6.7 us); beyond that the sums of many workgroups would queue in their atomic
// additions (440 x 768: 7.4 us with 42 large ones, 7.9 with 165 small ones).
static inline int gradient_threads(int64_t groups) { return groups <= 64 * 256 ? 256 : CAL_THREADS; }

__global__ void zero_words_kernel(uint32_t *p, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0u;
}

// Address of group w (8 elements) of an [M, K] tensor with rows of ldx elements.  CONTIG: ldx == K, no split into
// row and column (a 64-bit division for every eight elements: a third of the vector operations of these kernels).
template <typename T, bool CONTIG>
__device__ __forceinline__ const T *group_at(const T *x, int64_t w, int64_t groups_per_row, int64_t ldx)
{
    if (CONTIG) return x + w * 8;
    const int64_t m = w / groups_per_row;
    return x + m * ldx + (w - m * groups_per_row) * 8;
}

// Eight values of a tensor as they are fetched
struct Floats8 {
    float v[8];
    template <typename T>
    __device__ __forceinline__ void load(const T *p) { load8<T>(p, v); }
};

// Calls f with the eight values (a Group) of every group that this thread owns.  AHEAD groups are fetched before the first of
// them is used, so that a thread has as many loads in flight.  A batch that reaches past the end fetches its first group
// again, which is cheaper than a branch per load (25.7 instead of 27.0 us for a counting pass over 16384 x 4096 binary16
// values) -- unless rows have gaps: the address of a group is a 64-bit division then, so whole batches go first, without
// checks, and the last one skips what does not exist (percentile of 128 rows of 768 + 64 binary32 values 21.2 -> 18.3 us).
// WINDOW (contiguous tensors): the groups of a batch are neighbours, so that all workgroups together read one window of memory
// that moves on, instead of AHEAD of them megabytes apart; only batches that the whole grid fills, so that the rest is spread
// as evenly as before.
template <class Group, typename T, bool CONTIG, int AHEAD, bool WINDOW = false, class F>
__device__ __forceinline__ void for_each_group(const T *__restrict__ x, int64_t total, int64_t groups_per_row, int64_t ldx,
                                               F &&f)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    int64_t w = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if constexpr (WINDOW && CONTIG) {
        const int64_t span = AHEAD * stride, whole = total < span ? 0 : (int64_t)((uint32_t)total / (uint32_t)span) * span;
        const T *at = x + ((int64_t)blockIdx.x * blockDim.x * AHEAD + threadIdx.x) * 8;
        for (int64_t done = 0; done < whole; done += span, at += span * 8) {
            Group v[AHEAD];
#pragma unroll
            for (int a = 0; a < AHEAD; ++a) v[a].load(at + a * (int64_t)blockDim.x * 8);
#pragma unroll
            for (int a = 0; a < AHEAD; ++a) f(v[a]);
        }
        w += whole;
    }
    if constexpr (!CONTIG) {
        for (; w + (AHEAD - 1) * stride < total; w += AHEAD * stride) {
            Group v[AHEAD];
#pragma unroll
            for (int a = 0; a < AHEAD; ++a) v[a].load(group_at<T, CONTIG>(x, w + a * stride, groups_per_row, ldx));
#pragma unroll
            for (int a = 0; a < AHEAD; ++a) f(v[a]);
        }
    }
    for (; w < total; w += AHEAD * stride) {
        Group v[AHEAD];
#pragma unroll
        for (int a = 0; a < AHEAD; ++a) {
            const int64_t wa = w + a * stride;
            if (!CONTIG && wa >= total) break;
            v[a].load(group_at<T, CONTIG>(x, wa < total ? wa : w, groups_per_row, ldx));
        }
#pragma unroll
        for (int a = 0; a < AHEAD; ++a)
            if (w + a * stride < total) f(v[a]);
    }
}

// The largest of eight values, NaN if any of them is: two values per instruction (v_maximum3_f32)
__device__ __forceinline__ float maximum8(const float (&x)[8])
{
    float m = x[0];
#pragma unroll
    for (int e = 1; e < 7; e += 2) m = __builtin_elementwise_maximum(__builtin_elementwise_maximum(m, x[e]), x[e + 1]);
    return __builtin_elementwise_maximum(m, x[7]);
}

// The codes of Eq. 1 for eight values, as floats, without a division per value (QuantStep): one branch to the
// division if any of the eight lies within the margin of a rounding boundary or is NaN or infinite.
template <int BITS>
__device__ __forceinline__ void codes8(const float (&x)[8], const QuantStep &q, float (&c)[8])
{
    constexpr float lo = (BITS == 4) ? (float)QMIN : -128.0f, hi = (BITS == 4) ? (float)QMAX : 127.0f;
    float far[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const float v = x[e] * q.rs, r = __builtin_rintf(v);
        // beyond the clamp range the product's error may exceed the margin, and either quotient clamps alike
        far[e] = fabsf(v - r);
        c[e] = __builtin_amdgcn_fmed3f(r, lo, hi);
    }
    // (a comparison per value takes as many scalar operations besides: gradients of 16384 x 4096 binary16 values 35.3 us, with one
    // comparison of their maximum 29.5.  The same in the epilogues of the linears was no gain: FFN-up with
    // GELU and codes out 46.3 -> 47.2.)
    if (__builtin_expect(!(maximum8(far) <= q.thr), 0)) {
#pragma unroll
        for (int e = 0; e < 8; ++e) c[e] = (float)((BITS == 4) ? quantize_code(x[e], q.s) : quantize_code8(x[e], q.s));
    }
}

// g[0] += sum_i ( round(x_i/s) - x_i/s ),  g[1] += 2 sum_i ( Q[x_i] - x_i ) round(x_i/s)
// with round() = the code of Eq. 1 (clamp included), decided in binary32 like the quantizer;
// the terms and sums are binary64.
// A binary64 atomic addition is a compare-and-swap loop, and workgroups that meet in it are served one after the
// other: with 2048 workgroups that was most of the kernel's time.  Few, large workgroups therefore (at most one per
// CU).
template <typename T, int BITS, bool CONTIG>
__global__ __launch_bounds__(CAL_THREADS) void scale_gradients_kernel(const T *__restrict__ x, int64_t M, int64_t K,
                                                              int64_t ldx, float s, double *__restrict__ g)
{
    __shared__ double part[2][CAL_THREADS / 64];
    const double sd = (double)s, inv = 1.0 / sd;
    const QuantStep qs = quant_step<BITS>(s);
    const int64_t groups_per_row = K / 8;
    const int64_t total = M * groups_per_row;
    // sum(c - x/s) = sum c - (sum x)/s and sum((s c - x) c) = s sum c^2 - sum(x c): the sums of c and c^2 of eight
    // values are whole numbers that binary32 holds exactly, so binary64 is left with two sums per element, not three
    double sc = 0.0, scc = 0.0, sx = 0.0, sxc = 0.0;
    for_each_group<Floats8, T, CONTIG, 4>(x, total, groups_per_row, ldx, [&](const Floats8 &g8) {
        const float(&v)[8] = g8.v;
        float c[8], c1 = 0.0f, c2 = 0.0f;
        codes8<BITS>(v, qs, c);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            c1 += c[e];
            c2 = __builtin_fmaf(c[e], c[e], c2);
            const double xd = (double)v[e];
            sx += xd;
            sxc = __builtin_fma(xd, (double)c[e], sxc);
        }
        sc += (double)c1;
        scc += (double)c2;
    });
    double ste = __builtin_fma(-sx, inv, sc), mse = __builtin_fma(sd, scc, -sxc);
    ste = wave_sum_f64(ste);
    mse = wave_sum_f64(mse);
    if ((threadIdx.x & 63) == 0) {
        part[0][threadIdx.x >> 6] = ste;
        part[1][threadIdx.x >> 6] = mse;
    }
    __syncthreads();
    if (threadIdx.x < 2) {  // one lane per sum: the two loops run side by side
        double sum = 0.0;
        for (int i = 0; i < (int)blockDim.x / 64; ++i) sum += part[threadIdx.x][i];
        atomicAdd(g + threadIdx.x, threadIdx.x ? 2.0 * sum : sum);
    }
}

// ---- percentile calibration: exact k-th largest of |x| by radix selection -------------
// |x| >= 0, so its bit pattern orders like an unsigned integer: the 31 bits of a binary32 value, the 15 of a binary16 one
// (with six zeros behind them).  Passes over the tensor count, among the elements whose higher bits equal the prefix
// chosen so far, the next 11, 10 and 10 bits; after each the last workgroup to finish walks the counts from the
// top and fixes the digit in which the k-th largest falls.  Two passes for binary16, three for binary32.
// In a graph, us, binary16 as binary32 patterns (three passes, the last of which finds nothing but zeros in its digit)
// -> this: 64 x 768 17.5 -> 13.6, 4096 x 768 32.6 -> 25.1, 16384 x 4096 84.0 -> 55.7.
// (A bound from a sample of the tensor spares most of the first pass's additions, but its own pass costs more, at every
// size.)
constexpr int PCT_BINS = 2048;
// What is selected on: the bits of a key, and a group of eight values as fetched, with keys() for NaN as 0
template <typename T>
struct PctKey;
template <>
struct PctKey<float> {
    static constexpr int BITS = 31, PASSES = 3;
    __device__ static float value(uint32_t key) { return __uint_as_float(key); }
    struct Group {
        float4 a, b;
        __device__ __forceinline__ void load(const float *p)
        {
            a = *reinterpret_cast<const float4 *>(p);
            b = *reinterpret_cast<const float4 *>(p + 4);
        }
        __device__ __forceinline__ void keys(uint32_t (&k)[8]) const
        {
            const float v[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
            for (int e = 0; e < 8; ++e) k[e] = (v[e] != v[e]) ? 0u : (__float_as_uint(v[e]) & 0x7FFFFFFFu);
        }
    };
};
template <>
struct PctKey<__half> {
    static constexpr int BITS = 21, PASSES = 2;
    __device__ static float value(uint32_t key) { return half_bits_to_float((uint16_t)(key >> 6)); }
    struct Group {
        uint4 a;
        __device__ __forceinline__ void load(const __half *p) { a = *reinterpret_cast<const uint4 *>(p); }
        __device__ __forceinline__ void keys(uint32_t (&k)[8]) const
        {
            const uint32_t w[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const uint32_t h = (e & 1) ? (w[e >> 1] >> 16) & 0x7FFFu : w[e >> 1] & 0x7FFFu;
                k[e] = h > 0x7C00u ? 0u : h << 6;
            }
        }
    };
};
// Patterns of two binary16 values without their signs
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ u16x2 magnitudes(uint32_t w) { return __builtin_bit_cast(u16x2, w & 0x7FFF7FFFu); }
// bits of a key below the digit of a pass
template <typename T>
constexpr int pct_shift(int pass) { return PctKey<T>::BITS - 11 - 10 * pass; }

struct PctWorkspace {
    uint32_t hist[3][PCT_BINS];
    uint32_t prefix;  // bits fixed so far
    uint32_t k;       // rank still to find inside the prefix
    uint32_t done;    // workgroups of the running pass that have added their counts
    uint32_t pad;
};

__device__ __forceinline__ uint32_t load_agent(const uint32_t *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// One workgroup, of which 256 threads own bins.  PASS 0 starts from rank k0; the later passes from the rank left over.
// Thread t owns PER consecutive bins; the thread whose bins hold the k-th largest (fewer
// than k elements in the bins above its own, at least k from its lowest bin up) fixes
// the digit.  After the last pass the prefix is the whole key of T and the step
// T / qmax is written.  scratch: 272 words of LDS.
template <typename KT, int PASS>
__device__ __forceinline__ void percentile_select(PctWorkspace *__restrict__ ws, uint32_t k0, float qmax,
                                                  float *__restrict__ s_out, uint32_t *scratch)
{
    constexpr int NB = PASS == 0 ? 2048 : 1024;
    constexpr int PER = NB / 256;
    uint32_t *const chunk = scratch, *const group = scratch + 256;
    const int t = threadIdx.x;
    const bool owner = t < 256;
    uint32_t mine[PER], sum = 0;
    if (owner) {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            mine[i] = load_agent(&ws->hist[PASS][t * PER + i]);
            sum += mine[i];
        }
        chunk[t] = sum;
    }
    const uint32_t k = PASS ? ws->k : k0;
    const uint32_t old_prefix = PASS ? ws->prefix : 0u;
    __syncthreads();
    if (t < 16) {
        uint32_t gs = 0;
#pragma unroll
        for (int u = 0; u < 16; ++u) gs += chunk[16 * t + u];
        group[t] = gs;
    }
    __syncthreads();
    if (!owner) return;
    // elements in the bins above this thread's: later threads of its group of 16, later groups
    uint32_t above = 0;
#pragma unroll
    for (int u = 1; u < 16; ++u) above += ((t & 15) + u < 16) ? chunk[t + u] : 0u;
#pragma unroll
    for (int g = 1; g < 16; ++g) above += ((t >> 4) + g < 16) ? group[(t >> 4) + g] : 0u;
    if (above < k && above + sum >= k) {
        uint32_t cum = above;
        int b = 0;  // the lowest bin is taken when none above it reaches k
        bool found = false;
#pragma unroll
        for (int i = PER - 1; i > 0; --i) {
            if (!found) {
                if (cum + mine[i] >= k) {
                    found = true;
                    b = i;
                } else {
                    cum += mine[i];
                }
            }
        }
        const uint32_t prefix = PASS == 0 ? (uint32_t)(t * PER + b) : ((old_prefix << 10) | (uint32_t)(t * PER + b));
        ws->prefix = prefix;
        ws->k = k - cum;
        if (PASS == PctKey<KT>::PASSES - 1) {
            const float tv = PctKey<KT>::value(prefix);
            s_out[0] = (tv > 0.0f) ? tv / qmax : 1.0f;
        }
    }
}

// Four copies of the counts, chosen by lane % 4: activations pile up in a few dozen bins
// (a binade of binary32 is 8 bins of pass 0), and lanes of one LDS atomic that hit the same counter
// are served one after the other.
// (workgroups of 1024 threads: a quarter of the atomic additions on the few bins that all of them hit)
template <typename T, int PASS, bool CONTIG>
__global__ __launch_bounds__(CAL_THREADS) void percentile_hist_kernel(const T *__restrict__ x, int64_t M, int64_t K,
                                                              int64_t ldx, PctWorkspace *__restrict__ ws, uint32_t k0,
                                                              float qmax, float *__restrict__ s_out)
{
    constexpr int COPIES = 4;  // interleaved, so the copies of one bin sit in different banks
    __shared__ uint32_t h[PCT_BINS * COPIES];
    for (int i = threadIdx.x; i < COPIES * PCT_BINS; i += CAL_THREADS) h[i] = 0u;
    __syncthreads();
    uint32_t *const mine = h + (threadIdx.x & (COPIES - 1));
    const uint32_t prefix = PASS ? ws->prefix : 0u;
    const int64_t groups_per_row = K / 8;
    const int64_t total = M * groups_per_row;
    using Group = typename PctKey<T>::Group;
    constexpr int SHIFT = pct_shift<T>(PASS);
    for_each_group<Group, T, CONTIG, sizeof(T) == 2 ? 8 : 4, sizeof(T) == 2>(x, total, groups_per_row, ldx, [&](const Group &g) {
        if constexpr (sizeof(T) == 2) {
            // Binary16, where vector issue and not memory was the bound: eight patterns are looked at in four words, and the general
            // way is left for groups in which one of them may need it.  16384 x 4096 values, us under the tracer, every key by itself ->
            // this: first pass 28.2 -> 26.7 (then bound by the additions in LDS), second 26.6 -> 23.5 (by memory).
            const uint32_t w[4] = {g.a.x, g.a.y, g.a.z, g.a.w};
            if (PASS == 0) {
                // infinities and NaN, whose patterns share a digit
                const u16x2 top = __builtin_elementwise_max(__builtin_elementwise_max(magnitudes(w[0]), magnitudes(w[1])),
                                                            __builtin_elementwise_max(magnitudes(w[2]), magnitudes(w[3])));
                if (__builtin_expect(max(top.x, top.y) < 0x7C00u, 1)) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) atomicAdd(&mine[((w[e >> 1] >> (4 + 16 * (e & 1))) & 0x7FFu) * COPIES], 1u);
                    return;
                }
            } else {
                // a pattern has the digit found so far if it is less than 16 past the digit's first one (of digit 0 are the NaN, too)
                const u16x2 first = (uint16_t)(prefix << 4);
                const u16x2 past = __builtin_elementwise_min(__builtin_elementwise_min(magnitudes(w[0]) - first, magnitudes(w[1]) - first),
                                                             __builtin_elementwise_min(magnitudes(w[2]) - first, magnitudes(w[3]) - first));
                if (__builtin_expect(prefix != 0u && min(past.x, past.y) >= 16u, 1)) return;
            }
        }
        uint32_t key[8];
        g.keys(key);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            if (PASS == 0) {
                atomicAdd(&mine[(key[e] >> SHIFT) * COPIES], 1u);
            } else {
                if ((key[e] >> (SHIFT + 10)) == prefix) atomicAdd(&mine[((key[e] >> SHIFT) & 1023u) * COPIES], 1u);
            }
        }
    });
    __syncthreads();
    for (int i = threadIdx.x; i < PCT_BINS; i += CAL_THREADS) {
        const uint32_t c = (h[4 * i] + h[4 * i + 1]) + (h[4 * i + 2] + h[4 * i + 3]);
        if (c) atomicAdd(&ws->hist[PASS][i], c);
    }
    // the last workgroup to get here selects the digit: its ticket is drawn after every wave's counts have
    // reached memory (the counts and the ticket are agent-scope atomics), nobody waits for anybody
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) {
        const uint32_t old = __hip_atomic_fetch_add(&ws->done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        h[0] = old == gridDim.x - 1;
        if (old == gridDim.x - 1) __hip_atomic_store(&ws->done, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    if (h[0] != 0u) percentile_select<T, PASS>(ws, k0, qmax, s_out, h + 64);
}

static inline int stream_grid(int64_t items, int threads, int max_blocks)
{
    int64_t b = ceil_div(items, threads);
    if (b < 1) b = 1;
    if (b > max_blocks) b = max_blocks;
    return (int)b;
}

}  // namespace mkq

using namespace mkq;

static int check_tensor(const void *x, int x_dtype, int64_t M, int64_t K, int64_t ldx)
{
    if (x_dtype != MKQ_F32 && x_dtype != MKQ_F16) return MKQ_ERR_DTYPE;
    if (M <= 0 || K <= 0 || (K % 8) != 0 || ldx < K || (ldx % 8) != 0) return MKQ_ERR_SHAPE;
    if (!x) return MKQ_ERR_NULL;
    if (!aligned16(x)) return MKQ_ERR_ALIGN;
    return MKQ_OK;
}

extern "C" int mkq_scale_gradients(const void *x, int x_dtype, int64_t M, int64_t K, int64_t ldx, float s, int bits,
                                   double *g_out, void *stream)
{
    const int rc = check_tensor(x, x_dtype, M, K, ldx);
    if (rc != MKQ_OK) return rc;
    if (bits != 4 && bits != 8) return MKQ_ERR_DTYPE;
    if (!scale_ok(s)) return MKQ_ERR_SCALE;
    if (!g_out) return MKQ_ERR_NULL;
    if (reinterpret_cast<uintptr_t>(g_out) & 7u) return MKQ_ERR_ALIGN;
    hipStream_t st = as_stream(stream);
    zero_words_kernel<<<1, 64, 0, st>>>((uint32_t *)g_out, 4);
    const int threads = gradient_threads(M * (K / 8));
    const int grid = stream_grid(M * (K / 8), threads, 256);
#define MKQ_SG(T, B)                                                                                             \
    if (ldx == K) scale_gradients_kernel<T, B, true><<<grid, threads, 0, st>>>((const T *)x, M, K, ldx, s, g_out); \
    else scale_gradients_kernel<T, B, false><<<grid, threads, 0, st>>>((const T *)x, M, K, ldx, s, g_out)
    if (x_dtype == MKQ_F32) {
        if (bits == 4) { MKQ_SG(float, 4); } else { MKQ_SG(float, 8); }
    } else {
        if (bits == 4) { MKQ_SG(__half, 4); } else { MKQ_SG(__half, 8); }
    }
#undef MKQ_SG
    return launch_status();
}

extern "C" size_t mkq_percentile_scale_workspace_bytes(void) { return sizeof(PctWorkspace); }

extern "C" int mkq_percentile_scale(const void *x, int x_dtype, int64_t M, int64_t K, int64_t ldx, int64_t top_ppm,
                                    int bits, float *s_out, void *workspace, size_t workspace_bytes, void *stream)
{
    const int rc = check_tensor(x, x_dtype, M, K, ldx);
    if (rc != MKQ_OK) return rc;
    if (bits != 4 && bits != 8) return MKQ_ERR_DTYPE;
    if (top_ppm < 0 || top_ppm > 1000000) return MKQ_ERR_SHAPE;
    if (!s_out) return MKQ_ERR_NULL;
    if (reinterpret_cast<uintptr_t>(s_out) & 3u) return MKQ_ERR_ALIGN;
    if (!workspace || workspace_bytes < sizeof(PctWorkspace) || !aligned16(workspace)) return MKQ_ERR_WORKSPACE;
    const int64_t n = M * K;
    if (n > 0xFFFFFFFFLL) return MKQ_ERR_UNSUPPORTED;  // 32-bit counts
    int64_t k = n * top_ppm / 1000000;
    if (k < 1) k = 1;
    const float qmax = bits == 4 ? 7.0f : 127.0f;
    PctWorkspace *ws = (PctWorkspace *)workspace;
    hipStream_t st = as_stream(stream);
    constexpr int words = (int)(sizeof(PctWorkspace) / 4);
    zero_words_kernel<<<(words + 255) / 256, 256, 0, st>>>((uint32_t *)ws, words);
    const int grid = stream_grid(M * (K / 8), CAL_THREADS, 256 * 2);  // all resident at once
#define MKQ_HIST(T, P, C) percentile_hist_kernel<T, P, C><<<grid, CAL_THREADS, 0, st>>>((const T *)x, M, K, ldx, ws, (uint32_t)k, qmax, s_out)
#define MKQ_PASS(T, P)                                                    \
    if (ldx == K) { MKQ_HIST(T, P, true); } else { MKQ_HIST(T, P, false); }
    if (x_dtype == MKQ_F32) {
        MKQ_PASS(float, 0);
        MKQ_PASS(float, 1);
        MKQ_PASS(float, 2);
    } else {
        MKQ_PASS(__half, 0);
        MKQ_PASS(__half, 1);
    }
#undef MKQ_PASS
#undef MKQ_HIST
    return launch_status();
}
