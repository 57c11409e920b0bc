// The linear of a few sentences with float activations, in one launch: a workgroup quantizes the 32 tokens of its tile
// into LDS and multiplies them there (the workgroups of the first channel tile also leave the codes in the caller's
// workspace, where the quantizer's own launch puts them).
//
// What bounds this call is launches and trips to memory, not work: as two launches (quantizer, GEMM) M = 128, K = N =
// 768 took 3.0 + 5.7 us of kernels and 14 us from call to call.  Every workgroup of a token tile quantizes the same rows
// again, ceil(N / 32) times in all, which is why the route ends where that re-reading would cost more than a launch
// (small_quantizing_ok).  The weight fragments are fetched first, so their trip overlaps the quantizer's.
#include <type_traits>

#include "gemm_i4_params.h"

namespace mkq {

struct SmallCfg {
    static constexpr int BM = 32, BN = 32, WTM = 32, WTN = 32, TM = 1, TN = 1;
    static constexpr int THREADS = 512, WAVES = 8;
    static constexpr int UNITS = 2;  // 64-code pieces of a weight row per wave, at most (K <= 1024)
    static constexpr int RED_BYTES = WAVES * 64 * 16 * 4;
};
static inline size_t small_lds(int64_t K)
{
    const size_t codes = 32 * ((size_t)K / 2 + 16);
    return codes > (size_t)SmallCfg::RED_BYTES ? codes : (size_t)SmallCfg::RED_BYTES;
}

// AHEAD: groups of eight values that a thread fetches before it uses the first.
template <typename T, int AHEAD, class Epi>
__global__ __launch_bounds__(SmallCfg::THREADS) void gemm_i4_small_kernel(const GemmI4Params p, const T *__restrict__ x,
                                                                           uint8_t *__restrict__ codes_out)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int fr = lane & 31, fh = lane >> 5;
    const int tiles_m = (p.M + 31) / 32;
    const int m0 = (int)(blockIdx.x % tiles_m) * 32, n0 = (int)(blockIdx.x / tiles_m) * 32;
    const int row_bytes = p.K / 2, units = p.K / 64;
    const int pitch = row_bytes + 16;  // LDS row of codes; 16 bytes more so that the rows of a fragment spread over the banks

    int wrow = n0 + w_row_perm(fr);
    wrow = wrow < p.N ? wrow : p.N - 1;  // rows past the edge are never stored
    const uint8_t *wp = p.W + (size_t)wrow * row_bytes + fh * 16;
    uint4 fw[SmallCfg::UNITS];
#pragma unroll
    for (int i = 0; i < SmallCfg::UNITS; ++i) {
        const int u = wave + i * SmallCfg::WAVES;
        if (u < units) fw[i] = *reinterpret_cast<const uint4 *>(wp + u * 32);
    }

    // quantize the tile's rows, eight values per thread and turn.  Rows past the edge stay as the LDS happens to hold
    // them: they are only multiplied into sums that are never stored (with the last row in their place, M = 1, K = N =
    // 1024 took 6.5 us, two launches 5.5; now 3.9).
    const QuantStep qs = quant_step<4>(p.s_x);
    const int gpr = p.K / 8, rows = p.M - m0 < 32 ? p.M - m0 : 32, total = rows * gpr;
    auto batch = [&](int g0, auto whole) {
        float v[AHEAD][8];
        int at[AHEAD], to[AHEAD];
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) {
            const int g = g0 + i * SmallCfg::THREADS;
            if (!whole.value && g >= total) break;
            const int r = g / gpr, c = g - r * gpr;
            at[i] = r * pitch + c * 4;
            to[i] = (m0 + r) * row_bytes + c * 4;
            load8<T>(x + (size_t)(m0 + r) * p.K + c * 8, v[i]);
        }
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) {
            if (!whole.value && g0 + i * SmallCfg::THREADS >= total) break;
            const uint32_t codes = quantize8<4>(v[i], qs).x;
            *reinterpret_cast<uint32_t *>(smem + at[i]) = codes;
            if (n0 == 0) *reinterpret_cast<uint32_t *>(codes_out + to[i]) = codes;
        }
    };
    // Whole batches carry no checks (with them in every batch, binary16, K = N =
    // 768, M = 64 took 5.6 us instead of 5.3, K = N = 1024 6.3 instead of 6.0).
    int g0 = tid;
    for (int last = (AHEAD - 1) * SmallCfg::THREADS; g0 + last < total; g0 += AHEAD * SmallCfg::THREADS) batch(g0, std::true_type());
    for (; g0 < total; g0 += AHEAD * SmallCfg::THREADS) batch(g0, std::false_type());
    __syncthreads();

    v16i acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0;
#pragma unroll
    for (int i = 0; i < SmallCfg::UNITS; ++i) {
        const int u = wave + i * SmallCfg::WAVES;
        if (u < units) {
            const uint4 fa = *reinterpret_cast<const uint4 *>(smem + fr * pitch + u * 32 + fh * 16);
            acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(widen(fw[i].x, fw[i].y), widen(fa.x, fa.y), acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(widen(fw[i].z, fw[i].w), widen(fa.z, fa.w), acc, 0, 0, 0);
        }
    }
    __syncthreads();  // the codes are read: their area takes the partial sums

    int4 *const red = reinterpret_cast<int4 *>(smem);  // [wave][4][64 lanes]
#pragma unroll
    for (int q = 0; q < 4; ++q) red[(wave * 4 + q) * 64 + lane] = make_int4(acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]);
    __syncthreads();
    if (wave == 0) {
        v16i sum[1][1];
#pragma unroll
        for (int v = 0; v < 16; ++v) sum[0][0][v] = acc[v];
#pragma unroll
        for (int w = 1; w < SmallCfg::WAVES; ++w)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int4 t = red[(w * 4 + q) * 64 + lane];
                sum[0][0][4 * q] += t.x; sum[0][0][4 * q + 1] += t.y;
                sum[0][0][4 * q + 2] += t.z; sum[0][0][4 * q + 3] += t.w;
            }
        gemm_i4_epilogue<SmallCfg, Epi>(p, sum, m0, n0, 0, 0, fr, fh);
    }
}

// At most one tile per CU and rows that a thread fetches in one go.  Kernel times inside a graph, us, two launches ->
// one: K = 768, N = 768, binary32, M = 1 / 16 / 64 / 128 / 256 5.3 -> 3.7, 6.1 -> 4.6, 7.0 -> 5.9, 7.4 -> 5.8, 7.5 -> 6.0;
// binary16 M = 256 7.2 -> 5.9; N = 3072, M = 64 7.1 -> 5.9; K = 1024, N = 1024, M = 1 / 8 / 32 5.6 -> 3.9, 6.2 -> 4.4, 6.8 -> 6.6;
// K = 1024, N = 8192, M = 32, the least favourable, 6.8 -> 6.9.  With two tiles per CU (M = 384, N = 768) 7.4 -> 10.1; with K = 3072 9.7 -> 14.0.
constexpr int64_t SMALL_MAX_TILES = 256, SMALL_MAX_K = 1024;

// Whether the one-launch route takes a linear with activations a of the given element size.
bool small_quantizing_ok(const GemmI4Params &p, const void *a, int elem_bytes)
{
    if ((p.K % 64) != 0 || p.K > SMALL_MAX_K) return false;
    const int64_t tiles = ceil_div(p.M, 32) * ceil_div(p.N, 32);
    if (tiles > SMALL_MAX_TILES) return false;
    // an output that overlaps the activations would be written while other workgroups still read them, one that
    // overlaps the workspace while others still leave their codes there (the quantizer as a launch of its own has
    // read and written everything before)
    auto apart = [](const void *q, int64_t q_bytes, const void *r, int64_t r_bytes) {
        const uintptr_t q0 = reinterpret_cast<uintptr_t>(q), r0 = reinterpret_cast<uintptr_t>(r);
        return !q || q0 + (uintptr_t)q_bytes <= r0 || r0 + (uintptr_t)r_bytes <= q0;
    };
    const int64_t a_bytes = (int64_t)p.M * p.K * elem_bytes, code_bytes = (int64_t)p.M * p.K / 2;
    auto untouched = [&](const void *q, int64_t bytes) { return apart(q, bytes, a, a_bytes) && apart(q, bytes, p.A, code_bytes); };
    const int64_t pitch = p.q_pitch ? p.q_pitch : p.N;
    const int64_t out_bytes = p.out_dtype == MKQ_I4 ? p.M * pitch / 2 : (int64_t)p.M * p.N * (p.out_dtype == MKQ_F32 ? 4 : 2);
    return apart(p.A, code_bytes, a, a_bytes) && untouched(p.out, out_bytes) && untouched(p.q_out, p.M * pitch / 2) &&
           untouched(p.acc_out, (int64_t)p.M * p.N * 4);
}

int run_gemm_i4_small(const GemmI4Params &p, const void *a, int a_dtype, hipStream_t st)
{
    const unsigned grid = (unsigned)(ceil_div(p.M, 32) * ceil_div(p.N, 32));
    const size_t lds = small_lds(p.K);
    uint8_t *const codes = const_cast<uint8_t *>(p.A);
    // K = 768 is six groups per thread, K = 1024 eight: everything in flight at once, nothing fetched twice
#define MKQ_SMALL(T, AHEAD)                                                                                                   \
    if (tail) gemm_i4_small_kernel<T, AHEAD, EpiGeluTail><<<grid, SmallCfg::THREADS, lds, st>>>(p, (const T *)a, codes);     \
    else gemm_i4_small_kernel<T, AHEAD, EpiGeneric><<<grid, SmallCfg::THREADS, lds, st>>>(p, (const T *)a, codes)
    const bool tail = epi_gelu_tail(p.act, p.out_dtype);
    if (a_dtype == MKQ_F32) {
        if (p.K <= 768) { MKQ_SMALL(float, 6); } else { MKQ_SMALL(float, 8); }
    } else {
        if (p.K <= 768) { MKQ_SMALL(__half, 6); } else { MKQ_SMALL(__half, 8); }
    }
#undef MKQ_SMALL
    return launch_status();
}

}  // namespace mkq
