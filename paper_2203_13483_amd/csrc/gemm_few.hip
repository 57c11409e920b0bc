// The 4- and 8-bit linears of few tokens, and small linears altogether: calls that are over before the persistent tile kernels have
// got going.
//
// What bounds them is trips to memory and the instructions of the longest chain, not bandwidth and not the matrix cores: in a tile
// kernel a lone wave takes 0.45-0.55 us per 128-byte stage, six times the products themselves, and loads in the operand layout, sixteen
// rows in sixteen neighbouring lanes, come at 16 bytes per cycle and CU.  Here a workgroup of eight waves owns 16 * NT channels of
// 16 * MT tokens; the waves share K by PB-byte pieces of the rows, and each copies the pieces of its weight and activation rows into
// LDS of its own (whole lines, 40-50 bytes per cycle and CU) and multiplies them: no wave waits for another before the partial sums
// meet in LDS, and as many waves as the tile has blocks of 32 tokens x 16 channels run the epilogue.  A second piece in flight per
// wave (twice the LDS, half the workgroups per CU) gained nothing at any size.
// us of a launch, before -> here (before: operands straight from memory to registers up to 64 tokens, then 64x64 tiles):
// M = 16, K = N = 4096 6.5 -> 3.3; M = 64 9.0 -> 4.5; M = 16, K = 768, N = 30522 17.5 -> 6.0; M = 1, K = N = 8192 9.0 -> 7.4; with a
// residual at M = 440, N = 768, K = 768 5.1 -> 3.4, K = 3072 7.6 -> 5.1.
#include "gemm_i4_params.h"

namespace mkq {

// The epilogue of 32 tokens x 16 channels
struct FewCfg {
    static constexpr int BM = 32, BN = 16, WTM = 32, WTN = 32, TM = 1, TN = 1, HALVES = 1;
};
// PB: bytes of a row that a wave takes at a time
template <int NT, int MT, int PB>
struct FewLds {
    static constexpr int PIECE = (NT + MT) * 16 * PB;
    static constexpr int SUMS = NT * MT * 1024;  // a wave's partial sums take the place of its piece
    static constexpr int WAVE = PIECE > SUMS ? PIECE : SUMS, BYTES = 8 * WAVE;
    static_assert(BYTES <= 160 * 1024, "LDS is 160 KiB per CU");
};

template <int NT, int MT, int PB, int BITS, class Epi>
__global__ __launch_bounds__(512) void gemm_few_kernel(const GemmI4Params p)
{
    using L = FewLds<NT, MT, PB>;
    extern __shared__ __attribute__((aligned(16))) uint8_t smem_all[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    uint8_t *const smem = smem_all + wave * L::WAVE;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)smem;
    FewPlace at = {(int)blockIdx.x, (int)blockIdx.y};
    if (p.group_m) at = few_place(blockIdx.x, gridDim.x, {(unsigned)p.group_m, (unsigned)p.ks, p.by_rows});
    const int n0 = at.channels * (16 * NT), m0 = at.tokens * (16 * MT);
    const uint32_t row_bytes = (uint32_t)p.K / 8 * BITS;
    const int pieces = (int)(row_bytes / PB);
    const int g0 = pieces * wave / 8, n = pieces * (wave + 1) / 8 - g0;  // this wave's share

    // A copy fills 1024 / PB rows.  16-byte parts are XOR-swizzled with the row on the global side, so that sixteen rows of one
    // part spread over the banks.  Rows past the edge re-read the last one: their sums are never stored.
    constexpr int RPC = 1024 / PB, PARTS = PB / 16, CW = NT * 16 / RPC, C = (NT + MT) * 16 / RPC;
    auto swizzle = [](int r) { return PB == 128 ? r & 7 : (r >> 1) & 3; };
    uint32_t goff[C];
    const int c_row = lane / PARTS, c_part = ((lane % PARTS) ^ swizzle(c_row)) * 16;
    const uint8_t *w_k = p.W + (size_t)n0 * row_bytes + (size_t)g0 * PB, *a_k = p.A + (size_t)m0 * row_bytes + (size_t)g0 * PB;
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const int limit = c < CW ? p.N - n0 : p.M - m0;
        int r = (c < CW ? c : c - CW) * RPC + c_row;
        r = r < limit ? r : limit - 1;
        goff[c] = (uint32_t)r * row_bytes + c_part;
    }
    auto fetch = [&]() {
        static_for<C>([&](auto cc) {
            constexpr int c = decltype(cc)::value;
            dma_copy16<c * 1024>(c < CW ? w_k : a_k, goff[c], lds0);
        });
        w_k += PB;
        a_k += PB;
    };
    if (n > 0) fetch();

    // the epilogue's scales, biases and residual are first touched here, by the waves that will run it
    const int fr = lane & 31, fh = lane >> 5;
    constexpr int UNITS = (MT + 1) / 2;  // blocks of 32 tokens
    static_assert(UNITS * NT <= 8, "a wave for every block of 32 tokens x 16 channels");
    const int unit = wave / NT, ut = wave % NT;
    float touched = 0.0f;
    if (wave < UNITS * NT) {
        const int c = n0 + ut * 16 + (lane & 15), cn = c < p.N ? c : p.N - 1;
        touched = p.s_w[cn] + (p.bias ? p.bias[cn] : 0.0f);
        const int m = m0 + unit * 32 + fr, cr = n0 + ut * 16;
        if (p.residual && m < p.M && cr < p.N) {
            const size_t o = (size_t)m * p.N + cr;
            touched += p.residual_dtype == MKQ_F32 ? ((const float *)p.residual)[o] : (float)((const uint16_t *)p.residual)[o];
        }
    }

    v4i acc[NT][MT];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int j = 0; j < MT; ++j) acc[t][j] = v4i{0, 0, 0, 0};
    constexpr int H = PB / 64;
    const int row = lane & 15, quarter = lane >> 4;
    int rd[H];
#pragma unroll
    for (int h = 0; h < H; ++h) rd[h] = row * PB + (((4 * h + quarter) ^ swizzle(row)) * 16);
    // Which codes of a piece a lane holds does not matter to the product as long as weights and activations agree.
    auto multiply = [&]() {
#pragma unroll
        for (int h = 0; h < H; ++h) {
            uint4 w[NT], a[MT];
#pragma unroll
            for (int t = 0; t < NT; ++t) w[t] = *reinterpret_cast<const uint4 *>(smem + t * 16 * PB + rd[h]);
#pragma unroll
            for (int j = 0; j < MT; ++j) a[j] = *reinterpret_cast<const uint4 *>(smem + (NT + j) * 16 * PB + rd[h]);
            if constexpr (BITS == 8) {
#pragma unroll
                for (int t = 0; t < NT; ++t)
#pragma unroll
                    for (int j = 0; j < MT; ++j)
                        acc[t][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(__builtin_bit_cast(v4i, w[t]), __builtin_bit_cast(v4i, a[j]), acc[t][j], 0, 0, 0);
            } else {
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    v4i ww[NT], aa[MT];
#pragma unroll
                    for (int t = 0; t < NT; ++t) ww[t] = q ? widen(w[t].z, w[t].w) : widen(w[t].x, w[t].y);
#pragma unroll
                    for (int j = 0; j < MT; ++j) aa[j] = q ? widen(a[j].z, a[j].w) : widen(a[j].x, a[j].y);
#pragma unroll
                    for (int t = 0; t < NT; ++t)
#pragma unroll
                        for (int j = 0; j < MT; ++j) acc[t][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ww[t], aa[j], acc[t][j], 0, 0, 0);
                }
            }
        }
    };
    for (int g = 0; g < n; ++g) {
        wait_vmcnt<0>();
        multiply();
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): the piece has been read
        if (g + 1 < n) fetch();
    }
    asm volatile("" ::"v"(touched) : "memory");  // (keeps the early loads, and the sums below behind the last piece)

    // partial sums: lane l of a 16x16 tile holds channels 4 * (l / 16) .. + 3 of token l % 16
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int j = 0; j < MT; ++j) reinterpret_cast<v4i *>(smem)[(t * MT + j) * 64 + lane] = acc[t][j];
    __syncthreads();
    if (wave < UNITS * NT) {
        v16i sum[1][1];
#pragma unroll
        for (int v = 0; v < 16; ++v) sum[0][0][v] = 0;
        const int j = 2 * unit + (fr >> 4);  // token tile
        if (j < MT) {
#pragma unroll
            for (int w = 0; w < 8; ++w)
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const v4i v = reinterpret_cast<const v4i *>(smem_all + w * L::WAVE)[(ut * MT + j) * 64 + (2 * fh + q) * 16 + (fr & 15)];
#pragma unroll
                    for (int e = 0; e < 4; ++e) sum[0][0][4 * q + e] += v[e];
                }
        }
        gemm_i4_epilogue<FewCfg, Epi>(p, sum, m0 + unit * 32, n0 + ut * 16, 0, 0, fr, fh);
    }
}

template <int NT, int MT, int PB, int BITS>
static int launch_few(const GemmI4Params &p, hipStream_t st)
{
    constexpr int lds = FewLds<NT, MT, PB>::BYTES;
    const bool tail = epi_gelu_tail(p.act, p.out_dtype);
    // (the smaller tiles need no setup and do not ask for the device: call to call, 3 tokens, K = N = 768 5.5 us instead of 6.3)
    if constexpr (lds > 65536) {
        static PerDeviceOnce once[2];  // per instantiation
        const int ok = once[tail].get([&]() -> int {
            const void *const kernel = tail ? (const void *)gemm_few_kernel<NT, MT, PB, BITS, EpiGeluTail> : (const void *)gemm_few_kernel<NT, MT, PB, BITS, EpiGeneric>;
            return hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, lds) == hipSuccess ? 1 : -1;
        });
        if (ok <= 0) return MKQ_ERR_HIP;
    }
    if (p.setup_only) return MKQ_OK;
    const int64_t channel_tiles = ceil_div(p.N, 16 * NT), token_tiles = ceil_div(p.M, 16 * MT);
    const FewOrder order = few_order(p.M, p.N, (int64_t)p.K / 8 * BITS, 16 * NT, 16 * MT);
    const dim3 grid = order.inner ? dim3((unsigned)(channel_tiles * token_tiles)) : dim3((unsigned)channel_tiles, (unsigned)token_tiles);
    // (the order goes in the fields of the tile kernels' order: a second argument is 0.1 us of 4.6 on the host, call to call)
    GemmI4Params q = p;
    q.group_m = (int)order.inner; q.ks = (int)order.magic; q.by_rows = order.by_tokens;
    if (tail) gemm_few_kernel<NT, MT, PB, BITS, EpiGeluTail><<<grid, 512, lds, st>>>(q);
    else gemm_few_kernel<NT, MT, PB, BITS, EpiGeneric><<<grid, 512, lds, st>>>(q);
    return launch_status();
}

template <int BITS>
static int launch_few_by_tile(const GemmI4Params &p, FewTile t, hipStream_t st)
{
    switch (t) {
    case FEW_16x16: return launch_few<1, 1, 64, BITS>(p, st);
    case FEW_16x32: return launch_few<1, 2, 64, BITS>(p, st);
    case FEW_32x32: return launch_few<2, 2, 64, BITS>(p, st);
    case FEW_32x64: return launch_few<2, 4, 64, BITS>(p, st);
    case FEW_64x64: return launch_few<4, 4, 64, BITS>(p, st);
    case FEW_16x16_LONG: return launch_few<1, 1, 128, BITS>(p, st);
    case FEW_16x32_LONG: return launch_few<1, 2, 128, BITS>(p, st);
    case FEW_32x32_LONG: return launch_few<2, 2, 128, BITS>(p, st);
    case FEW_32x64_LONG: return launch_few<2, 4, 128, BITS>(p, st);
    case FEW_64x64_LONG: return launch_few<4, 4, 128, BITS>(p, st);
    default: return MKQ_ERR_UNSUPPORTED;
    }
}

int run_gemm_few(const GemmI4Params &p, int bits, FewTile t, hipStream_t st)
{
    return bits == 8 ? launch_few_by_tile<8>(p, t, st) : launch_few_by_tile<4>(p, t, st);
}

int setup_gemm_few()
{
    GemmI4Params p = {};
    p.M = p.N = p.K = 256;
    p.setup_only = true;
    for (int t = FEW_16x16; t <= FEW_64x64_LONG; ++t)
        for (int e = 0; e < 4; ++e) {
            p.out_dtype = e & 1 ? MKQ_F32 : MKQ_F16;
            p.act = e & 1 ? MKQ_ACT_GELU : MKQ_ACT_NONE;
            const int rc = run_gemm_few(p, e & 2 ? 8 : 4, (FewTile)t, nullptr);
            if (rc != MKQ_OK) return rc;
        }
    return MKQ_OK;
}

}  // namespace mkq
